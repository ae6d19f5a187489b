"""Attention in query blocks of 256 and 128: tiles whose scores are all -inf.  Needs an MI355X: run with ``-m gpu``."""
import os

import numpy as np
import pytest
import torch

from paper_2604_24013_amd import binding as cf
from paper_2604_24013_amd import inputs
from tests import harness as H

pytestmark = pytest.mark.gpu

TOL_ATTN = 2.0 ** -7                     # probabilities and output rounded to bf16 (2^-9 each)


def _bf16(x):
    bits = inputs.f32_to_bf16_bits(np.asarray(x, np.float32))
    return H.to_dev(bits, "bf16"), inputs.bf16_bits_to_f32(bits).astype(np.float64)


@pytest.fixture
def variant():
    """Forces 32 * waves queries per workgroup and a number of key splits; yields the registered workspace."""
    ws = torch.empty(16 << 20, dtype=torch.uint8, device=H.DEV)
    cf.set_workspace(ws)
    torch.cuda.synchronize()

    def use(waves, ksplit):
        os.environ.update(COMMFUSE_ATTN_QT={0: "0", 8: "1", 4: "2"}[waves], COMMFUSE_ATTN_KSPLIT=str(ksplit))
        return ws
    yield use
    for v in ("COMMFUSE_ATTN_QT", "COMMFUSE_ATTN_KSPLIT"):
        os.environ.pop(v, None)
    torch.cuda.synchronize()
    cf.set_workspace(None)


def _attend(Qd, Kd, Vd, scale):
    B, h, S, _ = Qd.shape
    out = torch.full((B * S, h * 128), float("nan"), dtype=torch.bfloat16, device=H.DEV)
    cf.attn_slice(cf.attn_desc(1, 0, B, h, S, 128, 64, scale), 0, Qd, Kd, Vd, out, None)
    torch.cuda.synchronize()
    return H.to_host_f64(out)


@pytest.mark.parametrize("waves", [8, 4, 0])
@pytest.mark.parametrize("ksplit,first,last", [
    (1, 0, 64), (1, 0, 512), (1, 192, 320), (1, 960, 1010),          # the first keys, tiles on both buffers, the last
    (2, 512, 576), (3, 320, 448),                                    # the first keys of a split
    (2, 0, 512), (3, 640, 1010)])                                    # all keys of a split
def test_tiles_of_minus_infinity_have_no_weight(variant, waves, ksplit, first, last):
    rng = np.random.default_rng(first + last)
    S, h, scale = 1010, 2, 128 ** -0.5
    variant(waves, ksplit)
    Qd, Q = _bf16(np.abs(rng.standard_normal((1, h, S, 128))) + 0.01)
    K = rng.standard_normal((1, h, S, 128))
    K[:, :, first:last] = -np.inf
    Kd, K = _bf16(K)
    Vd, V = _bf16(rng.standard_normal((1, h, S, 128)))
    got = _attend(Qd, Kd, Vd, scale)
    keep = np.r_[0:first, last:S]
    ref = np.empty_like(got)
    for a in range(h):
        s = Q[0, a] @ K[0, a][keep].T * scale
        P = np.exp(s - s.max(axis=1, keepdims=True))
        ref[:, a * 128:(a + 1) * 128] = P @ V[0, a][keep] / P.sum(axis=1, keepdims=True)
    assert not np.isnan(got).any()
    assert H.rel_err(got, ref) <= TOL_ATTN


@pytest.mark.parametrize("waves", [8, 4])
def test_small_probabilities_add_up_in_the_row_sum(variant, waves):
    """The parked sum of a row, 64 keys of probability 1 and then 64 tiles of 64 keys of 2^-20: a lane adds up half of them, and
    two such keys are half a unit in the last place of its 32.  A pair of tiles adds up by itself first: in the first pair that
    loses the second tile's 2^-15 (sixteen roundings of 2^-19), all others are exact, and so is the sum of the 33 pairs but for
    2^-19 each."""
    S, p, ksplit = 64 * 130, 65, 2
    c, nt = S // p, 64 * waves
    ws = variant(waves, ksplit)
    q, k = np.zeros((1, 1, S, 128)), np.zeros((1, 1, S, 128))
    q[..., 0] = 1.0
    k[0, 0, 64:, 0] = -20.0                                          # scores in units of log2(e): 0, and -20
    Vd, _ = _bf16(np.random.default_rng(3).standard_normal((1, 1, S, 128)))
    out = torch.full((c, 128), float("nan"), dtype=torch.bfloat16, device=H.DEV)
    cf.attn_slice(cf.attn_desc(p, 0, 1, 1, S, 128, 64, float(np.log(2.0))), 0, _bf16(q)[0], _bf16(k)[0], Vd, out, None)
    torch.cuda.synchronize()
    parts = ws[64 << 10:].view(torch.float32)[:ksplit * 66 * nt].view(ksplit, 66, nt).cpu().double()
    used = slice(0, min(nt, 2 * c))                                  # two lanes hold a query
    assert bool((parts[0, 64, used] == 0).all()) and bool((parts[1, 64, used] + 20 < 1e-4).all())   # the references
    assert float((parts[0, 65, used] - (64 + 2.0 ** -8)).abs().max()) <= 2 * (16 + 33) * 2.0 ** -19
    assert bool((parts[1, 65, used] == 65 * 64).all())


@pytest.mark.parametrize("waves", [8, 4])
@pytest.mark.parametrize("ksplit", [1, 2])
@pytest.mark.parametrize("tiles", [2, 5, 8])
def test_references_that_rise_from_tile_to_tile(variant, waves, ksplit, tiles):
    """Scores of query i grow by g_i (in units of log2(e)) from one 64-key tile to the next, in the last by half of that: nine and
    twenty are beyond what the reference may lag behind (eight) and raise it in every tile, from either pair of buffers; three,
    one half and a fall do not by themselves, but share a wave with those that do -- and keep a visible part of every tile.  In the
    second half of the queries every other tile falls back, so that the reference rises in tiles of one pair of buffers only."""
    rng = np.random.default_rng(tiles)
    S = 64 * tiles - 24
    grow = np.array([9.0, 0.5, 3.0, -1.0, 20.0, 0.0, 1.0, 8.5])[np.arange(S) % 8]
    lone = np.arange(S) // 32 % 2 == 1                               # waves in which nothing rises by more than three
    grow[lone] = np.minimum(grow[lone], 3.0)
    tile = np.arange(S) // 64
    step = tile - 0.5 * (tile == tiles - 1)
    q, k = 0.05 * rng.standard_normal((1, 1, S, 128)), rng.standard_normal((1, 1, S, 128))
    q[..., :2], k[..., :2] = 0.0, 0.0
    half = S // 2
    q[0, 0, :half, 0], q[0, 0, half:, 1] = grow[:half], grow[half:]
    k[0, 0, :, 0], k[0, 0, :, 1] = step, np.where(tile % 2 == 0, step, 0.0)
    v = rng.standard_normal((1, 1, S, 128)) + 4.0 * (tile % 3)[None, None, :, None]     # a tile that counts wrongly shows
    variant(waves, ksplit)
    (Qd, Q), (Kd, K), (Vd, V) = _bf16(q), _bf16(k), _bf16(v)
    scale = float(np.float32(np.log(2.0)))
    got = _attend(Qd, Kd, Vd, scale)
    s = Q[0, 0] @ K[0, 0].T * scale
    P = np.exp(s - s.max(axis=1, keepdims=True))
    ref = P @ V[0, 0] / P.sum(axis=1, keepdims=True)
    assert not np.isnan(got).any()
    assert float((np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)).max()) <= TOL_ATTN     # query by query
