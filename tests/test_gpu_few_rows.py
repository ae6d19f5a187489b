"""The kernel for few rows (waves that split the k range, every step's rows packed into one launch) against the oracle:
each of its tile shapes at the edges of its row tiles, column tiles and k slices, single steps and whole rank steps.

Bounds: fp32 sums of K <= 8192 exact products, about sqrt(K) 2^-24 of the largest partial sum: 1e-5 for fp32 operands
(the benchmark's bound), 1e-5 for bf16 operands too (K <= 4096 here); a bf16 output adds 2^-9 of the element."""
import os

import numpy as np
import pytest
import torch

import oracle
from paper_2604_24013_amd import binding as cf
from paper_2604_24013_amd import inputs
from tests import harness as H

pytestmark = pytest.mark.gpu

SHAPES = ["1x1x1", "1x2x1", "1x4x1", "2x1x1", "2x2x1", "2x4x1", "4x2x1", "4x4x1", "1x2x3", "4x4x2"]   # last: k split over workgroups
ONE_LAUNCH = cf.CF_PERSISTENT | cf.CF_SERIAL


@pytest.fixture
def rows(request):
    """Forces one shape of the kernel (None: its own rule) and registers a workspace for the k split."""
    ws = torch.empty(64 << 20, dtype=torch.uint8, device=H.DEV)
    cf.set_workspace(ws)
    torch.cuda.synchronize()

    def force(shape):
        os.environ.pop("COMMFUSE_ROWS", None)
        if shape is not None:
            os.environ["COMMFUSE_ROWS"] = shape
    yield force
    os.environ.pop("COMMFUSE_ROWS", None)
    torch.cuda.synchronize()
    cf.set_workspace(None)


def _rs(p, mc, n, k, dtype, salt):
    w = inputs.scaled(inputs.CONFIGS["c2_rs_7b"], p=p, m_chunk=mc, n=n, k=k, dtype=dtype)
    data = inputs.make_rs(w, salt=salt)
    ref = oracle.rs_rank_steps(inputs.as_f64(data["A"], dtype), inputs.as_f64(data["W"], dtype),
                               [None] + [r.astype(np.float64) for r in data["R"][1:]], p, p - 1)
    return w, data, ref


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("layout", [cf.CF_W_KN, cf.CF_W_NK])
@pytest.mark.parametrize("dims", [(2, 1, 8, 8), (2, 15, 72, 56), (3, 17, 264, 64), (2, 65, 136, 1096), (2, 33, 520, 4096)])
def test_single_steps(dims, layout, dtype, rows):
    """m_chunk around the row tiles (1, 15, 17, 33, 65), n around the column tiles, k below / at / beyond a slice, and an
    input of small integers bit for bit."""
    p, mc, n, k = dims
    w, data, ref = _rs(p, mc, n, k, dtype, 3)
    wi, di = w, inputs.make_rs(w, salt=4)
    rng = np.random.default_rng(5)
    for name in ("A", "W"):
        v = inputs.small_int_like(di[name].shape, rng)
        di[name] = inputs.f32_to_bf16_bits(v) if dtype == "bf16" else v
    di["R"] = [None] + [inputs.small_int_like(r.shape, rng) for r in di["R"][1:]]
    refi = oracle.rs_rank_steps(inputs.as_f64(di["A"], dtype), inputs.as_f64(di["W"], dtype),
                                [None] + [r.astype(np.float64) for r in di["R"][1:]], p, p - 1)
    for shape in SHAPES + [None]:
        rows(shape)
        outs = H.RsRun(w, data, p - 1, layout).run_steps()
        for i in range(p):
            assert not np.isnan(outs[i]).any()
            assert H.rel_err(outs[i], ref[i]) <= 1e-5, f"{shape} step {i}"
        for got, want in zip(H.RsRun(wi, di, p - 1, layout).run_steps(), refi):
            assert np.array_equal(got, want), shape


@pytest.mark.parametrize("carry", [0, cf.CF_FUSED_COPY])
@pytest.mark.parametrize("layout", [cf.CF_W_KN, cf.CF_W_NK])
@pytest.mark.parametrize("dims", [(8, 1, 40, 72), (4, 9, 264, 520), (6, 22, 136, 200), (2, 64, 200, 8)])
def test_packed_rank_steps(dims, layout, carry, rows):
    """All steps of a rank step in one launch: tiles that hold rows of several steps, the deliveries copied in front or
    landed by the launch, reduce-scatter on the ring and pairwise, all-gather with both output types."""
    p, mc, n, k = dims
    w, data, ref = _rs(p, mc, n, k, "bf16", 6)
    refp = oracle.rs_pair_rank_steps(inputs.as_f64(data["A"], "bf16"), inputs.as_f64(data["W"], "bf16"),
                                     [None] + [r.astype(np.float64) for r in data["R"][1:]], p, p - 1)
    for shape in ("1x2x1", "2x2x1", "4x4x1", "1x4x2", None):
        rows(shape)
        for Run, kw, want in ((H.RsRun, dict(each=True), ref), (H.RsPairRun, dict(keep_all=True), refp)):
            run = Run(w, data, p - 1, layout, **kw)
            for t in run.each + run.send_each + [run.O]:
                t.fill_(float("nan"))
            run.run_schedule(ONE_LAUNCH | carry)
            for i in range(p):
                got = H.to_host_f64(run.send_each[i] if i < p - 1 else run.O)
                assert H.rel_err(got, want[i]) <= 1e-5, f"{Run.__name__} {shape} step {i}"
            assert all(torch.equal(a, b) for a, b in zip(run.each, run.stage)), f"{Run.__name__} {shape}"
        for out_dtype in ("f32", "bf16"):
            wa = inputs.scaled(inputs.CONFIGS["c3_ag_7b"], p=p, m_chunk=mc, n=n, k=k, out_dtype=out_dtype)
            da = inputs.make_ag(wa, salt=7)
            refa = oracle.ag_rank(inputs.as_f64(da["X"], "bf16"), [None] + [inputs.as_f64(s, "bf16") for s in da["S"][1:]],
                                  inputs.as_f64(da["W"], "bf16"), p, p - 1)
            run = H.AgRun(wa, da, p - 1, layout, each=True)
            for t in run.each:
                t.fill_(float("nan"))
            run.run_schedule(ONE_LAUNCH | carry)
            assert H.rel_err(H.to_host_f64(run.O), refa) <= (2.0 ** -8 if out_dtype == "bf16" else 1e-5), shape
            assert all(torch.equal(a, b) for a, b in zip(run.each, run.stage)), shape


@pytest.mark.parametrize("dims", [(4, 9, 264, 520), (4, 272, 1032, 264)])      # all rows in one launch / the tile kernels
def test_peers_buffers_off_the_16_byte_grid(dims, rows):
    """CF_FUSED_COPY with peers' buffers that start 8 bytes (bf16 slices) or 4 bytes (partial sums) off the grid: the
    deliveries land as they are and the sums are those of the copies in front."""
    p, mc, n, k = dims
    rows(None)

    def shifted(t, elems):
        s = torch.empty(t.numel() + 16, dtype=t.dtype, device=t.device)[elems:elems + t.numel()].view(t.shape)
        return s.copy_(t)
    w, data, _ = _rs(p, mc, n, k, "bf16", 8)
    wa = inputs.scaled(inputs.CONFIGS["c3_ag_7b"], p=p, m_chunk=mc, n=n, k=k, out_dtype="f32")
    da = inputs.make_ag(wa, salt=9)
    pair, ag = H.RsPairRun(w, data, 1, keep_all=True), H.AgRun(wa, da, 1, each=True)
    for run, elems, kind in ((pair, 1, cf.CF_KIND_RS_PAIR), (ag, 4, cf.CF_KIND_AG)):
        got = []
        for flags, off in ((0, 0), (cf.CF_FUSED_COPY, elems)):
            stage = [shifted(t, off) for t in run.stage]
            is_ag = run is ag
            bufs = cf.make_buffers(run.X if is_ag else run.A, run.W, run.O, stage, (None, None), (None, None), None, run.each,
                                   None if is_ag else run.send_each)
            for t in run.each + [run.O]:
                t.fill_(float("nan"))
            torch.cuda.synchronize()
            cf.run_schedule(run.desc, kind, bufs, run.cs, run.cs, ONE_LAUNCH | flags)
            run.cs.synchronize()
            assert all(torch.equal(a, b) for a, b in zip(run.each, run.stage))
            got.append(run.O.clone())
        assert torch.equal(got[0], got[1])


def test_fp32_steps_and_packed_rank_steps_leave_the_workspace_alone(rows):
    """A long k range on few tiles: only a single bf16 step may split it through the workspace.  fp32 steps and one-launch
    rank steps may be in flight on streams that share a process-wide workspace."""
    ws = torch.full((32 << 20,), 0x5A, dtype=torch.uint8, device=H.DEV)
    cf.set_workspace(ws)
    torch.cuda.synchronize()
    before = ws.clone()
    w, data, ref = _rs(2, 8, 256, 8192, "f32", 10)
    for got, want in zip(H.RsRun(w, data, 1).run_steps(), ref):
        assert H.rel_err(got, want) <= 1e-5
    w, data, ref = _rs(2, 8, 256, 8192, "bf16", 11)
    run = H.RsRun(w, data, 1, each=True)
    run.run_schedule(ONE_LAUNCH | cf.CF_FUSED_COPY)
    assert H.rel_err(H.to_host_f64(run.O), ref[-1]) <= 2e-5       # (sqrt(2) more than at k = 4096)
    torch.cuda.synchronize()
    assert torch.equal(ws, before)


@pytest.mark.parametrize("flags", [cf.CF_PERSISTENT, cf.CF_PERSISTENT | cf.CF_FUSED_COPY])
@pytest.mark.parametrize("dims", [(4, 9, 264, 520), (8, 2, 72, 4104), (4, 272, 1032, 264)])      # few rows (k not a multiple of 64) / tiles
def test_two_streams_deliver_behind_the_copy_streams_work(dims, flags, rows):
    """One-launch modes on two streams: what the peers deliver is written by work enqueued on the copy stream, behind a
    long kernel there, and the schedule is called without a synchronisation: the new data arrive."""
    p, mc, n, k = dims
    rows(None)
    w, data, ref = _rs(p, mc, n, k, "bf16", 12)
    wa = inputs.scaled(inputs.CONFIGS["c3_ag_7b"], p=p, m_chunk=mc, n=n, k=k, out_dtype="f32")
    da = inputs.make_ag(wa, salt=13)
    refa = oracle.ag_rank(inputs.as_f64(da["X"], "bf16"), [None] + [inputs.as_f64(s, "bf16") for s in da["S"][1:]],
                          inputs.as_f64(da["W"], "bf16"), p, p - 1)
    busy = torch.zeros(1 << 28, device=H.DEV)                # a pass over it takes longer than the whole rank step
    for run, want, kind in ((H.RsRun(w, data, p - 1, each=True), ref[-1], cf.CF_KIND_RS),
                            (H.AgRun(wa, da, p - 1, each=True), refa, cf.CF_KIND_AG)):
        if kind == cf.CF_KIND_RS and flags & cf.CF_FUSED_COPY:
            continue                                         # (packed partial sums are carried by every launch: the copy stream is unused)
        fresh = [t.clone() for t in run.stage]
        for t in run.stage + run.each + [run.O]:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        with torch.cuda.stream(run.xs):
            for _ in range(8):
                busy.add_(1.0)
            for t, f in zip(run.stage, fresh):
                t.copy_(f)
        cf.run_schedule(run.desc, kind, run.bufs, run.cs, run.xs, flags)
        run.cs.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(run.each, fresh))
        assert H.rel_err(H.to_host_f64(run.O), want) <= 1e-5
        for _ in range(3):                                   # captured and replayed, everything synchronised: the same
            for t in run.each + [run.O]:
                t.fill_(float("nan"))
            run.run_schedule(flags | cf.CF_GRAPH)
            assert all(torch.equal(a, b) for a, b in zip(run.each, fresh))
            assert H.rel_err(H.to_host_f64(run.O), want) <= 1e-5


def _which(run):
    """Kernel that a call takes by rule, told by the bits of its result: every kernel sums in an order of its own."""
    out = {}
    for name, v in (("rule", None), ("tiles", "0"), ("rows", "4x4x1")):
        os.environ.pop("COMMFUSE_ROWS", None)
        if v is not None:
            os.environ["COMMFUSE_ROWS"] = v
        try:
            out[name] = run()
        finally:
            os.environ.pop("COMMFUSE_ROWS", None)
    assert not torch.equal(out["tiles"], out["rows"])
    assert H.rel_err(H.to_host_f64(out["tiles"]), H.to_host_f64(out["rows"])) <= 2e-5
    return "tiles" if torch.equal(out["rule"], out["tiles"]) else "rows"


# (rows, n, k, dtype, workspace): the kernel that is the faster one
RULE_STEPS = [
    # a k range that the tile kernel splits through a workspace
    ((384, 4096, 8192, "bf16", True), "tiles"), ((384, 4096, 8192, "bf16", False), "rows"), ((256, 2048, 4096, "bf16", True), "rows"),
    # rows off the 128-byte lines over a long k range, and on them
    ((575, 2080, 7328, "bf16", False), "tiles"), ((575, 2080, 7360, "bf16", False), "rows"),
    ((85, 7512, 6304, "bf16", True), "tiles"), ((85, 7552, 6336, "bf16", True), "rows"), ((85, 1512, 6304, "bf16", True), "rows"),
    # fp32: grids of one round, of several rounds over short and long k ranges, and grids that 128 x 128 tiles fill
    ((1000, 1000, 256, "f32", False), "rows"), ((335, 2328, 160, "f32", False), "tiles"), ((768, 4096, 256, "f32", False), "tiles"), ((512, 4096, 2048, "f32", False), "rows"),
    ((4096, 2048, 512, "f32", False), "tiles"), ((1536, 4096, 1024, "f32", False), "rows"), ((2048, 4096, 1024, "f32", False), "tiles"),
]


@pytest.mark.parametrize("case,want", RULE_STEPS)
def test_rule_for_single_steps(case, want, rows):
    mc, n, k, dtype, workspace = case
    if not workspace:
        cf.set_workspace(None)
    g = torch.Generator(device=H.DEV)
    g.manual_seed(mc + n + k)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    A, W = (torch.empty(s, device=H.DEV).normal_(0.0, 0.5, generator=g).to(dt) for s in ((2 * mc, k), (k, n)))
    recv = torch.empty((mc, n), device=H.DEV).normal_(generator=g)
    desc = cf.layer_desc(2, 0, mc, n, k, dtype, "f32")

    def run():
        out = torch.full((mc, n), float("nan"), device=H.DEV)
        cf.rs_step(desc, 1, A, W, recv, out, None)
        torch.cuda.synchronize()
        return out
    assert _which(run) == want


# p, rows per step, n, k
@pytest.mark.parametrize("dims,want", [((8, 64, 8192, 512), "tiles"), ((8, 64, 8192, 1024), "tiles"), ((4, 128, 4096, 8192), "rows"),
                                       ((2, 96, 8192, 8192), "tiles"), ((8, 8, 1536, 4096), "rows"), ((6, 130, 72, 96), "rows")])
def test_rule_for_packed_rank_steps(dims, want, rows):
    p, mc, n, k = dims
    g = torch.Generator(device=H.DEV)
    g.manual_seed(mc + n + k)
    W, own = (torch.empty(s, device=H.DEV).normal_(0.0, 0.5, generator=g).to(torch.bfloat16) for s in ((k, n), (p * mc, k)))
    stage = [torch.empty((mc, n), device=H.DEV).normal_(generator=g) for _ in range(p - 1)]
    desc = cf.layer_desc(p, 0, mc, n, k, "bf16", "f32")
    st = torch.cuda.Stream()

    def run():
        O, each, sends = torch.empty((mc, n), device=H.DEV), [torch.empty_like(t) for t in stage], [torch.empty_like(t) for t in stage]
        bufs = cf.make_buffers(own, W, O, stage, (None, None), (None, None), None, each, sends)
        torch.cuda.synchronize()
        cf.run_schedule(desc, cf.CF_KIND_RS, bufs, st, st, ONE_LAUNCH | cf.CF_FUSED_COPY)
        st.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(each, stage))
        return torch.cat(sends + [O])
    assert _which(run) == want


@pytest.mark.parametrize("mc", [1, 4, 8])
def test_the_advertised_workspace_takes_the_k_split(mc, rows):
    """commfuse_workspace_bytes covers the partial tiles of a few-rows step whose long k range is split."""
    w, data, ref = _rs(2, mc, 520, 8192, "bf16", 14)
    run = H.RsRun(w, data, 1)
    ws = torch.full((cf.workspace_bytes(run.desc, cf.CF_KIND_RS),), 0xFF, dtype=torch.uint8, device=H.DEV)
    cf.set_workspace(ws)
    for got, want in zip(run.run_steps(), ref):
        assert H.rel_err(got, want) <= 2e-5                       # (sqrt(2) more than at k = 4096)
    assert bool((ws[64 * 1024:] != 0xFF).any())


@pytest.mark.parametrize("carry", [True, False])
def test_padded_rows_carried_and_copied(carry, rows):
    """Row strides beyond the rows, few rows: a delivery that the launch carries lands without the padding of its rows, which
    keeps what it held; COMMFUSE_CARRY=0 has it copied in front, padding and all, also under CF_FUSED_COPY."""
    p, mc, n, k, ldo, lda = 4, 9, 72, 72, 88, 80
    rows(None)
    g = torch.Generator(device=H.DEV)
    g.manual_seed(15)
    rnd = lambda *shape: torch.empty(shape, device=H.DEV).normal_(generator=g)
    nan = lambda *shape, dtype=torch.float32: torch.full(shape, float("nan"), dtype=dtype, device=H.DEV)
    W = rnd(k, n).to(torch.bfloat16)
    st = torch.cuda.Stream()
    if not carry:
        os.environ["COMMFUSE_CARRY"] = "0"
    try:
        A, stage, each = rnd(p * mc, lda).to(torch.bfloat16), [rnd(mc, ldo) for _ in range(p - 1)], [nan(mc, ldo) for _ in range(p - 1)]
        O, sends = nan(mc, ldo), [nan(mc, ldo) for _ in range(p - 1)]
        desc = cf.layer_desc(p, 1, mc, n, k, "bf16", "f32", lda=lda, ldo=ldo)
        bufs = cf.make_buffers(A, W, O, stage, (None, None), (None, None), None, each, sends)
        torch.cuda.synchronize()
        cf.run_schedule(desc, cf.CF_KIND_RS, bufs, st, st, ONE_LAUNCH | cf.CF_FUSED_COPY)
        st.synchronize()
        for j in range(p):
            l = cf.chunk_index(cf.CF_KIND_RS, p, 1, j)
            want = A[l * mc:(l + 1) * mc, :k].double() @ W.double() + (stage[j - 1][:, :n].double() if j else 0.0)
            got = sends[j] if j < p - 1 else O
            assert H.rel_err(H.to_host_f64(got[:, :n]), H.to_host_f64(want)) <= 1e-5
            assert bool(got[:, n:].isnan().all())
        moved = [(each, stage, n)]
        own, stage, each = rnd(mc, lda).to(torch.bfloat16), [rnd(mc, lda).to(torch.bfloat16) for _ in range(p - 1)], \
            [nan(mc, lda, dtype=torch.bfloat16) for _ in range(p - 1)]
        O = nan(p * mc, ldo)
        bufs = cf.make_buffers(own, W, O, stage, (None, None), (None, None), None, each)
        torch.cuda.synchronize()
        cf.run_schedule(desc, cf.CF_KIND_AG, bufs, st, st, ONE_LAUNCH | cf.CF_FUSED_COPY)
        st.synchronize()
        for j in range(p):
            l = cf.chunk_index(cf.CF_KIND_AG, p, 1, j)
            got = O[l * mc:(l + 1) * mc]
            want = (stage[j - 1] if j else own)[:, :k].double() @ W.double()
            assert H.rel_err(H.to_host_f64(got[:, :n]), H.to_host_f64(want)) <= 1e-5
            assert bool(got[:, n:].isnan().all())
        for land, sent, width in moved + [(each, stage, k)]:
            for a, b in zip(land, sent):
                assert torch.equal(a[:, :width], b[:, :width])
                assert bool(a[:, width:].isnan().all()) if carry else torch.equal(a[:, width:], b[:, width:])
    finally:
        os.environ.pop("COMMFUSE_CARRY", None)


@pytest.mark.parametrize("override", ["K_ROTATE=0", "K_ROTATE=1", "XCD_STEPS=0", "XCD_BANDS=1", "STREAM_RECV=0", "PREFETCH=0", "PERSIST_WGS=64",
                                      "MFMA16=0", "DEEP=0", "TILE=128x128"])
def test_overrides_of_the_tile_kernels_keep_a_launch_on_them(override, rows):
    """A rank step that the rule gives to the few-rows kernel, told by its bits: with an override of the tile kernels set it
    runs there."""
    w, data, _ = _rs(8, 9, 264, 1096, "bf16", 16)
    run = H.RsRun(w, data, 1, each=True)

    def result():
        run.run_schedule(ONE_LAUNCH)
        return torch.cat(run.send_each + [run.O]).clone()
    rows(None)
    by_rule = result()
    rows("0")
    tiles = result()
    rows(None)
    name, value = ("COMMFUSE_" + override).split("=")
    os.environ[name] = value
    try:
        got = result()
    finally:
        os.environ.pop(name, None)
    assert not torch.equal(by_rule, tiles)
    assert not torch.equal(got, by_rule)
    assert H.rel_err(H.to_host_f64(got), H.to_host_f64(tiles)) <= 1e-5
