"""What a call enqueues -- which kernels, in which grid, and which copies -- read off the library's host code without a GPU."""
import os
import re

import pytest

from paper_2604_24013_amd import binding as cf
from tests.dry import Dry

ONE_LAUNCH = cf.CF_PERSISTENT | cf.CF_SERIAL


def P(i):
    return (i + 1) << 33                              # fake, aligned, far apart


@pytest.fixture(scope="module")
def dry(tmp_path_factory):
    return Dry(str(tmp_path_factory.mktemp("dry")))


@pytest.mark.parametrize("cus", [32, 64, 256])
def test_grids_follow_the_devices_compute_units(dry, monkeypatch, cus):
    monkeypatch.setenv("COMMFUSE_DRY_CUS", str(cus))
    step = cf.layer_desc(1, 0, 4096, 8192, 1024)
    calls = [lambda: cf.ag_step(step, 0, P(0), P(1), P(2)), lambda: cf.rs_step(cf.layer_desc(2, 0, 4096, 8192, 1024), 1, P(0), P(1), P(2), P(3)),
             lambda: cf.wgrad_step(cf.layer_desc(1, 0, 1024, 8192, 4096), 0, P(0), P(1), P(2)),
             lambda: cf.run_schedule(cf.layer_desc(2, 0, 4096, 8192, 1024), cf.CF_KIND_AG,
                                     cf.make_buffers(P(0), P(1), P(2), [P(3)], (None, None), recv_each=[P(4)]), None, None,
                                     ONE_LAUNCH | cf.CF_FUSED_COPY)]
    for call in calls:
        (kernel, grid, block), = dry.calls(call)
        assert kernel.startswith("gemm_bf16_dl_kernel<256, 256,") and (grid, block) == (cus, 512)


def _tables(p):
    return [[P(10 * t + i) for i in range(p - 1)] for t in (1, 3, 5)]


@pytest.mark.parametrize("seq,heads,n", [(8192, 10, 8192), (8192, 8, 8192), (512, 2, 264)])
@pytest.mark.parametrize("pad", [0, 64])
def test_attention_layers_padded_partial_sums_are_copied_in_front(dry, seq, heads, n, pad):
    """A copy lands the padding between the rows of a partial sum, the projection's epilogue does not."""
    p = 8
    stage, each, sends = _tables(p)
    bufs = cf.make_attn_buffers(P(0), P(1), P(2), P(3), P(4), P(5), stage, (None, None), (None, None), None, each, sends)
    desc = cf.attn_desc(p, 1, 1, heads, seq, 128, n, 0.1, ldo=n + pad)
    kernels = [c[0] for c in dry.calls(lambda: cf.run_attn_schedule(desc, bufs, None, None, ONE_LAUNCH | cf.CF_FUSED_COPY))]
    few_rows = kernels[-1].startswith("gemm_rows_kernel")             # (carried without the padding)
    assert ["copy" in k for k in kernels] == ([True, False, False] if pad and not few_rows else [False, False])


@pytest.mark.parametrize("tile,mc,n,k,copied", [
    (None, 512, 8192, 1280, False), (None, 512, 8192, 1152, False), (None, 512, 8192, 1088, True),   # eighteen whole k-tiles and more
    (None, 512, 8192, 1288, False), (None, 512, 8192, 1160, True),                                   # ... twenty with a ragged one
    (None, 200, 232, 1288, True), ("256x256", 200, 232, 1288, False),                                # the override counts
    ("128x128", 512, 8192, 1280, True), ("256x256", 200, 232, 1160, True)])
def test_padded_partial_sums_are_carried_on_large_tiles_over_long_k(dry, monkeypatch, tile, mc, n, k, copied):
    p = 8
    stage, each, sends = _tables(p)
    bufs = cf.make_buffers(P(0), P(1), P(2), stage, (None, None), (None, None), None, each, sends)
    monkeypatch.setenv("COMMFUSE_ROWS", "0")
    if tile:
        monkeypatch.setenv("COMMFUSE_TILE", tile)
    desc = cf.layer_desc(p, 1, mc, n, k, ldo=n + 64)
    kernels = [c[0] for c in dry.calls(lambda: cf.run_schedule(desc, cf.CF_KIND_RS, bufs, None, None, ONE_LAUNCH | cf.CF_FUSED_COPY))]
    assert ["copy" in kern for kern in kernels] == ([True, False] if copied else [False])


def test_kernels_read_every_pointer_of_the_launch_argument():
    """A buffer or flag that a caller may set and no kernel looks at would be ignored in silence."""
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2604_24013_amd", "csrc")
    read = lambda name: re.sub(r"//[^\n]*", "", open(os.path.join(csrc, name)).read())
    struct = re.search(r"struct GemmParams \{(.*?)\n\};", read("cf_internal.h"), re.S)[1]
    pointers = re.findall(r"\*(?:const )?(\w+)(?:\[\w+\])? = ", struct)
    assert {"A", "W", "recv", "out", "wait_flag"} <= set(pointers)
    kernels = read("gemm_bf16_dl.hip") + read("gemm_rows.hip") + read("gemm_f32.hip")
    assert [p for p in pointers if not re.search(rf"\b[Pg]\.{p}\b", kernels)] == []


@pytest.mark.parametrize("mc,n,k,past_the_caches", [
    (4096, 8192, 1024, False), (4096, 8192, 3584, False), (2048, 4096, 1024, True), (2304, 4096, 1024, False),   # 32 MiB of output, and more
    (4096, 7936, 1024, True), (4096, 6144, 1024, True), (4096, 8200, 1024, False),    # rows 31, 24 KiB apart; rows off the lines
    (8192, 8192, 1024, False), (8192, 8192, 3584, True)])                             # 288 MiB and more moved
def test_outputs_stay_in_the_caches_where_rows_lie_16_kib_apart(dry, mc, n, k, past_the_caches):
    shape = lambda p: cf.layer_desc(p, 0, mc, n, k)
    ag, = dry.calls(lambda: cf.ag_step(shape(1), 0, P(0), P(1), P(2)))
    rs, = dry.calls(lambda: cf.rs_step(shape(2), 1, P(0), P(1), P(2), P(3)))
    nt = lambda call: call[0].split(", ")[-1] == "true>"
    assert nt(ag) == past_the_caches
    assert nt(rs) == (n % 32 == 0)                    # with a B_in: wherever rows begin and end on the lines


@pytest.mark.parametrize("add,mc,n,k,tile", [
    (False, 8192, 3072, 1024, "256, 256"),            # 59 us; on 256x128 75
    (False, 4864, 7296, 3136, "256, 256"),            # 224; 233
    (True, 2048, 8192, 1024, "256, 256"),             # whole rounds of whole tiles: 53; 59
    (False, 4992, 7168, 384, "128, 128"),             # few k-tiles: 42; on 256x256 53
    (True, 3712, 6144, 1280, "256, 128"),             # with a B_in, added behind the main loop: 78; on 256x256 90
    (True, 3200, 4992, 8000, "256, 128"),             # 228; 325 (260 tiles of 256x256 on 256 compute units)
])
def test_tile_of_large_steps(dry, add, mc, n, k, tile):
    if add:
        calls = dry.calls(lambda: cf.rs_step(cf.layer_desc(2, 0, mc, n, k, w_layout=cf.CF_W_NK), 1, P(0), P(1), P(2), P(3)))
    else:
        calls = dry.calls(lambda: cf.ag_step(cf.layer_desc(1, 0, mc, n, k, w_layout=cf.CF_W_NK), 0, P(0), P(1), P(2)))
    assert [c[0].startswith(f"gemm_bf16_dl_kernel<{tile},") for c in calls] == [True]


@pytest.mark.parametrize("kind,p,mc,n,k,layout,few_rows", [
    # us on the few-rows kernel and on the tile kernel
    (cf.CF_KIND_RS, 8, 32, 5272, 816, cf.CF_W_KN, False),        # 27; 18
    (cf.CF_KIND_RS, 8, 192, 512, 192, cf.CF_W_KN, False),        # 10.3; 7.7
    (cf.CF_KIND_RS, 2, 80, 4864, 3712, cf.CF_W_KN, True),        # 22; 30
    (cf.CF_KIND_RS, 2, 272, 1152, 2368, cf.CF_W_NK, True),       # 16; 20
    (cf.CF_KIND_AG, 8, 144, 4224, 3328, cf.CF_W_KN, False),      # 111; 62
    (cf.CF_KIND_AG, 4, 80, 3200, 512, cf.CF_W_NK, False),        # 13.1; 8.4
    (cf.CF_KIND_AG, 4, 80, 1408, 640, cf.CF_W_NK, True),         # 7.2; 9.0
    (cf.CF_KIND_AG, 8, 34, 7040, 5096, cf.CF_W_NK, True),        # ragged k-tiles: the tile kernel's deliveries are copied in front
])
def test_rule_between_few_rows_and_tiles_for_rank_steps(dry, kind, p, mc, n, k, layout, few_rows):
    stage, each, sends = _tables(p)
    bufs = cf.make_buffers(P(0), P(1), P(2), stage, (None, None), (None, None), None, each, sends)
    desc = cf.layer_desc(p, p - 1, mc, n, k, w_layout=layout)
    calls = dry.calls(lambda: cf.run_schedule(desc, kind, bufs, None, None, ONE_LAUNCH | cf.CF_FUSED_COPY))
    assert ["gemm_rows_kernel" in c[0] for c in calls] == [few_rows]


@pytest.mark.parametrize("p,mc,n,k", [(4, 72, 136, 1376), (6, 130, 72, 96), (8, 264, 392, 200)])
def test_pairwise_steps_and_rank_steps_take_the_same_kernel(dry, p, mc, n, k):
    """(whose sums are then the same bits)"""
    stage, each, sends = _tables(p)
    bufs = cf.make_buffers(P(0), P(1), P(2), stage, (None, None), (None, None), None, each, sends)
    desc = cf.layer_desc(p, 0, mc, n, k)
    one, = dry.calls(lambda: cf.run_schedule(desc, cf.CF_KIND_RS_PAIR, bufs, None, None, ONE_LAUNCH | cf.CF_FUSED_COPY))
    step, = dry.calls(lambda: cf.rs_pair_step(desc, 0, P(0), P(1), None, None, P(3)))
    assert one[0].startswith("gemm_rows_kernel") and step[0].startswith("gemm_rows_kernel")


@pytest.mark.parametrize("k,pad,off,copied", [(1096, 0, 0, False), (1096, 8, 0, True), (1096, 0, 8, True), (1088, 64, 0, False), (1088, 0, 0, False)])
def test_slices_over_a_ragged_k_range_are_carried(dry, monkeypatch, k, pad, off, copied):
    """... unless a copy would move the padding between their rows, or lies off the 16-byte grid."""
    p = 8
    stage, each, _ = _tables(p)
    stage[2] += off
    bufs = cf.make_buffers(P(0), P(1), P(2), stage, (None, None), (None, None), None, each)
    desc = cf.layer_desc(p, 1, 512, 1536, k, lda=k + pad)
    kernels = [c[0] for c in dry.calls(lambda: cf.run_schedule(desc, cf.CF_KIND_AG, bufs, None, None, ONE_LAUNCH | cf.CF_FUSED_COPY))]
    assert kernels[-1].startswith("gemm_bf16_dl_kernel") and (len(kernels) > 1) == copied


@pytest.mark.parametrize("kind,p,mc,n,k,carried", [
    (cf.CF_KIND_AG, 8, 512, 1536, 1096, True), (cf.CF_KIND_AG, 2, 512, 1536, 4104, True),             # a ragged k range
    (cf.CF_KIND_AG, 8, 8, 1536, 4096, True), (cf.CF_KIND_RS, 8, 8, 4096, 1376, True),                 # few rows
    (cf.CF_KIND_AG, 8, 512, 1536, 1096, False), (cf.CF_KIND_RS, 8, 8, 4096, 1376, False)])
@pytest.mark.parametrize("capturing", [False, True])
def test_the_copy_streams_work_stays_in_order_with_the_deliveries(dry, monkeypatch, kind, p, mc, n, k, carried, capturing):
    """On two streams: what the copy stream holds comes before the kernel that reads the peers' buffers or before the copies on
    that stream, and what is enqueued there later comes after them, whoever delivers.  Under capture the copy stream joins first."""
    if capturing:
        monkeypatch.setenv("COMMFUSE_DRY_CAPTURING", "1")
    compute, copy = 0x10, 0x20
    stage, each, sends = _tables(p)
    bufs = cf.make_buffers(P(0), P(1), P(2), stage, (None, None), (None, None), None, each, sends)
    desc = cf.layer_desc(p, 1, mc, n, k)
    flags = cf.CF_PERSISTENT | (cf.CF_FUSED_COPY if carried else 0)
    seen = dry.order(lambda: cf.run_schedule(desc, kind, bufs, compute, copy, flags))
    launches = [i for i, (op, stream, _) in enumerate(seen) if op == "launch" and stream == compute]
    if not carried:
        assert any(op in ("launch", "copy") and stream == copy for op, stream, _ in seen)
        return
    assert len(launches) == 1 and not any(op in ("launch", "copy") and stream == copy for op, stream, _ in seen)
    handed_over = lambda ops, a, b: any(x[0] == "record" and x[1] == a and ("wait", b, x[2]) in ops[i:] for i, x in enumerate(ops))
    assert handed_over(seen[:launches[0]], copy, compute) and handed_over(seen[launches[0]:], compute, copy)
    assert seen[0][:2] == ("record", compute if capturing else copy) and len(seen) == (7 if capturing else 5)


@pytest.mark.parametrize("p,batch,heads,seq,room,kernel,grid", [
    # keys over waves, 32 queries per workgroup: the only choice without a workspace where query blocks leave a quarter of the chip
    # idle, and with one as many splits as pay and fit
    (1, 1, 1, 64, 0, "keys_over_waves", 2), (4, 2, 3, 1120, 0, "keys_over_waves", 54), (4, 2, 3, 1120, 8, "keys_over_waves", 54 * 3),
    (8, 1, 1, 8192, 8, "keys_over_waves", 32 * 8), (8, 1, 8, 8192, 0, "keys_over_waves", 256), (2, 4, 2, 2362, 1024, "keys_over_waves", 296),
    # query blocks of 256: the chip is full, or their partials fit
    (1, 4, 8, 4096, 0, "slice_kernel<8>", 512), (2, 2, 8, 4638, 1024, "slice_kernel<8>", 160 * 2), (2, 2, 8, 4638, 8, "keys_over_waves", 1168),
    # query blocks of 128, two workgroups per compute unit
    (8, 1, 8, 8192, 1024, "slice_kernel<4>", 64 * 8), (1, 4, 4, 2048, 1024, "slice_kernel<4>", 256 * 2), (2, 1, 2, 6152, 1024, "slice_kernel<4>", 50 * 10)])
def test_kernel_and_key_splits_of_an_attention_slice(dry, p, batch, heads, seq, room, kernel, grid):
    """(`room`: the registered workspace in MiB; 0: none)"""
    desc = cf.attn_desc(p, 0, batch, heads, seq, 128, 64, 0.1)
    calls = dry.calls(lambda: (cf.set_workspace(P(9), room << 20) if room else None, cf.attn_slice(desc, 0, P(0), P(1), P(2), P(3)),
                               cf.set_workspace(None)))
    (name, workgroups, _), = [c for c in calls if "attn" in c[0]]
    assert kernel in name and workgroups == grid


@pytest.mark.parametrize("m,n,rows,tiles,splits", [(552, 536, 5768, 25, 7), (520, 856, 2544, 35, 4), (776, 1368, 912, 77, 1), (2048, 2048, 8192, 256, 1)])
def test_splits_of_a_weight_gradient(dry, m, n, rows, tiles, splits):
    cf_lib = dry.calls(lambda: (cf.set_workspace(P(9), 1 << 30), cf.wgrad_step(cf.layer_desc(1, 0, rows, n, m), 0, P(0), P(1), P(2)), cf.set_workspace(None)))
    (kernel, grid, _), = [c for c in cf_lib if "gemm" in c[0]]
    assert grid == tiles * splits or (splits == 1 and grid < tiles)


@pytest.mark.parametrize("m,n,rows,tiles,splits", [(136, 152, 848, 4, 1), (168, 552, 912, 10, 1), (72, 112, 920, 1, 1), (568, 72, 1048, 5, 3),
                                                   (1168, 296, 1232, 30, 3), (248, 120, 1472, 2, 4)])
def test_short_weight_gradients_are_split_where_it_pays(dry, m, n, rows, tiles, splits):
    """us whole / split: 9.6 / 10.8, 10.2 / 11.1, 9.9 / 10.8; 11.5 / 11.3, 13.6 / 12.7, 13.4 / 11.7."""
    calls = dry.calls(lambda: (cf.set_workspace(P(9), 1 << 30), cf.wgrad_step(cf.layer_desc(1, 0, rows, n, m), 0, P(0), P(1), P(2)), cf.set_workspace(None)))
    assert [c[1] for c in calls if "gemm" in c[0]] == [tiles * splits]


@pytest.mark.parametrize("m,n,rows,tiles,splits,short,fits", [
    (552, 536, 5768, 25, 7, 6, 5), (480, 304, 4608, 12, 6, 5, 5), (304, 1680, 4600, 42, 4, 3, 4), (144, 640, 7000, 10, 8, 7, 4), (64, 64, 4608, 1, 6, 5, 2)])
def test_splits_that_a_smaller_workspace_takes(dry, m, n, rows, tiles, splits, short, fits):
    """Tiles of 64 KiB: all splits to the byte, fewer 16 bytes short, in 8 m n floats the best that fits, in less than two none."""
    grids = []
    for size in (tiles * splits << 16, (tiles * splits << 16) - 16, 8 * m * n * 4, (tiles * 2 << 16) - 16):
        calls = dry.calls(lambda: (cf.set_workspace(P(9), (64 << 10) + size), cf.wgrad_step(cf.layer_desc(1, 0, rows, n, m), 0, P(0), P(1), P(2)),
                                   cf.set_workspace(None)))
        grids += [c[1] for c in calls if "gemm" in c[0]]
    assert grids == [tiles * splits, tiles * short, tiles * fits, tiles]


@pytest.mark.parametrize("rows,n,k,few_rows", [(363, 3216, 3512, False), (164, 2800, 4640, False), (29, 1024, 8192, True)])
def test_steps_split_as_far_as_the_workspace_goes(dry, rows, n, k, few_rows):
    """The rule against the few-rows kernel prices the split that will run: with room for two splits either kernel, never a tile
    kernel that was priced for four and runs whole."""
    desc = cf.layer_desc(1, 0, rows, n, k)
    tiles = -(-rows // 128) * -(-n // 128)
    seen = []
    for size in (1 << 30, (64 << 10) + (2 * tiles << 16)):
        calls = dry.calls(lambda: (cf.set_workspace(P(9), size), cf.ag_step(desc, 0, P(0), P(1), P(2)), cf.set_workspace(None)))
        seen += [c for c in calls if "gemm" in c[0]]
    rows_kernel = [c[0].startswith("gemm_rows_kernel") for c in seen]
    assert rows_kernel[0] == few_rows
    assert rows_kernel[1] or seen[1][1] == 2 * tiles


@pytest.mark.parametrize("kind,p,mc,n,k", [(cf.CF_KIND_WGRAD_X, 8, 721, 536, 552), (cf.CF_KIND_RS, 2, 213, 3496, 6448), (cf.CF_KIND_RS, 2, 130, 5000, 8184),
                                           (cf.CF_KIND_AG, 2, 200, 712, 8192)])
def test_workspace_bytes_cover_the_splits(dry, kind, p, mc, n, k):
    """A workspace of that size lets a call split as a larger one does."""
    desc = cf.layer_desc(p, 0, mc, n, k)
    need = cf.workspace_bytes(desc, kind)
    def grid(size):
        def call():
            cf.set_workspace(P(9), size)
            if kind == cf.CF_KIND_WGRAD_X:
                cf.wgrad_step(cf.layer_desc(1, 0, p * mc, n, k), 0, P(0), P(1), P(2))
            elif kind == cf.CF_KIND_RS:
                cf.rs_step(desc, 1, P(0), P(1), P(2), P(3))
            else:
                cf.ag_step(desc, 1, P(0), P(1), P(2))
            cf.set_workspace(None)
        return [c for c in dry.calls(call) if "gemm" in c[0]]
    assert grid(need) == grid(1 << 32)


@pytest.mark.parametrize("kind", [cf.CF_KIND_WGRAD_X, cf.CF_KIND_WGRAD_G])
@pytest.mark.parametrize("mc,k,n,pad,off,copied", [
    (1024, 8192, 3584, 0, 0, False), (1024, 3584, 8192, 0, 0, False), (1000, 8192, 3584, 0, 0, True), (1024, 8192, 3592, 0, 0, True),
    (1024, 8192, 3584, 64, 0, True), (1024, 8192, 3584, 0, 8, True), (64, 8192, 3584, 0, 0, True)])
def test_weight_gradients_of_whole_tiles_carry_their_deliveries(dry, kind, mc, k, n, pad, off, copied):
    """(padding between the rows that travel lands with a copy only; the kernel's loads are 16 bytes wide)"""
    p, rank = 8, 3
    width = k if kind == cf.CF_KIND_WGRAD_X else n
    hop = mc * (width + pad) * 2
    block = lambda c: P(20) + c * hop
    stage = [P(10 + i) + off for i in range(p - 1)]
    each = [block((rank - i) % p) for i in range(1, p)]
    left = kind == cf.CF_KIND_WGRAD_X
    desc = cf.layer_desc(p, rank, mc, n, k, lda=k + pad * left, ldw=n + pad * (not left))
    bufs = cf.make_buffers(block(rank), P(1), P(2), stage, (None, None), (None, None), None, each)
    kernels = [c[0] for c in dry.calls(lambda: cf.run_schedule(desc, kind, bufs, None, None, ONE_LAUNCH | cf.CF_FUSED_COPY))]
    assert kernels[-1].startswith("gemm_bf16_dl_kernel") and (len(kernels) > 1) == copied


@pytest.mark.parametrize("room,copied", [(None, False), (32 << 20, True), (1 << 20, False)])
def test_weight_gradients_that_are_split_copy_their_deliveries(dry, monkeypatch, room, copied):
    """The rule that carries looks at the launch as it will run, workspace and all."""
    monkeypatch.setenv("COMMFUSE_TILE", "256x256")
    p, mc, k, n = 8, 512, 1024, 1024
    block = lambda c: P(20) + c * mc * k * 2
    bufs = cf.make_buffers(block(3), P(1), P(2), [P(10 + i) for i in range(p - 1)], (None, None), (None, None), None,
                           [block((3 - i) % p) for i in range(1, p)])
    calls = dry.calls(lambda: (cf.set_workspace(P(9), room) if room else None,
                               cf.run_schedule(cf.layer_desc(p, 3, mc, n, k), cf.CF_KIND_WGRAD_X, bufs, None, None, ONE_LAUNCH | cf.CF_FUSED_COPY),
                               cf.set_workspace(None)))
    kernels = [c[0] for c in calls if "copy" in c[0] or "gemm" in c[0]]
    assert kernels[-1].startswith("gemm_bf16_dl_kernel<256, 256,") and (len(kernels) > 1) == copied
