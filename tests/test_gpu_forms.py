"""Forms of a launch that a rule on sizes, types or alignment chooses: each at the sizes where it can go wrong."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2511_22880_amd import binding as L
from paper_2511_22880_amd import workloads as wl

import gpu_util as G
from test_gpu_parity import _linear_case
from test_launch_routes import (HALVES, LARGE_TILES, LARGE_TILES_MEETING, LARGE_TILES_PADDED, LINEAR_ORDERS, SLICES, TILES_IN_PAIRS,
                                halves_groups, halves_options)

pytestmark = pytest.mark.gpu


def _packed(A, B, r8):
    """The arena bytes of one adapter as include/lora.h states them (element by element)."""
    n_in, r = A.shape
    n_out = B.shape[1]
    Ap = np.zeros((n_in, r8), dtype=np.uint16)
    Ap[:, :r] = A
    Bp = np.zeros((r8, n_out), dtype=np.uint16)
    Bp[:r] = B
    a = np.empty(n_in * r8, dtype=np.uint16)
    k, j = np.meshgrid(np.arange(n_in), np.arange(r8), indexing="ij")
    jb = j // 16
    h = np.minimum(16, r8 - 16 * jb)
    a[16 * jb * n_in + k // 32 * 32 * h + (k % 32 // 8 * h + j % 16) * 8 + k % 8] = Ap
    b = np.empty(n_out * r8, dtype=np.uint16)
    j, c = np.meshgrid(np.arange(r8), np.arange(n_out), indexing="ij")
    b[128 * (c // 128) * r8 + ((c % 8 * (r8 // 8) + j // 8) * 16 + c % 128 // 8) * 8 + j % 8] = Bp
    return a, b


@pytest.mark.parametrize("rank", [1, 7, 8, 9, 16, 24, 100, 128, 255, 256])
@pytest.mark.parametrize("shape", [(64, 128), (320, 384), (1088, 256)])
@pytest.mark.parametrize("offset", [0, 1, 8])
def test_packed_adapter_is_the_documented_layout(rank, shape, offset):
    """lora_pool_load with 16-byte loads (rank a multiple of 8, sources aligned) and without (other ranks, sources
    `offset` elements past an aligned address), into a live pool's second place; bytes outside stay."""
    n_in, n_out = shape
    r8 = (rank + 7) // 8 * 8
    rng = np.random.default_rng([rank, n_in, offset])
    A = rng.integers(0, 1 << 16, size=(n_in, rank)).astype(np.uint16)
    B = rng.integers(0, 1 << 16, size=(rank, n_out)).astype(np.uint16)
    ranks, scales = np.array([3, rank], dtype=np.int32), np.ones(2, dtype=np.float32)
    nbytes = L.lora_pool_bytes(n_in, n_out, ranks, scales)
    arena = torch.full((nbytes + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    pool = L.lora_pool_create(n_in, n_out, ranks, scales, arena, arena_bytes=nbytes)
    src = []
    for m in (A, B):
        t = torch.zeros(offset + m.size, dtype=torch.int16, device="cuda")
        t[offset:] = torch.from_numpy(m.reshape(-1).view(np.int16)).cuda()
        src.append(t[offset:])
    L.lora_pool_load(pool, 1, src[0], src[1])
    torch.cuda.synchronize()
    info = L.lora_pool_adapter_info(pool, 1)
    got = arena.view(torch.int16).cpu().numpy().view(np.uint16)
    a, b = _packed(A, B, r8)
    assert np.array_equal(got[info["a_offset"]:info["a_offset"] + a.size], a)
    assert np.array_equal(got[info["b_offset"]:info["b_offset"] + b.size], b)
    end = info["b_offset"] + b.size
    assert (got[:info["a_offset"]] == 0xA5A5).all() and (got[end:] == 0xA5A5).all()
    L.lora_pool_destroy(pool)


@pytest.mark.parametrize("kind", ["pinned", "pinned, 2 bytes on", "pageable"])
@pytest.mark.parametrize("rank, n_in, n_out", [(1, 64, 128), (24, 320, 384), (255, 2048, 6144), (256, 4160, 4096)])  # 4 MB in between
def test_staged_loads_by_kernel_and_by_copies(kind, rank, n_in, n_out):
    """Pinned sources at 16-byte addresses up to 4 MB are read by a kernel, others copied: the same bytes, also where the host memory
    changes between two loads."""
    rng = np.random.default_rng([rank, n_in])
    r8 = (rank + 7) // 8 * 8
    ranks = np.array([rank], dtype=np.int32)
    arena = torch.zeros(L.lora_pool_bytes(n_in, n_out, ranks, np.ones(1, dtype=np.float32)), dtype=torch.uint8, device="cuda")
    pool = L.lora_pool_create(n_in, n_out, ranks, np.ones(1, dtype=np.float32), arena)
    staging = torch.empty(L.lora_pool_load_staging_bytes(pool, 0), dtype=torch.uint8, device="cuda")
    off = 1 if kind == "pinned, 2 bytes on" else 0
    host = [torch.empty(n + off, dtype=torch.int16, pin_memory=kind != "pageable")[off:] for n in (n_in * rank, rank * n_out)]
    for _ in range(2):
        A, B = (rng.integers(0, 1 << 16, size=s).astype(np.uint16) for s in ((n_in, rank), (rank, n_out)))
        for t, m in zip(host, (A, B)):
            t.copy_(torch.from_numpy(m.reshape(-1).view(np.int16)))
        L.lora_pool_load_staged(pool, 0, host[0], host[1], staging)
        torch.cuda.synchronize()
        info = L.lora_pool_adapter_info(pool, 0)
        got = arena.view(torch.int16).cpu().numpy().view(np.uint16)
        a, b = _packed(A, B, r8)
        assert np.array_equal(got[info["a_offset"]:info["a_offset"] + a.size], a)
        assert np.array_equal(got[info["b_offset"]:info["b_offset"] + b.size], b)
    L.lora_pool_destroy(pool)


def test_what_memory_a_kernel_may_read():
    """The questions asked before a kernel takes the place of copies, about memory as the runtime knows it (nothing reads it)."""
    lib = L.lib()
    pinned_holds, allocation_holds = lib._ZN4lora12pinned_holdsEPKvm, lib._ZN4lora16allocation_holdsEPKvm
    for f in (pinned_holds, allocation_holds):
        f.argtypes, f.restype = (ctypes.c_void_p, ctypes.c_size_t), ctypes.c_bool
    n, beyond = 1 << 20, 1 << 40
    pinned, pageable = torch.empty(n, dtype=torch.uint8, pin_memory=True), np.empty(n, dtype=np.uint8)
    device = torch.empty(n, dtype=torch.uint8, device="cuda")
    h, d = pinned.data_ptr(), device.data_ptr()
    assert pinned_holds(h, n) and pinned_holds(h + 16, n - 16) and not pinned_holds(h, beyond) and not pinned_holds(h + 16, beyond)
    assert allocation_holds(d, n) and allocation_holds(d + 256, n - 256) and not allocation_holds(d, beyond)
    assert not pinned_holds(d, n) and not pinned_holds(pageable.ctypes.data, n)


# ---- token-heavy groups: units cut along k, column runs down to one strip, the two halves apart -----------------
@pytest.mark.parametrize("shape, most", [((64, 128), 1), ((2112, 640), 2), ((3072, 1152), 3), ((4160, 4224), 4)])
@pytest.mark.parametrize("sizes", [
    # (tokens, rank): every bucket of the shrink bodies, tiles of 64 and 32 with one row, one short of full and full
    [(33, 8), (65, 24), (64, 40), (127, 64), (96, 72)],
    [(64, 100), (129, 128), (63, 136), (65, 192), (32, 200), (33, 256)],
    [(40, 16), (70, 160), (3, 64), (1, 256)],  # beside decode-sized groups
])
@pytest.mark.parametrize("cut", ["whole", "most", "built in"])
def test_token_heavy_units_cut_along_k(shape, most, sizes, cut):
    """lora_apply against the oracle, uncut and in as many k-slices as the in_features allow (1 to 4), and lora_shrink +
    lora_expand, whose v is one rounding away from the one lora_apply hands over."""
    b = _batch(*shape, sizes, idle=3, seed=len(sizes))
    dp = G.DevicePool(b)
    limit = {"whole": 0, "most": 1 << 20, "built in": -1}[cut]
    seg = L.lora_segments_build(dp.pool, b.token_adapter, options=L.plan_options(heavy_min_batch=64, heavy_k_cut_max_units=limit))
    u = L.lora_segments_export_units(seg)["shrink"]
    heavy = u[(u[:, 0] >= 0) & (np.diff(L.lora_segments_export(seg)["seg_start"])[u[:, 0]] >= 32)]
    slices = int(heavy[:, 5].max()) + 1
    assert slices == {"whole": 1, "most": most, "built in": slices}[cut]
    x_bits, y0 = b.x_bits(), np.zeros((b.T, b.out_features), dtype=np.uint16)
    x, y = G.bits_to_dev(x_bits), G.bits_to_dev(y0)
    ws = torch.empty(max(L.lora_apply_workspace_bytes(dp.pool, seg), 256), dtype=torch.uint8, device="cuda")
    for _ in range(2):  # the counters are left as they were found
        y.zero_()
        ws.fill_(0xFF)
        L.lora_apply(dp.pool, seg, x, y, ws)
        torch.cuda.synchronize()
        G.check_all_rows(dp, x_bits, y0, G.dev_to_bits(y))
    v = torch.full((L.lora_segments_info(seg)["v_floats"],), float("nan"), dtype=torch.float32, device="cuda")
    vws = torch.full((max(L.lora_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    y.zero_()
    L.lora_shrink(dp.pool, seg, x, v, vws)
    L.lora_expand(dp.pool, seg, v, y)
    torch.cuda.synchronize()
    G.check_all_rows(dp, x_bits, y0, G.dev_to_bits(y))
    L.lora_segments_destroy(seg)
    dp.close()


@pytest.mark.parametrize("pad", [0, 64])
@pytest.mark.parametrize("in_features", [8192, 16384, 24576, 8256])
@pytest.mark.parametrize("cut", [0, 1 << 20])
def test_token_heavy_tiles_that_begin_with_another_pass(in_features, pad, cut):
    """Quarters of whole multiples of 4 KB (8192, 16384 and, uncut, 24576 features; not 8256) up to rank 64, and above always: adapters 0 to 6
    begin with different passes."""
    b = _batch(in_features, 128, [(300, 8), (33, 24), (600, 32), (200, 64), (130, 72), (200, 160), (100, 256)], idle=2, seed=in_features)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    seg = L.lora_segments_build(dp.pool, b.token_adapter, options=L.plan_options(heavy_k_cut_max_units=cut))
    x = torch.full((b.T, in_features + pad), float("nan"), dtype=torch.bfloat16, device="cuda")
    x[:, :in_features] = G.bits_to_dev(x_bits)
    y = G.bits_to_dev(y0)
    ws = torch.full((max(L.lora_apply_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    L.lora_apply(dp.pool, seg, x[:, :in_features], y, ws)
    torch.cuda.synchronize()
    rows = np.arange(0, b.T, 7)
    G.check_parity(G.dev_to_bits(y), G.oracle_apply(dp, x_bits, y0, rows=rows), y0, b.token_adapter, rows=rows)
    L.lora_segments_destroy(seg)
    dp.close()


@pytest.mark.parametrize("groups", [
    [(300, 8), (33, 24), (600, 32), (200, 64), (130, 72), (200, 128), (200, 160), (100, 256)],  # whole
    [(200, 64), (130, 72), (200, 128), (200, 160), (500, 256)],                               # few units: rank halves
    [(300, 32), (130, 64), (900, 8)],
], ids=["many", "halves", "low"])
@pytest.mark.parametrize("in_features", [8192, 16384, 4096])
@pytest.mark.parametrize("cut", [0, 1 << 20])
def test_a_row_has_the_same_bits_wherever_its_token_sits(in_features, groups, cut):
    """Any order of the tokens, those of one group among themselves too, and padded rows of x: adapters' units begin with different passes
    along k, tiles of one adapter do not."""
    b = _batch(in_features, 128, groups, idle=2, seed=in_features)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")

    def apply(order, pad):
        seg = L.lora_segments_build(dp.pool, b.token_adapter[order], options=L.plan_options(heavy_k_cut_max_units=cut))
        x = torch.full((b.T, in_features + pad), float("nan"), dtype=torch.bfloat16, device="cuda")
        x[:, :in_features] = G.bits_to_dev(x_bits[order])
        y = G.bits_to_dev(y0[order])
        ws = torch.full((max(L.lora_apply_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
        L.lora_apply(dp.pool, seg, x[:, :in_features], y, ws)
        torch.cuda.synchronize()
        L.lora_segments_destroy(seg)
        return G.dev_to_bits(y)

    want = apply(np.arange(b.T), 0)
    order = np.random.default_rng(1).permutation(b.T)
    assert np.array_equal(apply(order, 0), want[order])
    assert np.array_equal(apply(np.arange(b.T), 64), want)
    dp.close()


@pytest.mark.parametrize("n_out", [128, 384, 640])
@pytest.mark.parametrize("groups", [
    [(33, 16)], [(47, 64)], [(64, 128)], [(65, 256)],               # the list of token indices ends within a wavefront's 16, or with them
    [(81, 8), (40, 32), (35, 72), (113, 200)],                      # other groups' tokens follow
    [(600, 128), (577, 96)],                                        # more tiles of 64 tokens than a tile of B^T has sub-blocks
], ids=lambda g: "-".join(f"{n}x{r}" for n, r in g))
def test_rows_of_64_token_expand_units(groups, n_out):
    """A wavefront reads its tokens' indices 16 at a time, also where the group has fewer; rows of absent tokens stay as they are."""
    b = _batch(192, n_out, groups, idle=0, seed=n_out)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    seg = L.lora_segments_build(dp.pool, b.token_adapter, options=L.plan_options(heavy_min_batch=1))
    ws = torch.full((max(L.lora_apply_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    v = torch.full((L.lora_segments_info(seg)["v_floats"],), float("nan"), dtype=torch.float32, device="cuda")
    x, apart = G.bits_to_dev(x_bits), G.bits_to_dev(y0)
    y = torch.cat([G.bits_to_dev(y0), torch.zeros(16, n_out, dtype=torch.bfloat16, device="cuda")])
    L.lora_apply(dp.pool, seg, x, y[:b.T], ws)
    L.lora_shrink(dp.pool, seg, x, v, ws)
    L.lora_expand(dp.pool, seg, v, apart)
    torch.cuda.synchronize()
    assert (y[b.T:] == 0).all()
    want = G.oracle_apply(dp, x_bits, y0)
    for got in (y[:b.T], apart):
        G.check_parity(G.dev_to_bits(got), want, y0, b.token_adapter)
    L.lora_segments_destroy(seg)
    dp.close()


@pytest.mark.parametrize("n_out, runs", [(128, -1), (1152, -1), (2176, 0), (4096, -1), (8192, 0), (12928, -1)])
@pytest.mark.parametrize("groups", [
    [(1024, 256)], [(1089, 136)], [(33, 8), (33, 32), (65, 64), (40, 128), (300, 192), (900, 249)], [(64, 160)] * 20, [(63 * 64, 200)],
], ids=lambda g: f"{len(g)}of{g[-1][0]}x{g[-1][1]}")
def test_expand_alone_of_ranks_above_128(groups, n_out, runs):
    """lora_expand in work groups that walk their units, whole or a part, or take 256 columns, by the number of units and their width: one
    strip, odd numbers of them, strips in turn (runs and rows of whole multiples of 4 KB), units of every rank beside, partial tiles, rows
    behind the batch."""
    b = _batch(64, n_out, groups, idle=3, seed=n_out)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    seg = L.lora_segments_build(dp.pool, b.token_adapter, options=L.plan_options(big_runs_max_units=runs))
    v = torch.full((L.lora_segments_info(seg)["v_floats"],), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.full((max(L.lora_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    y = torch.cat([G.bits_to_dev(y0), torch.zeros(16, n_out, dtype=torch.bfloat16, device="cuda")])
    L.lora_shrink(dp.pool, seg, G.bits_to_dev(x_bits), v, ws)
    L.lora_expand(dp.pool, seg, v, y[:b.T])
    torch.cuda.synchronize()
    assert (y[b.T:] == 0).all()
    rows = np.unique(np.concatenate([np.arange(0, b.T, 5), np.arange(b.T - 3, b.T)]))
    G.check_parity(G.dev_to_bits(y[:b.T]), G.oracle_apply(dp, x_bits, y0, rows=rows), y0, b.token_adapter, rows=rows)
    L.lora_segments_destroy(seg)
    dp.close()


@pytest.mark.parametrize("in_features, groups", [(4096, [(900, 64)]), (4096, [(128, 256)] * 4), (9024, [(65, 128)] * 11)])
def test_small_batches_of_token_heavy_units(in_features, groups):
    """Fewer than 1024 tokens: the whole apply, the halves apart, the adapted layer's shrink (that they are token-heavy is tested in
    test_launch_routes.py)."""
    b = _batch(in_features, 384, groups, idle=3, seed=in_features)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    x = G.bits_to_dev(x_bits)
    seg = L.lora_segments_build(dp.pool, b.token_adapter)
    ws = torch.full((max(L.lora_apply_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    vws = torch.full((max(L.lora_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    v = torch.full((L.lora_segments_info(seg)["v_floats"],), float("nan"), dtype=torch.float32, device="cuda")
    y, apart, none = (G.bits_to_dev(y0) for _ in range(3))
    L.lora_apply(dp.pool, seg, x, y, ws)
    L.lora_shrink(dp.pool, seg, x, v, vws)
    L.lora_expand(dp.pool, seg, v, apart)
    w = torch.empty(in_features * 384, dtype=torch.bfloat16, device="cuda")
    L.lora_linear_pack_weight(torch.zeros(384, in_features, dtype=torch.bfloat16, device="cuda"), in_features, 384, w)
    ws.fill_(0xFF)
    L.lora_linear(dp.pool, seg, x, w, none, ws)
    torch.cuda.synchronize()
    rows = np.arange(0, b.T, 3)
    for got, start in ((y, y0), (apart, y0), (none, np.zeros_like(y0))):
        G.check_parity(G.dev_to_bits(got), G.oracle_apply(dp, x_bits, start, rows=rows), start, b.token_adapter, rows=rows)
    L.lora_segments_destroy(seg)
    dp.close()


@pytest.mark.parametrize("in_features, groups", [
    (4096, [(900, 64)]),                            # two work groups a unit
    (4096, [(530, 256), (33, 24), (70, 72)]),       # more than one list of units, partial tiles
    (9024, [(64, 128)] * 11 + [(47, 192), (33, 8)]),
    (4160, [(1000, 248)]),
])
def test_cut_token_heavy_units_without_memory_for_their_slices(in_features, groups):
    """A small batch in the workspace that its units of 16 tokens would take: the first of a tile's cut units does all of k.  The bytes
    behind that workspace stay as they are."""
    b = _batch(in_features, 384, groups, idle=3, seed=in_features)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    x = G.bits_to_dev(x_bits)
    seg = L.lora_segments_build(dp.pool, b.token_adapter)
    of_16 = L.lora_segments_build(dp.pool, b.token_adapter, options=L.plan_options(heavy_min_batch=1024))
    n, stated = (L.lora_apply_workspace_bytes(dp.pool, s) for s in (of_16, seg))
    assert n < stated and L.lora_workspace_bytes(dp.pool, of_16) == 0
    w = torch.empty(in_features * 384, dtype=torch.bfloat16, device="cuda")
    L.lora_linear_pack_weight(torch.zeros(384, in_features, dtype=torch.bfloat16, device="cuda"), in_features, 384, w)
    v = torch.full((L.lora_segments_info(seg)["v_floats"],), float("nan"), dtype=torch.float32, device="cuda")
    y, apart, none = (G.bits_to_dev(y0) for _ in range(3))
    ws = torch.full((stated,), 0xFF, dtype=torch.uint8, device="cuda")
    for _ in range(2):  # (the counters too are as a cut launch would leave them)
        y.copy_(G.bits_to_dev(y0))
        L.lora_apply(dp.pool, seg, x, y, ws[:n])
    L.lora_shrink(dp.pool, seg, x, v, None)
    L.lora_expand(dp.pool, seg, v, apart)
    L.lora_linear(dp.pool, seg, x, w, none, ws[:n])
    cut = G.bits_to_dev(y0)
    assert (ws[n:] == 0xFF).all()
    L.lora_apply(dp.pool, seg, x, cut, ws)
    torch.cuda.synchronize()
    rows = np.arange(0, b.T, 3)
    for got, start in ((y, y0), (apart, y0), (cut, y0), (none, np.zeros_like(y0))):
        G.check_parity(G.dev_to_bits(got), G.oracle_apply(dp, x_bits, start, rows=rows), start, b.token_adapter, rows=rows)
    L.lora_segments_destroy(seg)
    L.lora_segments_destroy(of_16)
    dp.close()


@pytest.mark.parametrize("in_features, ranks, slices", HALVES)
def test_rank_halves_of_few_token_heavy_units(in_features, ranks, slices):
    """Launches of few token-heavy units: halves of the rank rows, even and not, of units of 32 and 64 tokens, whole and cut along
    k; the last tile of a group has 5 tokens (one counter for both halves) or 20.  (That they take the halves is tested in
    test_launch_routes.py.)"""
    b = _batch(in_features, 256, halves_groups(ranks), idle=3, seed=in_features)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    seg = L.lora_segments_build(dp.pool, b.token_adapter, options=halves_options(ranks, slices))
    u = L.lora_segments_export_units(seg)["shrink"]
    assert {int(k) for k in u[u[:, 0] >= 0][:, 5]} == set(range(slices))
    x, y = G.bits_to_dev(x_bits), G.bits_to_dev(y0)
    ws = torch.full((max(L.lora_apply_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    for _ in range(2):  # the counters are left as they were found
        y.copy_(G.bits_to_dev(y0))
        L.lora_apply(dp.pool, seg, x, y, ws)
        torch.cuda.synchronize()
        G.check_all_rows(dp, x_bits, y0, G.dev_to_bits(y))
    v = torch.full((L.lora_segments_info(seg)["v_floats"],), float("nan"), dtype=torch.float32, device="cuda")
    vws = torch.full((max(L.lora_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    y.copy_(G.bits_to_dev(y0))
    L.lora_shrink(dp.pool, seg, x, v, vws)
    L.lora_expand(dp.pool, seg, v, y)
    torch.cuda.synchronize()
    G.check_all_rows(dp, x_bits, y0, G.dev_to_bits(y))
    L.lora_segments_destroy(seg)
    dp.close()


@pytest.mark.parametrize("out_features, pad", [(8192, 0), (16384, 0), (8192, 64), (8320, 0), (8192, 2048)])
def test_strips_of_token_heavy_expand_units_in_any_order(out_features, pad):
    """Runs of 4 KB and its multiples are walked from another strip by every tile of tokens, others (8320 columns, padded rows)
    from the first: 16, 17 and 32 strips a run, ranks with one buffer and with two, the last tile of a group short."""
    b = _batch(64, out_features, [(700, 16), (257, 136), (190, 72)], idle=2, seed=4)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    seg = L.lora_segments_build(dp.pool, b.token_adapter, options=L.plan_options(big_runs_max_units=0))
    ws = torch.empty(max(L.lora_apply_workspace_bytes(dp.pool, seg), 256), dtype=torch.uint8, device="cuda")
    y = torch.full((b.T, out_features + pad), 7.0, dtype=torch.bfloat16, device="cuda")
    y[:, :out_features] = G.bits_to_dev(y0)
    L.lora_apply(dp.pool, seg, G.bits_to_dev(x_bits), y[:, :out_features], ws)
    torch.cuda.synchronize()
    assert bool((y[:, out_features:] == 7.0).all())
    rows = np.arange(0, b.T, 3)
    G.check_parity(G.dev_to_bits(y[:, :out_features].contiguous()), G.oracle_apply(dp, x_bits, y0, rows=rows), y0, b.token_adapter, rows=rows)
    L.lora_segments_destroy(seg)
    dp.close()


@pytest.mark.parametrize("decode", [[], [(3, 40), (1, 200)]], ids=["alone", "beside decode"])
@pytest.mark.parametrize("outs", [
    [384], [1408],             # runs of 3 strips, of 4 and of 3: a work group with one strip
    [1152, 128, 640, 2176],    # projections of unlike widths: 2, 1, 2 and 3 work groups a unit
    [256, 256, 4224],          # and of like ones, then a wider one
])
def test_work_groups_of_64_token_expand_units(outs, decode):
    """Two strips of a unit per work group, at every number of rank steps and chunks, whole and partial; tiles of 64 tokens with one
    wavefront's worth, one token more, one less; lists whose length is no multiple of 8."""
    groups = [(64, 8), (33, 24), (65, 32), (49, 40), (47, 64), (128, 72), (63, 128), (79, 136), (100, 200), (32, 256), (129, 16)]
    b = _batch(192, outs[0], groups + decode, idle=3, seed=len(outs))
    others = [_batch(192, o, groups + decode, idle=3, seed=len(outs)) for o in outs[1:]]
    dps = [G.DevicePool(q) for q in [b] + others]
    pools = [dp.pool for dp in dps]
    opts = L.plan_options(heavy_min_batch=64, big_runs_max_units=0)
    seg = (L.lora_segments_build_multi(pools, b.token_adapter, options=opts) if len(pools) > 1
           else L.lora_segments_build(pools[0], b.token_adapter, options=opts))
    x_bits = b.x_bits()
    y0 = np.concatenate([q.y0_bits("small") for q in [b] + others], axis=1)
    y = G.bits_to_dev(y0)
    ws = torch.full((max(L.lora_apply_workspace_bytes(pools[0], seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
    if len(pools) > 1:
        L.lora_apply_multi(pools, seg, G.bits_to_dev(x_bits), y, ws)
    else:
        L.lora_apply(pools[0], seg, G.bits_to_dev(x_bits), y, ws)
    torch.cuda.synchronize()
    got, at = G.dev_to_bits(y), 0
    for dp, q in zip(dps, [b] + others):
        part = slice(at, at + q.out_features)
        G.check_all_rows(dp, x_bits, np.ascontiguousarray(y0[:, part]), np.ascontiguousarray(got[:, part]))
        at += q.out_features
    L.lora_segments_destroy(seg)
    for dp in dps:
        dp.close()


# ---- batches of few units: one launch by themselves, two under capture ------------------------------------------
@pytest.mark.parametrize("case", [
    # (which of them take the one launch is tested in test_launch_routes.py)
    (64, 128, [(1, 1)]),
    (4096, 4096, [(1, 16)]),
    (1088, 384, [(5, 128), (16, 128)]),             # 16 shrink units
    (1088, 384, [(5, 128), (16, 128), (1, 8)]),     # 17: two launches
    (4160, 1152, [(17, 16), (2, 16)]),              # k-slices, two token tiles
    (512, 8192, [(3, 100)]),                        # 64 expand units
    (2048, [640, 128, 256], [(2, 16), (1, 40)]),    # three projections
])
def test_batches_of_few_units(case):
    """Two inputs in turn, the workspace full of NaNs before every apply and replay: an expand unit that did not wait for
    its v would show."""
    in_features, outs, groups = case
    outs = [outs] if isinstance(outs, int) else outs
    b = _batch(in_features, outs[0], groups, idle=2, seed=8)
    others = [_batch(in_features, o, groups, idle=2, seed=8) for o in outs[1:]]
    dps = [G.DevicePool(q) for q in [b] + others]
    pools = [dp.pool for dp in dps]
    build = L.lora_segments_build_multi if len(pools) > 1 else L.lora_segments_build
    x_bits = [b.x_bits(), np.ascontiguousarray(b.x_bits()[::-1])]
    x = [G.bits_to_dev(q) for q in x_bits]
    y0 = np.concatenate([q.y0_bits("small") for q in [b] + others], axis=1)
    segs = [build(pools if len(pools) > 1 else pools[0], b.token_adapter, options=o)
            for o in (None, L.plan_options(fused_apply=0), L.plan_options(decode_single_launch=0))]
    ws = torch.empty(max(L.lora_apply_workspace_bytes(pools[0], segs[0]), 256), dtype=torch.uint8, device="cuda")

    def apply(seg, i, y, **kw):
        if len(pools) > 1:
            L.lora_apply_multi(pools, seg, x[i], y, ws, **kw)
        else:
            L.lora_apply(pools[0], seg, x[i], y, ws, **kw)

    expect = [None, None]
    for seg in segs + segs:  # (each object twice: the counters are left as the next launch needs them)
        for i in (0, 1):
            y = G.bits_to_dev(y0)
            ws.fill_(0xFF)
            apply(seg, i, y)
            torch.cuda.synchronize()
            L.lora_segments_check(seg)
            got = G.dev_to_bits(y)
            if expect[i] is None:
                expect[i] = got
                at = 0
                for dp, q in zip(dps, [b] + others):
                    part = slice(at, at + q.out_features)
                    G.check_all_rows(dp, x_bits[i], np.ascontiguousarray(y0[:, part]), np.ascontiguousarray(got[:, part]))
                    at += q.out_features
            assert np.array_equal(got, expect[i])
    if len(pools) == 1:  # the library's own workspace, which holds the other input's v
        for i in (0, 1, 0):
            y = G.bits_to_dev(y0)
            L.lora_apply_static(pools[0], segs[0], x[i], y)
            torch.cuda.synchronize()
            L.lora_segments_check(segs[0])
            assert np.array_equal(G.dev_to_bits(y), expect[i])
    y, eager = G.bits_to_dev(y0), G.bits_to_dev(y0)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        apply(segs[0], 0, y, stream=torch.cuda.current_stream())
    for rep in range(4):
        y.copy_(G.bits_to_dev(y0))
        ws.fill_(0xFF)
        graph.replay()
        eager.copy_(G.bits_to_dev(y0))
        torch.cuda.synchronize()
        ws.fill_(0xFF)
        apply(segs[0], rep % 2, eager)
        torch.cuda.synchronize()
        L.lora_segments_check(segs[0])
        assert np.array_equal(G.dev_to_bits(y), expect[0]) and np.array_equal(G.dev_to_bits(eager), expect[rep % 2])
    del graph
    for seg in segs:
        L.lora_segments_destroy(seg)
    for dp in dps:
        dp.close()


# ---- lora_linear: small tiles, large tiles, both in one launch --------------------------------------------------
def _batch(in_features, out_features, groups, idle=0, seed=0):
    """groups: (tokens, rank) of one adapter each; `idle` tokens without adapter; tokens in random order."""
    ranks = np.array([r for _, r in groups] or [8], dtype=np.int32)
    ta = np.concatenate([np.full(n, a, dtype=np.int32) for a, (n, _) in enumerate(groups)]
                        + [np.full(idle, -1, dtype=np.int32)])
    ta = ta[np.random.default_rng([seed, 77]).permutation(ta.shape[0])]
    return wl.CoBatch(f"T{ta.shape[0]}_groups{len(groups)}_idle{idle}", in_features, out_features, ranks,
                      (np.float32(1.7) / ranks).astype(np.float32), ta, seed=seed, config=9)


@pytest.mark.parametrize("tokens", [1, 15, 16, 17, 31, 33, 63, 65, 129, 257])
@pytest.mark.parametrize("shape", [(64, 128), (576, 1024), (1088, 384)])
def test_linear_small_tiles(tokens, shape):
    """Every tile form of few tokens (fewer 64-wide pieces of k than wavefronts, remainders of rows and strips),
    with many adapters per block of 16 rows and ranks on both sides of the 32-wide steps."""
    ranks = (8, 1, 33, 64, 72, 130, 256, 16)
    sizes, left = [], tokens - tokens // 5
    while left > 0:
        sizes.append(min(left, 1 + len(sizes) % 5))
        left -= sizes[-1]
    groups = [(n, ranks[i % len(ranks)]) for i, n in enumerate(sizes)]
    _linear_case(_batch(*shape, groups, idle=tokens // 5, seed=tokens), 0.02, seed=tokens)


@pytest.mark.parametrize("case", [
    # large tiles alone, with a row tile and a strip that are not full
    (LARGE_TILES[1][1], LARGE_TILES[1][2], 0),
    # large tiles, idle rows, and small tiles for the rest of the rows and the small groups
    (4096, [(900, 16), (701, 128)] + [(n % 15 + 1, 8 * (n % 32) + 1) for n in range(40)], 100),
    # nothing but small groups, far too many for small tiles alone
    (2048, [(9, 8 + n % 60) for n in range(700)], 10),
])
def test_linear_large_and_small_tiles_together(case):
    out_features, groups, idle = case
    _linear_case(_batch(128, out_features, groups, idle=idle, seed=5), 0.02, seed=6)


@pytest.mark.parametrize("in_features", [64, 320, 1024])  # 64-wide pieces of k: fewer than a work group's four wavefronts, 5, 16
@pytest.mark.parametrize("tile, out_features, groups", TILES_IN_PAIRS)
def test_linear_small_tiles_beyond_one_per_compute_unit(in_features, tile, out_features, groups):
    _linear_case(_batch(in_features, out_features, groups, idle=1, seed=out_features), 0.02, seed=9)


@pytest.mark.parametrize("in_features, out_features, groups", LARGE_TILES, ids=[c[0] for c in LARGE_TILES])
def test_linear_large_tiles_from_one_pair_of_k_steps_on(in_features, out_features, groups):
    """Large tiles (one strip in the last column tile, rows left over; that no row is in a small one is tested in
    test_launch_routes.py) of 1 to 8 pairs of k steps: fewer than the copies' rings hold, as many, and beyond the first turn of
    both."""
    b = _batch(in_features, out_features, groups, seed=in_features)
    _linear_case(b, 0.02, seed=7, rows=np.arange(0, b.T, 3, dtype=np.int32))


@pytest.mark.parametrize("case", [c for c in LINEAR_ORDERS if c[3] or c[0] < 4096])
def test_linear_row_orders(case):
    """Groups side by side or in blocks of 16 rows of their own, large tiles, small tiles and both: the orders the planner
    chooses among (which one each shape takes is tested in test_launch_routes.py), on every 5th row."""
    b = _batch(*case[:3], idle=case[3], seed=12)
    _linear_case(b, 0.02, seed=13, rows=np.arange(0, b.T, 5, dtype=np.int32))


def test_linear_keeps_what_an_adapter_holds_to_its_own_tokens():
    """An adapter whose B holds infinities: its tokens are not finite, the neighbours in the same block of 16 rows are (small
    tiles; large ones with every group in blocks of its own; large ones whose blocks hold two or three groups)."""
    for in_features, out_features, groups in ((128, 256, [(3, 16), (5, 40), (4, 8)]),
                                              LARGE_TILES_PADDED, LARGE_TILES_MEETING):
        b = _batch(in_features, out_features, groups, seed=3)
        dp = G.DevicePool(b)
        A, B = b.adapter_bits(1)
        B[:] = 0x7F80
        L.lora_pool_load(dp.pool, 1, A, B)
        x = G.bits_to_dev(b.x_bits())
        wp = torch.zeros(in_features * out_features, dtype=torch.bfloat16, device="cuda")
        y = torch.zeros(b.T, out_features, dtype=torch.bfloat16, device="cuda")
        seg = L.lora_segments_build(dp.pool, b.token_adapter)
        ws = torch.empty(max(L.lora_apply_workspace_bytes(dp.pool, seg), 256), dtype=torch.uint8, device="cuda")
        L.lora_linear(dp.pool, seg, x, wp, y, ws)
        torch.cuda.synchronize()
        finite = torch.isfinite(y.float()).all(dim=1).cpu().numpy()
        assert np.array_equal(finite, b.token_adapter != 1)
        L.lora_segments_destroy(seg)
        dp.close()


# ---- k-slice units: what the shrink launch leaves, the expand launch adds up -------------------------------------------
@pytest.mark.parametrize("shape, groups, by", SLICES)
def test_k_slices_added_up_by_the_expand_units(shape, groups, by):
    """Every form of the batch gives the bits of every other, and the oracle's rows: two launches, one, four, each twice.  (Which
    side adds them up in two is tested in test_launch_routes.py.)"""
    b = _batch(*shape, groups, idle=3)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    x, ys = G.bits_to_dev(x_bits), []
    for o in ({"fused_apply": 0}, {"fused_apply": 1}, {"merged_launches": 0, "fused_apply": 0}):
        seg = L.lora_segments_build(dp.pool, b.token_adapter, options=L.plan_options(whole_k_limit=0, heavy_k_cut_max_units=0, **o))
        ws = torch.full((max(L.lora_apply_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
        for _ in range(2):
            y = G.bits_to_dev(y0)
            L.lora_apply(dp.pool, seg, x, y, ws)
            torch.cuda.synchronize()
            ys.append(G.dev_to_bits(y))
        L.lora_segments_check(seg)
        L.lora_segments_destroy(seg)
    assert all(np.array_equal(ys[0], other) for other in ys[1:])
    G.check_all_rows(dp, x_bits, y0, ys[0])
    dp.close()


# ---- whole-k decode batches: one launch or two, by the units of both kinds --------------------------------------------
@pytest.mark.parametrize("units, shape, one", [
    (64, (4096, 4096), False),
    # 6 units and the expand units (one per 512 columns and token tile) together at 2048
    (186, (4096, 2560), False), (187, (4096, 2560), True), (256, (1024, 1024), True), (255, (2112, 1152), True),
    (256, (1024, 7168), False),  # more expand units than one round holds
])
def test_decode_batches_on_either_side_of_the_one_launch_rule(units, shape, one):
    """Groups of one rank block each: the built-in choice, one launch and two launches give the same bits."""
    b = _batch(*shape, [(1 + i % 2, 16) for i in range(units)], seed=units)
    dp = G.DevicePool(b)
    x_bits, y0 = b.x_bits(), b.y0_bits("small")
    x, ys = G.bits_to_dev(x_bits), []
    for o in (None, L.plan_options(decode_single_launch=1), L.plan_options(decode_single_launch=0)):
        seg = L.lora_segments_build(dp.pool, b.token_adapter, options=o)
        if o is None:
            assert bool(L.lora_segments_info(seg)["single_launch"]) == one
        ws = torch.full((max(L.lora_apply_workspace_bytes(dp.pool, seg), 256),), 0xFF, dtype=torch.uint8, device="cuda")
        y = G.bits_to_dev(y0)
        L.lora_apply(dp.pool, seg, x, y, ws)
        torch.cuda.synchronize()
        L.lora_segments_check(seg)
        ys.append(G.dev_to_bits(y))
        L.lora_segments_destroy(seg)
    assert np.array_equal(ys[0], ys[1]) and np.array_equal(ys[0], ys[2])
    rows = np.arange(0, b.T, 7)
    G.check_parity(ys[0], G.oracle_apply(dp, x_bits, y0, rows=rows), y0, b.token_adapter, rows=rows)
    dp.close()
