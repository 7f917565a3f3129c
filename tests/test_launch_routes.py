"""Which launches a call takes, by rules on sizes, settings and capture: the library's host source against launchers
that record (launch_recorder.cpp).  No GPU."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest
import torch

from paper_2511_22880_amd import binding as L

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2511_22880_amd", "csrc")
HIP_INCLUDE = "/opt/rocm/include"
pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir(HIP_INCLUDE),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    """The binding on top of the recording library, for this module's tests."""
    so = str(tmp_path_factory.mktemp("recorder") / "liblora_recorder.so")
    cmd = ["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I" + HIP_INCLUDE,
           "-I" + os.path.join(ROOT, "include"), "-I" + CSRC, "-o", so, os.path.join(ROOT, "tests", "launch_recorder.cpp"),
           os.path.join(CSRC, "lora_host.cpp"), os.path.join(CSRC, "lora_place.cpp"), os.path.join(CSRC, "lora_memory.cpp")]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    path, loaded = L.LIB_PATH, L._lib
    L.LIB_PATH, L._lib = so, None
    lib = L.lib()
    lib.recorder_take.restype = lib.recorder_take_forms.restype = ctypes.c_char_p
    yield lib
    L.LIB_PATH, L._lib = path, loaded


@pytest.fixture(autouse=True)
def no_capture(recorder):
    yield
    recorder.recorder_capture(0)


class Batch:
    """A pool (or several side by side) with every adapter resident, in host memory."""

    def __init__(self, in_features, outs, groups, idle=0):
        self.ranks = np.array([r for _, r in groups], dtype=np.int32)
        self.scales = np.ones(len(groups), dtype=np.float32)
        outs = [outs] if isinstance(outs, int) else outs
        self.ta = np.concatenate([np.full(n, a, dtype=np.int32) for a, (n, _) in enumerate(groups)]
                                 + [np.full(idle, -1, dtype=np.int32)])
        base, at = 1 << 40, 0  # never touched: no kernel runs
        self.pools = []
        for o in outs:
            nbytes = L.lora_pool_bytes(in_features, o, self.ranks, self.scales)
            pool = L.lora_pool_create(in_features, o, self.ranks, self.scales, base + at, arena_bytes=nbytes)
            at += (nbytes + 4095) // 4096 * 4096
            for a in range(len(groups)):
                L.lora_pool_mark_resident(pool, a)
            self.pools.append(pool)
        self.in_features, self.out = in_features, sum(outs)

    def build(self, options=None):
        if len(self.pools) > 1:
            return L.lora_segments_build_multi(self.pools, self.ta, options=options)
        return L.lora_segments_build(self.pools[0], self.ta, options=options)

    def launches(self, lib, seg, call="apply", n=1 << 40, ws=1 << 47):
        """[(kernel, numbers ...), ...] of one call with n bytes of workspace."""
        lib.recorder_take()
        x, y, v = 1 << 44, 1 << 45, 1 << 46
        if call == "apply" and len(self.pools) > 1:
            L.lora_apply_multi(self.pools, seg, x, y, ws, ldx=self.in_features, ldy=self.out, ws_bytes=n)
        elif call == "apply":
            L.lora_apply(self.pools[0], seg, x, y, ws, ldx=self.in_features, ldy=self.out, ws_bytes=n)
        elif call == "static":
            L.lora_apply_static(self.pools[0], seg, x, y, ldx=self.in_features, ldy=self.out)
        elif call == "shrink":
            L.lora_shrink(self.pools[0], seg, x, v, ws, ldx=self.in_features, ws_bytes=n)
        elif call == "expand":
            L.lora_expand(self.pools[0], seg, v, y, ldy=self.out)
        else:
            L.lora_linear(self.pools[0], seg, x, 1 << 43, y, ws, ldx=self.in_features, ldy=self.out, ws_bytes=n)
        return [tuple(int(w) if w.lstrip("-").isdigit() else w for w in line.split())
                for line in lib.recorder_take().decode().splitlines()]

    def close(self):
        for p in self.pools:
            L.lora_pool_destroy(p)


def _names(launches):
    return [n[0] for n in launches]


# ---- the process-wide switches and the built-in choice ----------------------------------------------------------
def test_the_built_in_choice_of_launches_can_be_restored(recorder):
    """Off, on, and back to the choice the library makes before either is called: the same launches as at the start."""
    few, whole = Batch(4096, 4096, [(1, 16)]), Batch(3008, 1920, [(1, 16)] * 128)
    try:
        def forms():
            out = []
            for b in (few, whole):
                seg = b.build()
                out.append(_names(b.launches(recorder, seg)))
                L.lora_segments_destroy(seg)
            return out

        built_in = forms()
        assert built_in == [["apply_fused"], ["shrink_wide", "expand"]]
        L.lora_set_fused_apply(False)
        assert forms()[0] == ["shrink", "expand"]
        L.lora_set_fused_apply(-1)
        L.lora_set_decode_single_launch(False)
        assert forms() == [["shrink", "expand"], ["shrink_wide", "expand"]]
        L.lora_set_decode_single_launch(True)
        assert forms()[1] == ["decode_fused"]
        L.lora_set_decode_single_launch(-1)
        assert forms() == built_in
    finally:
        few.close()
        whole.close()


@pytest.mark.parametrize("in_features, out_features, groups, one", [
    # six times the shrink units and the expand units (of 512 columns here) at 2048: 11 per group
    (4096, 2560, [(1, 16)] * 186, False),
    (4096, 2560, [(1, 16)] * 187, True),
    # more expand units than one round holds
    (4096, 4096, [(1, 16)] * 200, False),
    # little to read in all, but units enough: the one launch was the faster form at 1024 -> 3456 and at 2752 -> 2560
    (1024, 3456, [(1, 64)] * 58, True),
    (2752, 2560, [(1, 64)] * 64, True),
    # nearly 256 shrink units, few expand units
    (14336, 384, [(1, 16)] * 256, False),
    (14336, 512, [(1, 16)] * 256, False),
    # ranks above 128
    (8192, 8192, [(1, 16)] * 190 + [(1, 256)], False),
    (12928, 2176, [(16, 255)] * 13, False),
])
def test_whole_k_decode_batches_in_one_launch(recorder, in_features, out_features, groups, one):
    b = Batch(in_features, out_features, groups)
    seg = b.build()
    assert L.lora_segments_info(seg)["single_launch"] == one
    assert _names(b.launches(recorder, seg)) == (["decode_fused"] if one else ["shrink_wide", "expand"])
    for state in (1, 2):  # two launches under capture, and on the legacy stream while a blocking stream captures
        recorder.recorder_capture(state)
        assert _names(b.launches(recorder, seg)) == ["shrink_wide", "expand"]
    recorder.recorder_capture(0)
    L.lora_segments_destroy(seg)
    b.close()


@pytest.mark.parametrize("in_features, outs, groups, single", [
    (4096, 4096, [(1, 16)], True),
    (1024, 1024, [(1, 128), (1, 128)], True),                      # 16 shrink units
    (1024, 1024, [(1, 128), (1, 128), (1, 8)], False),             # 17
    (2816, 7552, [(1, 256)], False),                               # rank above 128: 13.2 us in one launch, 11.7 in two
    (1024, 1024, [(1, 136)], False),
    (1024, 512 * 84, [(3, 64), (1, 8)], False),                    # many expand units
    (512, 512, [(16, 8)] * 4, True),                               # 64 tokens
    (512, 512, [(16, 8)] * 4 + [(1, 8)], False),                   # 65
    (4096, [4096, 1024, 1024], [(1, 16)], True),                   # q|k|v of one token: 12 shrink units
    (4096, [4096, 1024, 1024], [(1, 16), (1, 16)], False),         # 24
])
def test_batches_of_few_units_in_one_launch(recorder, in_features, outs, groups, single):
    """... by themselves, in lora_apply, lora_apply_multi and lora_apply_static; not under capture, nor where either switch
    is off."""
    b = Batch(in_features, outs, groups, idle=3)
    two = ["shrink", "expand"]
    for options, expect in ((None, single), (L.plan_options(fused_apply=0), False),
                            (L.plan_options(decode_single_launch=0), False), (L.plan_options(fused_apply=1), True)):
        seg = b.build(options)
        assert _names(b.launches(recorder, seg)) == (["apply_fused"] if expect else two)
        if options is None:
            for state in (1, 2):  # 2: the legacy stream while a blocking stream captures
                recorder.recorder_capture(state)
                assert _names(b.launches(recorder, seg)) == two
            recorder.recorder_capture(0)
            if len(b.pools) == 1:
                assert _names(b.launches(recorder, seg, "static")) == (["apply_fused"] if expect else two)
        L.lora_segments_destroy(seg)
    b.close()


# ---- token-heavy groups: how many k-slices their shrink units are cut into ---------------------------------------
def _heavy_slices(b):
    """Into how many slices the tiles of the groups of 32 tokens and more are cut, and how many such tiles there are."""
    seg = b.build()
    u = L.lora_segments_export_units(seg)["shrink"]
    sizes = np.diff(L.lora_segments_export(seg)["seg_start"])
    L.lora_segments_destroy(seg)
    tiles = {}
    for s, tok0, _nt, _p0, _pn, ks in u[u[:, 0] >= 0]:
        if sizes[s] >= 32:
            tiles.setdefault((int(s), int(tok0)), []).append(int(ks))
    slices = len(next(iter(tiles.values()))) // len(b.pools)
    assert all(sorted(k) == sorted(list(range(slices)) * len(b.pools)) for k in tiles.values())
    return slices, len(tiles)


@pytest.mark.parametrize("in_features, groups, slices", [
    # (measured: shrink launch in us, 1 / 2 / 4 slices)
    (64, [(2000, 128)], 1),                                        # nothing to cut
    (4096, [(2000, 128)], 4),                                      # 32 units
    (2176, [(656, 256)] * 10, 1),                                  # 210 units of rank 256: 23.3 / 28.9
    (5120, [(2352, 16), (2352, 32), (2352, 64), (2352, 8)], 2),    # 296 units: 44.0 / 30.8 / 36.6
    (13952, [(1200, 16), (1200, 32), (1200, 64), (1200, 128)], 4), # 134 units: 92.3 / 64.5 / 44.2
    (13952, [(1200, 16), (1200, 32), (1200, 64), (1200, 128)] + [(1, 16)] * 44, 4),
    # 169 + 305 units, the down projection beside 384 decode tokens: 79.4 / 83.1 in 2 / 4 slices
    (14336, [(1400, 8), (1400, 16), (1200, 32), (1200, 64), (320, 128)] + [(1, 16)] * 305, 2),
    # three slices at most: 30 units 27.0 / 20.0 / 16.8 in 1 / 2 / 3, 160 units 39.2 / 25.3 / 30.8, 196 units 30.6 / 23.4 / 25.6
    (3968, [(1920, 128)], 3),
    (3968, [(1249, 256), (1249, 8), (1249, 8), (1249, 256)], 2),
    (4096, [(2000, 128)] * 20, 1),                                 # 640 units
])
def test_token_heavy_shrink_units_are_cut_where_that_is_shorter(recorder, in_features, groups, slices):
    b = Batch(in_features, 512, groups)
    assert _heavy_slices(b)[0] == slices, _heavy_slices(b)
    b.close()
    # the units' cut does not depend on how many projections share the launch: their sums are the same bits
    b = Batch(in_features, [512, 128, 128], groups)
    assert _heavy_slices(b)[0] == slices
    b.close()


# ---- kernels that a launcher chooses between ----------------------------------------------------------------------
def _forms(b, lib, call="apply", options=None):
    seg = b.build(options)
    lib.recorder_take_forms()
    b.launches(lib, seg, call)
    L.lora_segments_destroy(seg)
    return lib.recorder_take_forms().decode().split()


@pytest.mark.parametrize("groups, form", [
    ([(2048, 40)] * 2, "halves"),                       # 128 units of 32 tokens
    ([(2048, 40)] * 2 + [(32, 40)], "whole"),           # 129
    ([(8192, 128)], "halves"),                          # 128 of 64 tokens
    ([(8192, 128), (64, 128)], "whole"),
    ([(2048, 32)] * 2, "whole"),                        # nothing above rank 32
    ([(2048, 32)] + [(2016, 16), (32, 33)], "halves"),
    ([(3000, 8), (1000, 256)], "halves"),               # 126 units; the XCDs' lists, of equal bytes, are filled up to 320 places
    ([(3000, 8), (1100, 256)], "whole"),                # 129
])
def test_few_token_heavy_shrink_units_as_two_work_groups_each(recorder, groups, form):
    b = Batch(1984, 128, groups)
    for call in ("apply", "static", "shrink", "linear"):
        forms = _forms(b, recorder, call, L.plan_options(heavy_k_cut_max_units=0))
        assert forms[0] == form
    b.close()


# (shape, groups, who adds the k-slices up) of batches that have them; test_gpu_forms.py runs them
SLICES = [
    ((64, 128), [(1, 1), (17, 8)], "by_expand"),                                     # one slice
    ((2048, 640), [(16, 24), (17, 33), (1, 256)], "by_expand"),                      # two
    ((3968, 384), [(5, 129), (33, 64), (16, 8)], "by_expand"),                       # three, the last of them short
    ((4096, 1152), [(1, 16)] * 24, "by_expand"),                                     # four
    ((4096, 256), [(40, 72), (1000, 16), (3, 136), (15, 255), (31, 8)], "by_expand"),  # beside token-heavy groups
    ((2048, 8192), [(1, 8)] * 40, "by_expand"),                                      # few shrink units, many expand units
    # 256 shrink units at most, or fewer expand units than twice as many
    ((2048, 4096), [(1, 8)] * 128, "by_expand"),                                     # 256 and 1024
    ((2048, 4096), [(1, 8)] * 129, "by_shrink"),
    ((2048, 1536), [(1, 8)] * 129, "by_expand"),                                     # 258 and 387
    ((2048, 2048), [(1, 8)] * 129, "by_shrink"),                                     # 258 and 516
    ((2048, 8192), [(1, 8)] * 150, "by_shrink"),
    ((2048, 4096), [(1000, 16), (40, 8)] + [(2, 24)] * 20, "by_shrink"),             # the same beside token-heavy groups
    ((1152, 4096), [(1000, 16), (17, 136), (3, 255), (9, 72), (40, 200)], "by_shrink"),  # the same above rank 128, several strips a unit
    ((4096, 640), [(1000, 16), (17, 136), (3, 255), (9, 24), (40, 200), (900, 64)], "by_expand"),
]


@pytest.mark.parametrize("case", SLICES)
def test_who_adds_the_k_slices_up(recorder, case):
    shape, groups, by = case
    b = Batch(*shape, groups, 3)
    two = dict(whole_k_limit=0, heavy_k_cut_max_units=0, fused_apply=0)
    assert _forms(b, recorder, "apply", L.plan_options(**two)) == [by] * 2
    assert _forms(b, recorder, "static", L.plan_options(**two)) == [by] * 2
    apart = L.plan_options(merged_launches=0, **two)  # the token-heavy groups' launches by themselves
    assert [f for f in _forms(b, recorder, "apply", apart) if f not in ("halves", "whole")] == [by] * 2
    assert "by_expand" not in _forms(b, recorder, "linear", L.plan_options(**two))
    assert "callers" in _forms(b, recorder, "shrink", L.plan_options(**two))
    b.close()


# (in, ranks, k-slices) of batches of few token-heavy units, each rank in a group that ends in a tile of 5 tokens and in one that ends
# in a tile of 20; test_gpu_forms.py runs them
HALVES = [(n, ranks, slices) for ranks in ([8, 40, 64], [72, 128], [136, 192], [200, 256], [33, 100, 255])
          for n, slices in ((64, 1), (4160, 1), (4096, 2), (3072, 3), (4160, 4))]


def halves_groups(ranks):
    tile = lambda r: 64 if 64 < (r + 7) // 8 * 8 <= 192 else 32
    return [g for r in ranks for g in ((2 * tile(r) + 5, r), (tile(r) + 20, r))]


def halves_options(ranks, slices):
    # five tiles a rank: twice as many slices would be beyond the limit
    return L.plan_options(heavy_min_batch=64, heavy_k_cut_max_units=5 * len(ranks) * slices if slices > 1 else 0)


@pytest.mark.parametrize("case", HALVES)
def test_batches_that_are_halves_only(recorder, case):
    in_features, ranks, slices = case
    b = Batch(in_features, 256, halves_groups(ranks), 3)
    seg = b.build(halves_options(ranks, slices))
    u = L.lora_segments_export_units(seg)["shrink"]
    assert {int(k) for k in u[u[:, 0] >= 0][:, 5]} == set(range(slices)) and (u[:, 0] >= 0).sum() == 5 * len(ranks) * slices
    for call in ("apply", "shrink"):
        recorder.recorder_take_forms()
        launches = b.launches(recorder, seg, call)
        assert recorder.recorder_take_forms() == b"halves "
        assert all(name in ("shrink_prefill", "expand_big", "reduce_slices") for name, *_ in launches)
    L.lora_segments_destroy(seg)
    b.close()


# ---- the adapted layer's row order and tiles ---------------------------------------------------------------------
# (in, out, groups, idle tokens, every group in blocks of its own, row tiles of 256 places as large tiles, of how many);
# test_gpu_forms.py runs them
LINEAR_ORDERS = [
    # large tiles for all rows, padded: small groups that would meet in a block; 1088 -> 8192 was 50 us so, 73 in small tiles
    (1088, 8192, [(170, 64), (150, 8), (96, 16)] + [(3, 8 * (n % 16) + 8) for n in range(56)], 120, True, 6, 6),
    (128, 8192, [(300, 128), (200, 16)] + [(n % 15 + 1, 8 * (n % 16) + 8) for n in range(40)], 60, True, 5, 5),
    # large tiles that fill the compute units, small ones behind them: padded, and not
    (128, 4096, [(900, 16), (701, 128)] + [(n % 15 + 1, 8 * (n % 32) + 1) for n in range(40)], 100, True, 8, 10),
    (576, 3072, [(1128, 8)] * 4, 0, True, 16, 18),
    (2176, 3072, [(1128, 8)] * 4, 0, False, 16, 18),
    # few row tiles, but a long k: 8192 -> 3328 was 218 us in small tiles, 159 in large ones
    (8192, 3328, [(400, 8), (400, 16), (400, 64), (400, 128)], 0, False, 4, 7),
    # large tiles for all rows, not padded
    (128, 2048, [(9, 8 + n % 60) for n in range(700)], 10, False, 25, 25),
    # small tiles
    (4096, 4096, [(2, 64)] * 128, 0, False, 0, 1),
    # short k and high ranks: v of whole wavefronts of rows is what a large tile starts with (27 us, in large tiles 33; 14, 20; 29, 34)
    (128, 512, [(1843, 256), (725, 40), (1232, 128)], 760, False, 0, 18),
    (128, 1280, [(500, 128), (341, 8)], 0, False, 0, 4),
    (192, 384, [(4000, 256), (397, 256)], 0, False, 0, 18),
    (64, 128, [], 5, False, 0, 1),
]


@pytest.mark.parametrize("case", LINEAR_ORDERS)
def test_row_order_and_tiles_of_the_adapted_layer(recorder, case):
    in_features, out_features, groups, idle, padded, big, tiles = case
    b = Batch(in_features, out_features, groups or [(0, 8)], idle)
    seg = b.build()
    name, places, got = b.launches(recorder, seg, "linear")[-1]
    assert name == "linear" and got == big and (places + 255) // 256 == tiles
    assert places <= sum((n + 15) // 16 * 16 for n, _ in groups) + idle + 16 if padded else places == len(b.ta)
    assert (places > len(b.ta)) == padded
    L.lora_segments_destroy(seg)
    b.close()


# (small tiles, out, groups) of more than a tile per compute unit: two work groups of four wavefronts share one; test_gpu_forms.py runs them
TILES_IN_PAIRS = [
    ("64x64", 8192, [(70, 24), (1, 256), (40, 8), (19, 130)]),  # 384 tiles
    ("32x64", 8064, [(33, 64), (29, 9), (3, 200)]),             # 378
    ("32x32", 4224, [(9, 16), (23, 72)]),                       # 264
    ("16x32", 8320, [(7, 40), (6, 255)]),                       # 260
]


@pytest.mark.parametrize("in_features", [64, 320, 1024])
@pytest.mark.parametrize("tiles, out, groups, pairs", [case + (True,) for case in TILES_IN_PAIRS] + [
    ("64x64", 4096, [(256, 8)], False),   # 256
    ("64x64", 8320, [(128, 8)], True),    # 260
    ("32x32", 4096, [(33, 8)], False),    # 256
    ("16x32", 8192, [(16, 8)], False),    # 256
    ("16x32", 8320, [(16, 8)], True),     # 260
])
def test_small_tiles_of_the_adapted_layer(recorder, in_features, tiles, out, groups, pairs):
    b = Batch(in_features, out, groups, 1 if (tiles, out, groups) in TILES_IN_PAIRS else 0)
    assert _forms(b, recorder, "linear")[-1] == tiles + ("_in_pairs" if pairs else "")
    b.close()


# (in, out, groups) of which every row is in a large tile: what test_gpu_forms.py checks the large tiles' copies, waits and
# deltas with.  The last column tile of the first ones holds one strip; the last batch is the one whose groups meet in blocks of 16.
LARGE_TILES = [(n, 4224, [(700, 128), (513, 8), (300, 40), (291, 200)]) for n in (64, 128, 192, 256, 320, 512)]
LARGE_TILES_PADDED = (64, 4096, [(1003, 16), (605, 40), (900, 8)])
LARGE_TILES_MEETING = (64, 2048, [(9, 8 + n % 60) for n in range(700)])


@pytest.mark.parametrize("case", LARGE_TILES + [LARGE_TILES_PADDED, LARGE_TILES_MEETING])
def test_batches_that_are_large_tiles_only(recorder, case):
    in_features, out_features, groups = case
    b = Batch(in_features, out_features, groups)
    seg = b.build()
    name, places, big = b.launches(recorder, seg, "linear")[-1]
    assert name == "linear" and big == (places + 255) // 256
    assert (places == len(b.ta)) == (case is LARGE_TILES_MEETING)
    L.lora_segments_destroy(seg)
    b.close()


@pytest.mark.parametrize("in_features, outs, groups, call, faster, plainer", [
    (1088, 8192, LINEAR_ORDERS[0][2], "linear", 
     [("shrink_wide", 296), ("linear", 1315, 6)], [("shrink_wide", 296), ("linear", 584, 0)]),
    (1024, 3456, [(1, 64)] * 58, "apply", 
     [("decode_fused", 256)], [("shrink_wide", 232), ("expand", 812)]),
    (4096, 8192, [(2000, 128)], "apply", 
     [("shrink_prefill", 128, 4), ("expand_big", 512)], [("shrink_prefill", 32, 4), ("expand_big", 128)]),
    (1024, 4096, [(600, 64)] * 2, "apply", 
     [("shrink_prefill", 40, 1), ("expand_big", 320)], [("shrink_prefill", 40, 1), ("expand_big", 80)]),
    (4096, [4096, 1024], [(600, 64)] * 3, "apply", 
     [("shrink_prefill", 464, 4), ("expand_big", 480)], [("shrink_prefill", 128, 4), ("expand_big", 180)]),
])
def test_a_caller_s_table_without_room_for_the_faster_form(recorder, in_features, outs, groups, call, faster, plainer):
    """lora_segments_rebuild into memory that holds the batch's units, but not padded rows, the one launch's lists, k-slices or
    short column runs: accepted, in the plainer form; refused where that has no room either."""
    b = Batch(in_features, outs, groups)
    def plan(ta):
        return L.lora_segments_plan_multi(b.pools, ta) if len(b.pools) > 1 else L.lora_segments_plan(b.pools[0], ta)

    seg = plan(b.ta)
    need = L.lora_segments_table_bytes(seg)
    L.lora_segments_destroy(seg)
    for size, expect in ((need, faster), (need - 256, plainer), (need // 4, None)):
        first = plan(b.ta[:1])
        dev, staging = (m[-m.data_ptr() % 256:][:size] for m in (torch.zeros(size + 256, dtype=torch.uint8) for _ in range(2)))
        L.lora_segments_upload_to(first, dev, staging)
        if expect is None:
            with pytest.raises(L.LoraError, match="OOM"):
                L.lora_segments_rebuild(first, b.ta)
        else:
            L.lora_segments_rebuild(first, b.ta)
            assert b.launches(recorder, first, call) == expect
        L.lora_segments_destroy(first)
    b.close()


# ---- batches of fewer than 1024 tokens that take token-heavy units all the same ------------------------------------------
@pytest.mark.parametrize("in_features, groups, heavy", [
    (4096, [(900, 64)], True), (4096, [(512, 64)], False),                      # up to rank 64: by the rank rows fetched again
    (4096, [(512, 256)], True), (4096, [(256, 256)], False),
    (14336, [(900, 256)], True), (14336, [(256, 256)], False),                  # ... and by the length of the walk along k
    (4096, [(128, 256)] * 4, True), (4096, [(128, 256)] * 3 + [(31, 8)], False),  # one group of fewer than 32 tokens
    (1600, [(646, 128)], False), (9024, [(700, 128)], True),
])
def test_small_batches_of_token_heavy_units(recorder, in_features, groups, heavy):
    """Every projection of one x decides alike, whatever its columns; the option and both halves' own calls are as for larger batches."""
    for outs in (128, 14336, [256, 14336]):
        b = Batch(in_features, outs, groups, idle=5)
        seg = b.build()
        names = _names(b.launches(recorder, seg))
        assert names == (["shrink_prefill", "expand_big"] if heavy else ["shrink_wide", "expand"])
        if outs == 128:
            assert ("shrink_prefill" in _names(b.launches(recorder, seg, "shrink"))) == heavy
            assert ("shrink_prefill" in _names(b.launches(recorder, seg, "linear"))) == heavy
            assert _names(b.launches(recorder, seg, "static")) == names
        L.lora_segments_destroy(seg)
        seg = b.build(L.plan_options(heavy_min_batch=1024))
        assert "expand_big" not in _names(b.launches(recorder, seg))
        L.lora_segments_destroy(seg)
        b.close()


def _in_a_table_of(b, size, tokens):
    """An object of b's pools whose table and staging hold `size` bytes, as planned for the first `tokens` tokens."""
    seg = L.lora_segments_plan_multi(b.pools, b.ta[:tokens]) if len(b.pools) > 1 else L.lora_segments_plan(b.pools[0], b.ta[:tokens])
    dev, staging = (m[-m.data_ptr() % 256:][:size] for m in (torch.zeros(size + 256, dtype=torch.uint8) for _ in range(2)))
    L.lora_segments_upload_to(seg, dev, staging)
    return seg


def _room(b, options=None):
    seg = L.lora_segments_plan(b.pools[0], b.ta, options) if len(b.pools) == 1 else L.lora_segments_plan_multi(b.pools, b.ta, options)
    n = L.lora_segments_table_bytes(seg)
    L.lora_segments_destroy(seg)
    return n


@pytest.mark.parametrize("in_features, outs, rank, tokens", [
    (4096, 4096, 256, (900, 400, 256, 31, 1)), (4096, 4096, 64, (900, 512, 100)), (8192, 8192, 128, (900, 200)),
    (4096, [1024, 4096], 256, (1023, 400, 256)), (14336, 128, 256, (700, 256)),
])
def test_a_table_made_for_the_largest_small_batch_holds_the_smaller_ones(recorder, in_features, outs, rank, tokens):
    """Token-heavy units take a smaller table than the units of 16 tokens that a batch of fewer tokens goes back to."""
    b = Batch(in_features, outs, [(tokens[0], rank)])
    room = _room(b)
    assert room >= _room(b, L.plan_options(heavy_min_batch=1024)) > _room(b, L.plan_options(heavy_min_batch=1))
    seg = _in_a_table_of(b, room, tokens[0])
    for n in tokens:
        L.lora_segments_rebuild(seg, b.ta[:n])
        names = _names(b.launches(recorder, seg))
        assert ("expand_big" in names) == (n == tokens[0])
    L.lora_segments_destroy(seg)
    with pytest.raises(L.LoraError, match="OOM"):
        _in_a_table_of(b, room - 256, tokens[0])
    b.close()


@pytest.mark.parametrize("outs", [4096, [4096, 1024]])
def test_a_table_without_room_for_the_cuts_of_a_small_batch_s_token_heavy_units(recorder, outs):
    """They lose their cuts along k and their short column runs, not their 64 tokens; units of 16 tokens would need more."""
    b = Batch(4096, outs, [(900, 256)])
    room = _room(b)
    cut = _room(b, L.plan_options(heavy_min_batch=1))  # (without the list of uncut units, for a workspace without slices)
    plain = _room(b, L.plan_options(heavy_min_batch=1, heavy_k_cut_max_units=0, big_runs_max_units=0))
    assert plain < cut < room
    made = {}
    for size in (room, cut, plain):
        seg = _in_a_table_of(b, size, 1)
        L.lora_segments_rebuild(seg, b.ta)
        made[size] = b.launches(recorder, seg)
        assert _names(made[size]) == ["shrink_prefill", "expand_big"]
        L.lora_segments_destroy(seg)
    assert made[room][0][1] > made[plain][0][1] and made[cut] == made[plain]
    seg = _in_a_table_of(b, plain - 256, 1)
    with pytest.raises(L.LoraError, match="OOM"):
        L.lora_segments_rebuild(seg, b.ta)
    L.lora_segments_destroy(seg)
    b.close()


@pytest.mark.parametrize("in_features, outs, groups, whole_k", [
    (4096, 512, [(900, 64)], True), (9024, 384, [(700, 128)], True), (4096, [512, 128, 128], [(900, 64)], True),
    (4096, 512, [(512, 256)], True), (4096, 512, [(1023, 256)], True),                # 512 and 1024 units of 16 tokens,
    (4096, 512, [(980, 256), (43, 256)], False), (28672, 512, [(512, 64)], False),    # 1040; beyond the longest whole k
])
def test_the_workspace_of_units_of_16_tokens_is_enough_for_a_small_batch(recorder, in_features, outs, groups, whole_k):
    """A workspace that units of 16 tokens over the whole of k fit, made for another batch, stays one that this batch can use:
    token-heavy units then run without their cuts.  One byte less is refused, as is less than stated where the units of 16 tokens
    would be cut too."""
    b = Batch(in_features, outs, groups)
    seg, of_16 = b.build(), b.build(L.plan_options(heavy_min_batch=1024))
    for call in ["apply"] + ["shrink", "linear"] * (len(b.pools) == 1):
        def shrinks(n, ws=1 << 47):  # (kernel, slices) of the launches in front of the expand or the product
            return [(k[0], k[-1]) for k in b.launches(recorder, seg, call, n, ws) if k[0] not in ("expand_big", "linear")]

        size = L.lora_workspace_bytes if call == "shrink" else L.lora_apply_workspace_bytes
        stated, enough = size(b.pools[0], seg), size(b.pools[0], of_16)
        assert (enough < stated) == whole_k and shrinks(stated)[0][0] == "shrink_prefill" and shrinks(stated)[0][1] > 1
        if whole_k:
            assert shrinks(enough) == [("shrink_prefill", 1)]
        if whole_k and call == "shrink":  # these do not look at the workspace
            assert enough == 0 and shrinks(0, 0) == shrinks(stated, (1 << 47) + 16) == [("shrink_prefill", 1)]
        else:
            with pytest.raises(L.LoraError, match="WORKSPACE"):
                shrinks(enough - 1)
    L.lora_segments_destroy(seg)
    L.lora_segments_destroy(of_16)
    b.close()


# ---- 64-token expand units: work groups per compute unit, runs of columns, order -----------------------------------------
@pytest.mark.parametrize("outs, groups, three", [
    (4096, [(4096, 128)], False), (4096, [(4097, 128)], True),       # 64 tiles of 16 work groups, all on the chip at four; one more tile
    (4096, [(4097, 8)], True), (4096, [(4097, 136)], False),         # above rank 128 four hide the copies
    ([4096, 1024], [(3200, 64)], False), ([4096, 1024], [(3300, 64)], True), (128, [(3000, 16)], False),
])
def test_work_groups_per_compute_unit_of_64_token_expand_units(recorder, outs, groups, three):
    """Three only where four would not hold the launch at once."""
    b = Batch(512, outs, groups)
    seg = b.build()
    b.launches(recorder, seg)
    assert recorder.recorder_big_spread() == three
    L.lora_segments_destroy(seg)
    b.close()


@pytest.mark.parametrize("out, tiles, units", [
    (14336, 32, 32 * 8), (3072, 63, 63 * 4), (5632, 32, 32 * 8), (5120, 24, 24 * 4),  # 16 runs would have 7 strips, 8 have 3, 16 3, 16 3 and 8 5
    (14336, 16, 16 * 28), (4096, 32, 32 * 16), (1024, 63, 63 * 8),                    # runs of 4 strips, 2 and one
    (9216, 62, 62 * 8), (11008, 50, 50 * 8),                                          # of 9 and 11
])
def test_runs_of_columns_hold_whole_work_groups(recorder, out, tiles, units):
    """A work group of 64-token expand units takes two strips of 128 columns: runs of 3, 5 or 7 are passed over."""
    b = Batch(512, out, [(64 * tiles, 64)])
    seg = b.build()
    assert b.launches(recorder, seg)[-1] == ("expand_big", units)
    L.lora_segments_destroy(seg)
    b.close()


@pytest.mark.parametrize("out, groups, strips", [
    (4096, [(63 * 64, 256)], 4), (14336, [(17 * 64, 160)], 5), (4096, [(300 * 64, 192)], 8),  # whole units, a third of one, several rounds
    (1024, [(300 * 64, 256)], 0), (2048, [(31 * 64, 256)], 0), (8064, [(17 * 64, 192)], 0),   # narrow; one strip a unit; too few to walk 4
    (4096, [(63 * 64, 128)], 0), (14336, [(125 * 64, 64)], 0),                              # one chunk of the rank
    (8064, [(1000, 8), (1000, 256)] * 4, 0), (8064, [(1000, 8)] * 2 + [(1000, 256)] * 6, 16),  # half of the units, and three quarters
    (4736, [(130 * 64, 192)], 0),                                                           # a second round of few walks
])
def test_expand_alone_walks_units_above_rank_128(recorder, out, groups, strips):
    """lora_expand's v is fp32 in rows: work groups that load it once, where they fill the chip; lora_apply's launches never."""
    b = Batch(512, out, groups)
    seg = b.build()
    assert _names(b.launches(recorder, seg, "expand")) == ["expand_big"] and recorder.recorder_walks() == strips
    b.launches(recorder, seg)
    assert recorder.recorder_walks() == 0
    L.lora_segments_destroy(seg)
    b.close()


# ---- the binding's own checks of arguments --------------------------------------------------------------------------
@pytest.mark.parametrize("adapter", ["0", None, 0.0, ctypes.c_int32(0)])
def test_an_adapter_that_is_no_whole_number_is_a_type_error(recorder, adapter):
    """... where A and B come from device memory, which nothing else looks at the number for; any kind of whole number is taken."""
    b = Batch(64, 128, [(1, 8)])
    pool = b.pools[0]
    device = torch.zeros(64, 8, dtype=torch.bfloat16), torch.zeros(8, 128, dtype=torch.bfloat16)
    with pytest.raises(TypeError):
        L.lora_pool_load(pool, adapter, *device)
    L.lora_pool_load(pool, np.int64(0), *device)
    b.close()


# ---- staged loads: what may be read by a kernel ------------------------------------------------------------------------
@pytest.fixture
def staged(recorder):
    """A pool of one adapter (rank 8, 128 -> 256), and pinned sources and a staging buffer as the runtime knows them."""
    ranks, n = np.array([8], dtype=np.int32), [128 * 8 * 2, 8 * 256 * 2]
    arena = np.zeros(L.lora_pool_bytes(128, 256, ranks, np.ones(1, dtype=np.float32)), dtype=np.uint8)
    pool = L.lora_pool_create(128, 256, ranks, np.ones(1, dtype=np.float32), arena.ctypes.data // 256 * 256, arena_bytes=arena.size)
    host = torch.empty(1 << 14, dtype=torch.uint8)
    at = [(host.data_ptr() + 255) // 256 * 256 + q * 4096 for q in range(3)]  # A, B and the staging, 4 KB apart
    recorder.recorder_memory.argtypes = [ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]

    def load(bytes_a=n[0], bytes_b=n[1], bytes_staging=sum(n), shift=0, pinned=1):
        for p, size, kind in zip(at, (bytes_a, bytes_b, bytes_staging), (pinned, pinned, 0)):
            recorder.recorder_memory(p, size, kind)
        for q in range(5):
            recorder.recorder_memory(None, 0, 0)  # (the oldest are forgotten)
        recorder.recorder_take()
        L._check(L.lib().lora_pool_load_staged(pool.handle, 0, at[0] + shift, at[1], at[2], sum(n), None))
        return recorder.recorder_take().decode().split()

    yield load
    L.lora_pool_destroy(pool)


def test_staged_loads_go_by_kernel_where_all_of_the_memory_is_known(staged):
    """The kernel reads and writes the adapter's size whatever is there; a copy refuses what exceeds an allocation."""
    by_kernel = ["copy_in", "2048", "4096"]
    assert staged() == staged(bytes_a=4096, bytes_b=4096) == by_kernel
    assert staged(bytes_a=2047) == [] and staged(bytes_b=4095) == []     # the first byte is pinned, the last is not
    assert staged(bytes_a=2063, shift=16) == [] and staged(bytes_a=2064, shift=16) == by_kernel
    assert staged(bytes_staging=6143) == []
    assert staged(pinned=0) == []


@pytest.mark.parametrize("make", [lambda n: np.zeros(n, dtype=np.uint16), lambda n: torch.zeros(n, dtype=torch.bfloat16)])
def test_staged_loads_refuse_sources_shorter_than_the_adapter(recorder, make):
    b = Batch(64, 128, [(1, 8)])
    pool, staging = b.pools[0], torch.empty(1 << 12, dtype=torch.uint8)
    for a, c in ((64 * 8 - 1, 8 * 128), (64 * 8, 8 * 128 - 1)):
        with pytest.raises(ValueError, match="shorter than rank 8"):
            L.lora_pool_load_staged(pool, 0, make(a), make(c), staging)
    L.lora_pool_load_staged(pool, 0, make(64 * 8), make(8 * 128 + 5), staging)
    L.lora_pool_load_staged(pool, np.int64(0), make(64 * 8), make(8 * 128), staging)
    for adapter in (-1, 1):
        with pytest.raises(L.LoraError):
            L.lora_pool_load_staged(pool, adapter, make(1), make(1), staging)
    with pytest.raises(L.LoraError):
        L.lora_pool_load_staged(pool, 0, None, make(8 * 128), staging)
    b.close()
