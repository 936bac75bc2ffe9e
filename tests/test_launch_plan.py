"""Host logic: what the launches would choose, asked of the library without a GPU.  The GEMM tests name the tiles that each of
their sizes stands for; operation (4) never cuts more panels than the workspace provides planes for."""
import ctypes as C
import os
import random

import pytest

import test_gpu_down_parts
import test_gpu_half_tiles
import test_gpu_streamed_operands
from gpu_util import launch_names
from paper_2510_00206_amd import binding
from test_gpu_small_tiles import PLANS, POISON_PLANS


@pytest.fixture(scope="module", autouse=True)
def _lib():
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    binding.load_library()
    yield
    binding.lora_set_row_tile(0)


def _offsets(lens):
    off = [0]
    for n in lens:
        off.append(off[-1] + n)
    return off


def _name(tiles):
    return "+".join(f"{r}x{c}" + (f"@{first}" if first else "") for r, c, first in tiles)


@pytest.mark.parametrize("case", list(PLANS) + list(POISON_PLANS), ids=lambda c: "x".join(map(str, c[:3] + c[3])))
def test_gemm_cases_take_the_tiles_they_stand_for(case):
    K, N, r, lens = case[:4]
    off = _offsets(lens)
    assert (_name(binding.lora_debug_gemm_tiles(K, N, r, off)), _name(binding.lora_debug_gemm_tiles(N, K, r, off))) == \
        (PLANS.get(case) or POISON_PLANS.get(case))


@pytest.mark.parametrize("plans", [PLANS, POISON_PLANS], ids=["values", "poison"])
def test_gemm_cases_cover_every_tile_both_ways(plans):
    small = {"32x64", "64x64", "128x64", "64x128", "128x128"}
    for way in (0, 1):
        names = [v[way] for v in plans.values()]
        first = {n.split("+")[0] for n in names}
        assert small | {"192x256", "256x256"} <= first and any("+" in n for n in names), (way, first)
        assert plans is POISON_PLANS or "128x256" in first


def test_row_tile_setting_fixes_the_tiles():
    for rows in (128, 256):
        binding.lora_set_row_tile(rows)
        assert all(_name(binding.lora_debug_gemm_tiles(K, N, r, _offsets(lens))) == f"{rows}x256" for K, N, r, lens in PLANS)
    binding.lora_set_row_tile(0)


def test_cases_take_the_kernels_they_stand_for():
    binding.lora_set_row_tile(0)
    for (K, r, lens), down in test_gpu_down_parts.CASES.items():
        assert launch_names(K, 64, r, lens)[0] == down, (K, r, lens)
    for case, want in test_gpu_half_tiles.CASES.items():
        assert launch_names(*case)[1:] == want, case
    for case, want in test_gpu_streamed_operands.CASES.items():
        assert launch_names(*case)[1:3] == want, case


def test_row_tile_setting_fixes_the_kernels():
    """The heights that the bit-for-bit tests compare against are other kernels than those they test."""
    cases = [(K, 64, r, lens) for K, r, lens in test_gpu_down_parts.CASES] + [*test_gpu_half_tiles.CASES, *test_gpu_streamed_operands.CASES]
    for setting, rows, tile in ((256, 32, "256x256x64:4"), (128, 16, "128x256x64:12")):
        binding.lora_set_row_tile(setting)
        for K, N, r, lens in cases:
            down, fwd, dx, _ = launch_names(K, N, r, lens)
            assert down.split()[0] == str(rows) and fwd.rstrip("+") == dx.rstrip("+") == tile
            assert setting == 256 or "+" not in fwd + dx
    binding.lora_set_row_tile(0)


def test_slab_lookahead_setting_and_lines_asked_for_ahead():
    """256-row tiles ask for lines only where their copies run two slabs ahead; 192-row tiles always do run so."""
    for slabs, tall, low in ((1, "256x256x64:4", "192x256x64:4+"), (2, "256x256x64:4+", "192x256x64:4+")):
        binding.lora_set_slab_lookahead(slabs)
        assert launch_names(8192, 16384, 64, (1088, 1984, 1024))[1:3] == (tall, tall)
        assert launch_names(28672, 4096, 16, (2999,))[1] == low
    binding.lora_set_slab_lookahead(0)


def test_stages_of_whole_narrow_tiles():
    """Two slabs to a stage: never in (2); in (5) by itself only where a row of W is a multiple of 512 bytes, the contraction has 16 slabs
    and all workgroups run at once."""
    binding.lora_set_row_tile(0)
    rnd = random.Random(19)
    seen = set()
    for it in range(4000):
        G = 1 if it % 2 else rnd.choice((2, 5, 12))
        lens = [rnd.randint(1, 260 // G + 1) for _ in range(G)]
        K, N = 64 * rnd.randint(1, 72), 64 * rnd.randint(1, 72)
        q = binding.lora_debug_launches(K, N, 64, _offsets(lens))
        for way, launches in (("fwd", q.fwd), ("dx", q.dx)):
            for g in launches:
                if (g.rows, g.columns) == (32, 64):
                    deep = way == "dx" and N >= 1024 and K % 256 == 0 and g.workgroups <= 512
                    assert (g.depth, g.stages) == ((128, 3) if deep else (64, 6)), (lens, K, N, way)
                    seen.add((way, deep, g.waves))
    assert seen == {("fwd", False, 7), ("dx", True, 7), ("dx", False, 4), ("dx", False, 8)}


def test_workgroups_beside_the_strips():
    """Whole tiles and strips: at most two workgroups to a compute unit; where halves of tiles take their place, up to half as many tiles more."""
    binding.lora_set_row_tile(0)
    rnd = random.Random(17)
    most = {}
    for it in range(4000):
        G = 1 if it % 2 else rnd.choice((2, 4, 5, 16))
        lens = [rnd.randint(1, 260 // G + 1) for _ in range(G)]
        K, N, r = 64 * rnd.randint(1, 72), 64 * rnd.randint(1, 72), rnd.choice((16, 32))
        if binding.lora_debug_bwd_plan(K, N, r, _offsets(lens)).with_dx:
            _, _, dx, n = launch_names(K, N, r, lens)
            most[dx] = max(most.get(dx, 0), n)
    assert set(most) == {"32x32x128:8", "32x64x128:7", "32x64x64:4", "64x64x64:8"}
    assert most["32x64x128:7"] <= 256 < most["32x64x64:4"] <= 512 < most["32x32x128:8"] <= 640 and most["64x64x64:8"] <= 512, most


def _panels(lens, height):
    return sum(n // height or (n > 0) for n in lens)


def test_da_planes_stay_within_the_workspace():
    """Planes of operation (4): at most what the workspace provides, and at most what the limit of the allocation-free
    backward counts (a plane per panel of the largest height of 1024 .. 64, 256 with the large heights fixed, that gives about
    one workgroup of 512 columns per compute unit)."""
    rnd = random.Random(7)
    lib = binding.load_library()
    rows, panels, bound = C.c_int32(), C.c_int64(), C.c_int64()
    seen = set()
    for it in range(2000):
        G = rnd.randint(1, 64) if it % 3 else rnd.randint(1, 3)
        top = rnd.choice((130, 1000, 6000, 40000))
        lens = [rnd.randrange(top) if it % 2 else 64 * rnd.randrange(top // 64 + 1) for _ in range(G)]
        if sum(lens) == 0:
            lens[0] = 1
        off = (C.c_int64 * (G + 1))(*_offsets(lens))
        for setting in (0, 128, 256):
            binding.lora_set_row_tile(setting)
            for K in (64, 512, 4096, 14336, 28672):
                assert lib.lora_debug_da_panels(sum(lens), K, G, off, C.byref(rows), C.byref(panels), C.byref(bound)) == 0
                h, chunks = 1024, (K + 511) // 512
                while h > (256 if setting == 256 else 64) and _panels(lens, h) * chunks < 224:
                    h //= 2
                assert panels.value == (_panels(lens, rows.value) if rows.value else 0)
                assert panels.value <= min(bound.value, _panels(lens, h)), (lens, K, setting, rows.value)
                assert rows.value == 0 or rows.value >= 256
                seen.add((setting, rows.value == 0))
    assert seen == {(0, True), (0, False), (128, True), (128, False), (256, False)}


@pytest.mark.parametrize("lens,K,height", [((8192,), 26496, 1024), ((6144,), 26496, 2048), ((4096,), 20480, 1024), ((6200,), 8192, 1024),
                                           ((6888, 5702), 4160, 1024), ((3712, 128, 1792), 8640, 512), ((6200,), 2048, 1024),
                                           ((2048,), 960, 256), ((8192,), 4096, 2048), ((5003,), 14336, 0)], ids=str)
def test_da_panel_heights(lens, K, height):
    """Heights that the fp32 error and the times beside plan_da belong to: none taller, none of more rounds."""
    binding.lora_set_row_tile(0)
    off, rows = (C.c_int64 * (len(lens) + 1))(*_offsets(lens)), C.c_int32()
    assert binding.load_library().lora_debug_da_panels(sum(lens), K, len(lens), off, C.byref(rows), C.byref(C.c_int64()), C.byref(C.c_int64())) == 0
    assert rows.value == height


def _noalloc_accepts(M, K, N, r):
    """The documented limit of the allocation-free backward: dS, its partial sums and a plane per panel of the fill rule."""
    def planes(C):
        h = 1024
        while h > 64 and _panels([M], h) * ((C + 511) // 512) < 224:
            h //= 2
        return _panels([M], h)
    up = lambda v: (v + 255) // 256 * 256
    return up(2 * M * r) + up(4 * M * r * ((N + 511) // 512)) + up(4 * planes(N) * r * N) + up(4 * planes(K) * r * K) <= binding.NOALLOC_SCRATCH_BYTES


def test_backward_plan_stays_within_the_scratch():
    """Partial sums and counters of any backward fit what the workspace query provides for; dB's strips, which nothing else adds,
    always have their counters; the allocation-free call sums over the same panels as the one with a workspace."""
    binding.lora_set_row_tile(0)
    rnd = random.Random(11)
    seen = set()
    for it in range(4000):
        G = 1 if it % 2 else rnd.choice((2, 5, 20, 64))
        lens = [int(2 ** rnd.uniform(0, 13.5)) // (1 if G < 5 else G // 4) for _ in range(G)]
        K, N = (64 * int(2 ** rnd.uniform(0, 9)) for _ in range(2))
        r, off = rnd.choice((16, 32, 64)), _offsets(lens)
        for rows in (0, 256):
            binding.lora_set_row_tile(rows)
            plan = binding.lora_debug_bwd_plan(K, N, r, off)
            assert plan.bytes <= binding.workspace_bytes(sum(lens), K, N, r, G), (lens, K, N, r)
            assert plan.added_in_strips or not (plan.ds_alone and (plan.panel_rows_db or plan.panel_rows_da)), (lens, K, N, r)
            assert not (rows and plan.ds_alone)
            seen.add((plan.ds_alone, plan.added_in_strips, plan.with_dx))
            if G == 1 and rows == 0 and _noalloc_accepts(lens[0], K, N, r):
                other = binding.lora_debug_bwd_plan(K, N, r, off, scratch=binding.NOALLOC_SCRATCH_BYTES)
                assert other.bytes <= binding.NOALLOC_SCRATCH_BYTES
                for f in ("ds_alone", "panel_rows_db", "panel_rows_da"):
                    assert getattr(plan, f) == getattr(other, f), (f, lens, K, N, r)
    binding.lora_set_row_tile(0)
    assert seen >= {(1, 1, 0), (1, 0, 0), (1, 0, 1), (1, 1, 1), (0, 1, 0), (0, 0, 0), (0, 0, 1)}, seen


def test_db_panels():
    """No panel of dB that is a whole segment of more than 1792 rows, none of 2048 rows or more."""
    binding.lora_set_row_tile(0)
    rnd = random.Random(13)
    for it in range(3000):
        lens = [int(2 ** rnd.uniform(5, 12.5)) for _ in range(1 if it % 2 else rnd.randint(2, 4))]
        K, N, off = 64 * rnd.randint(1, 80), 64 * rnd.randint(1, 64), _offsets(lens)
        plan = binding.lora_debug_bwd_plan(K, N, 16, off)
        if plan.ds_alone:
            h = plan.panel_rows_db or 1 << 30
            longest = [(n, h + n % h if n // h else n) if n % h else (n, h) for n in lens]
            assert all(m < 2048 and (m < n or m <= 1792) for n, m in longest), (lens, K, N, plan.panel_rows_db)


def test_finalize_launch_where_the_counters_do_not_fit():
    """Fewer than 64 rows with the large heights fixed leave no room behind the planes."""
    binding.lora_set_row_tile(256)
    plan = binding.lora_debug_bwd_plan(320, 64, 16, [0, 48, 53])
    binding.lora_set_row_tile(0)
    assert (plan.ds_alone, plan.panel_rows_da, plan.added_in_strips) == (0, 256, 0)


def test_diagnostics_refuse_what_the_entry_points_refuse():
    off = (C.c_int64 * 2)(0, 64)
    f = lambda M, k, c, r, G, o: binding.load_library().lora_debug_gemm_tiles(
        M, k, c, r, G, o, C.byref(C.c_int32()), (C.c_int32 * 2)(), (C.c_int32 * 2)(), (C.c_int64 * 2)())
    assert [f(64, 64, 64, 0, 1, off), f(64, 64, 64, 16, 1, None), f(64, 0, 64, 16, 1, off), f(64, 96, 64, 16, 1, off),
            f(64, 64, 64, 8, 1, off), f(128, 64, 64, 16, 1, off), f(64, 64, 64, 16, 65, off)] == [0, 1, 2, 7, 7, 5, 7]
    g = lambda M, K, G, o: binding.load_library().lora_debug_da_panels(
        M, K, G, o, C.byref(C.c_int32()), C.byref(C.c_int64()), C.byref(C.c_int64()))
    h = lambda M, K, N, r, G, o: binding.load_library().lora_debug_bwd_plan(M, K, N, r, G, o, 1, 0, C.byref(binding.BwdPlan()))
    q = lambda M, K, N, r, G, o: binding.load_library().lora_debug_launches(M, K, N, r, G, o, C.byref(binding.Launches()))
    assert [q(64, 64, 64, 16, 1, off), q(64, 64, 64, 16, 1, None), q(64, 0, 64, 16, 1, off), q(64, 96, 64, 16, 1, off), q(64, 64, 64, 8, 1, off),
            q(128, 64, 64, 16, 1, off), q(64, 64, 64, 16, 65, off)] == [0, 1, 2, 7, 7, 5, 7]
    none = binding.lora_debug_launches(64, 64, 16, [0, 0])
    assert bytes(none) == bytes(len(bytes(none)))
    assert [h(64, 64, 64, 16, 1, off), h(64, 64, 64, 16, 1, None), h(64, 0, 64, 16, 1, off), h(64, 96, 64, 16, 1, off), h(64, 64, 64, 8, 1, off),
            h(128, 64, 64, 16, 1, off), h(64, 64, 64, 16, 65, off)] == [0, 1, 2, 7, 7, 5, 7]
    assert [g(64, 64, 1, off), g(64, 64, 1, None), g(-1, 64, 1, off), g(128, 64, 1, off), g(64, 64, 65, off)] == [0, 1, 2, 5, 7]
