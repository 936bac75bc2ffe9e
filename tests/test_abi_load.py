"""The C-ABI library loads and exports every symbol the header declares; host-side validation
paths return the documented status codes without touching a GPU."""
import ctypes as C
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "include", "lorafusion.h")


@pytest.fixture(scope="module")
def lib():
    from paper_2510_00206_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    return binding.load_library()


def _declared():
    src = open(HEADER).read()
    src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
    return sorted(set(re.findall(r"\b((?:multi_)?lora_[a-z_]+)\s*\(", src)))


def test_every_declared_symbol_is_exported(lib):
    names = _declared()
    assert {"lora_fwd", "lora_bwd", "multi_lora_fwd", "multi_lora_bwd"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n


def test_version_and_status_strings(lib):
    assert lib.lora_version() >= 100
    assert [lib.lora_set_row_tile(v) for v in (128, 256, 64, -1, 0)] == [0, 0, 4, 4, 0]
    assert [lib.lora_set_slab_lookahead(v) for v in (1, 2, 3, -1, 0)] == [0, 0, 4, 4, 0]
    assert lib.lora_status_string(0) == b"ok"
    for code in range(1, 9):
        assert len(lib.lora_status_string(code)) > 3


def test_host_side_validation_needs_no_gpu(lib):
    """Validation fails before anything is enqueued, so these calls are safe on a CPU-only box."""
    ok_ptr = C.c_void_p(0x1000)
    f = lib.lora_fwd
    assert f(None, ok_ptr, ok_ptr, ok_ptr, 64, 64, 64, 16, 1.0, 0.1, 1, ok_ptr, ok_ptr, None) == 1
    assert f(ok_ptr, ok_ptr, ok_ptr, ok_ptr, -1, 64, 64, 16, 1.0, 0.1, 1, ok_ptr, ok_ptr, None) == 2
    assert f(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 64, 0, 64, 16, 1.0, 0.1, 1, ok_ptr, ok_ptr, None) == 2
    assert f(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 64, 96, 64, 16, 1.0, 0.1, 1, ok_ptr, ok_ptr, None) == 7
    assert f(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 64, 64, 64, 8, 1.0, 0.1, 1, ok_ptr, ok_ptr, None) == 7
    assert f(C.c_void_p(0x1008), ok_ptr, ok_ptr, ok_ptr, 64, 64, 64, 16, 1.0, 0.1, 1, ok_ptr, ok_ptr, None) == 3
    for bad_p in (-0.1, 1.0, float("nan")):
        assert f(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 64, 64, 64, 16, 1.0, bad_p, 1, ok_ptr, ok_ptr, None) == 4
    assert f(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 64, 64, 64, 16, float("inf"), 0.1, 1, ok_ptr, ok_ptr, None) == 4
    assert f(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 0, 64, 64, 16, 1.0, 0.1, 1, ok_ptr, ok_ptr, None) == 0   # M == 0: no-op
    # segments
    offs = (C.c_int64 * 3)(0, 128, 64)
    s = (C.c_float * 2)(1.0, 1.0)
    p = (C.c_float * 2)(0.1, 0.1)
    sd = (C.c_uint64 * 2)(1, 2)
    m = lib.multi_lora_fwd
    assert m(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 64, 64, 64, 16, 2, offs, s, p, sd, ok_ptr, ok_ptr, None) == 5
    offs = (C.c_int64 * 3)(0, 32, 128)
    assert m(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 64, 64, 64, 16, 2, offs, s, p, sd, ok_ptr, ok_ptr, None) == 5
    assert m(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 64, 64, 64, 16, 65, offs, s, p, sd, ok_ptr, ok_ptr, None) == 7
    # workspace
    need = lib.lora_bwd_workspace_bytes(256, 128, 128, 16, 1)
    assert need > 0 and lib.lora_bwd_workspace_bytes(256, 100, 128, 16, 1) == 0
    ws = C.c_void_p(0x100000)
    b = lib.lora_bwd
    assert b(ok_ptr, ok_ptr, ok_ptr, ok_ptr, ok_ptr, ok_ptr, 256, 128, 128, 16, 1.0, 0.1, 1,
             ok_ptr, ok_ptr, ok_ptr, 0, ws, need - 1, None) == 6
    assert b(ok_ptr, ok_ptr, ok_ptr, ok_ptr, ok_ptr, ok_ptr, 256, 128, 128, 16, 1.0, 0.1, 1,
             ok_ptr, ok_ptr, ok_ptr, 0, None, need, None) == 1
    assert lib.lora_debug_mask(4, 4, 1.5, 1, ok_ptr, None) == 4
    # per-adapter ranks: each 16, 32 or 64 and at most the allocated rank
    offs = (C.c_int64 * 3)(0, 64, 128)
    mr = lib.multi_lora_fwd_ranked
    for bad in ((16, 48), (64, 16), (0, 16)):
        ranks = (C.c_int32 * 2)(*bad)
        assert mr(ok_ptr, ok_ptr, ok_ptr, ok_ptr, 128, 64, 64, 32, 2, offs, ranks, s, p, sd, ok_ptr, ok_ptr, None) == 7
    ranks = (C.c_int32 * 2)(16, 32)
    assert mr(None, ok_ptr, ok_ptr, ok_ptr, 128, 64, 64, 32, 2, offs, ranks, s, p, sd, ok_ptr, ok_ptr, None) == 1
    need = lib.lora_bwd_workspace_bytes(128, 64, 64, 32, 2)
    mb = lib.multi_lora_bwd_ranked
    assert mb(ok_ptr, ok_ptr, ok_ptr, ok_ptr, ok_ptr, ok_ptr, 128, 64, 64, 32, 2, offs, ranks, s, p, sd,
              ok_ptr, ok_ptr, ok_ptr, 0, C.c_void_p(0x100000), need - 1, None) == 6


def test_noalloc_backward_validates_on_the_host(lib):
    """lora_bwd_noalloc refuses bad arguments and problems beyond its built-in scratch before it touches a GPU."""
    ok = C.c_void_p(0x1000)
    f = lib.lora_bwd_noalloc
    f.argtypes = [C.c_void_p] * 6 + [C.c_int64] * 3 + [C.c_int32, C.c_float, C.c_float, C.c_uint64] + [C.c_void_p] * 3 + [C.c_int, C.c_void_p]
    f.restype = C.c_int
    assert f(ok, None, ok, ok, ok, ok, 256, 128, 128, 16, 1.0, 0.1, 1, ok, ok, ok, 0, None) == 1
    assert f(ok, ok, ok, ok, ok, ok, 256, 100, 128, 16, 1.0, 0.1, 1, ok, ok, ok, 0, None) == 7
    assert f(ok, ok, ok, ok, ok, ok, 256, 128, 128, 16, 1.0, 1.5, 1, ok, ok, ok, 0, None) == 4
    assert f(ok, ok, ok, ok, ok, C.c_void_p(0x1004), 256, 128, 128, 16, 1.0, 0.1, 1, ok, ok, ok, 0, None) == 3
    assert f(ok, ok, ok, ok, ok, ok, 16384, 8192, 8192, 64, 1.0, 0.1, 1, ok, ok, ok, 0, None) == 6
    assert b"scratch" in lib.lora_status_string(6)


@pytest.mark.parametrize("M,K,N,r", [(8192, 4096, 4096, 32), (2048, 14336, 14336, 32), (40000, 4096, 4096, 16)])
def test_noalloc_limit_follows_the_sizes(lib, M, K, N, r):
    """The scratch limit counts a plane per panel of the fill rule, also where the launches write fewer planes or none
    (8192 x 4096 x 4096, r = 32: 2 x 16 MiB of planes, of which dA's launch writes 2 MiB)."""
    ok = C.c_void_p(0x1000)
    f = lib.lora_bwd_noalloc
    f.argtypes = [C.c_void_p] * 6 + [C.c_int64] * 3 + [C.c_int32, C.c_float, C.c_float, C.c_uint64] + [C.c_void_p] * 3 + [C.c_int, C.c_void_p]
    f.restype = C.c_int
    assert f(ok, ok, ok, ok, ok, ok, M, K, N, r, 1.0, 0.1, 1, ok, ok, ok, 0, None) == 6


def test_workspace_holds_every_panel_choice(lib):
    """Host logic: whatever row-panel height the streaming reductions pick (all three row-tile settings), the
    number of partial planes stays within what the workspace query provides for."""
    import random
    rnd = random.Random(5)
    f = lib.lora_debug_stream_panels
    f.argtypes = [C.c_int64, C.c_int64, C.c_int32, C.POINTER(C.c_int64), C.POINTER(C.c_int32),
                  C.POINTER(C.c_int64), C.POINTER(C.c_int64)]
    rows, panels, bound = C.c_int32(), C.c_int64(), C.c_int64()
    heights = set()
    try:
        for it in range(3000):
            G = rnd.randint(1, 64)
            mode = it % 4
            lens = [rnd.randrange(300) if mode == 0 else rnd.randrange(40) * 64 if mode == 1 else rnd.randrange(5000)
                    if mode == 2 else rnd.choice((0, rnd.randint(1, 130))) for _ in range(G)]
            if sum(lens) == 0:
                lens[0] = 1
            offs = [0]
            for v in lens:
                offs.append(offs[-1] + v)
            arr = (C.c_int64 * (G + 1))(*offs)
            for setting in (0, 128, 256):
                assert lib.lora_set_row_tile(setting) == 0
                for cols in (64, 512, 4096, 14336, 28672):
                    assert f(offs[-1], cols, G, arr, C.byref(rows), C.byref(panels), C.byref(bound)) == 0
                    assert rows.value in (64, 128, 256, 512, 1024) and (setting != 256 or rows.value >= 256)
                    assert 0 < panels.value <= bound.value, (offs, cols, setting, rows.value, panels.value, bound.value)
                    heights.add(rows.value)
    finally:
        lib.lora_set_row_tile(0)
    assert heights == {64, 128, 256, 512, 1024}


def test_ceiling_diagnostics_validate_on_the_host(lib):
    """The measured-ceiling launches check their arguments before anything is enqueued."""
    ok_ptr = C.c_void_p(0x1000)
    flops = C.c_double(0.0)
    m = lib.lora_ceiling_mfma
    assert m(None, ok_ptr, 256, 16, 16, C.byref(flops), None) == 1
    assert m(ok_ptr, None, 256, 16, 32, C.byref(flops), None) == 1
    assert m(ok_ptr, ok_ptr, 0, 16, 16, C.byref(flops), None) == 4
    assert m(ok_ptr, ok_ptr, 256, 0, 16, C.byref(flops), None) == 4
    assert m(ok_ptr, ok_ptr, 256, 16, 8, C.byref(flops), None) == 4          # neither MFMA shape
    assert m(C.c_void_p(0x1008), ok_ptr, 256, 16, 16, C.byref(flops), None) == 3
    r = lib.lora_ceiling_hbm_read
    assert r(None, 1 << 20, ok_ptr, 256, None) == 1
    assert r(ok_ptr, 1 << 20, None, 256, None) == 1
    assert r(ok_ptr, 8, ok_ptr, 256, None) == 4
    assert r(ok_ptr, 1 << 20, ok_ptr, 0, None) == 4
    assert r(C.c_void_p(0x1004), 1 << 20, ok_ptr, 256, None) == 3


def test_bench_refuses_more_than_one_gpu():
    """bench.py measures one GPU; a request for more ends with a message before anything touches a device."""
    import subprocess
    import sys
    out = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                         timeout=120)
    assert out.returncode != 0
    assert "ONE GPU" in (out.stderr + out.stdout)
