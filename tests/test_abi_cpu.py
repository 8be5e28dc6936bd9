"""Host-side checks of the C ABI that need no GPU: the library loads, exports
every function include/dfp4.h declares, reports the formatbook the oracle
uses, and rejects bad arguments before touching the device."""
import ctypes
import importlib.util
import os
import re

import pytest

from oracle import dfp4_oracle as O
from paper_2501_01144_amd import dfp4

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(dfp4.lib_path()):
        from paper_2501_01144_amd.build import build_library
        build_library(verbose=False)
    return dfp4.load()


def _declared_functions():
    text = open(os.path.join(ROOT, "include", "dfp4.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b((?:dfp4|mxfp4)_[a-z0-9_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = _declared_functions()
    assert len(names) >= 10
    assert sorted(dfp4.SYMBOLS) == names
    for n in names:
        assert getattr(lib, n) is not None


def test_formatbook_matches_the_oracle_table(lib):
    assert dfp4.formatbook() == O.FORMATBOOK_HALF_UNITS.tolist()


def test_strerror(lib):
    assert dfp4.strerror(0) == "ok"
    for code in range(-6, 0):
        assert dfp4.strerror(code) not in ("ok", "unknown error")
    assert dfp4.strerror(-99) == "unknown error"


def _t(codes=0, dialect=0, exponent=0, rows=0, K=0):
    return dfp4._CTensor(codes, dialect, exponent, rows, K)


def test_argument_errors_are_reported_without_a_device(lib):
    vp = ctypes.c_void_p
    # K not a multiple of 32, negative rows, ld < K, mismatched out shape
    assert lib.dfp4_quantize(vp(16), 4, 48, 48, _t(16, 16, 16, 4, 48), vp(0)) == -2
    assert lib.dfp4_quantize(vp(16), -1, 64, 64, _t(16, 16, 16, -1, 64), vp(0)) == -2
    assert lib.dfp4_quantize(vp(16), 4, 64, 32, _t(16, 16, 16, 4, 64), vp(0)) == -2
    assert lib.dfp4_quantize(vp(16), 4, 64, 64, _t(16, 16, 16, 4, 32), vp(0)) == -2
    # null pointers
    assert lib.dfp4_quantize(vp(0), 4, 64, 64, _t(16, 16, 16, 4, 64), vp(0)) == -1
    assert lib.dfp4_quantize(vp(16), 4, 64, 64, _t(16, 0, 16, 4, 64), vp(0)) == -1
    assert lib.mxfp4_quantize(vp(16), 4, 64, 64, _t(0, 0, 16, 4, 64), vp(0)) == -1
    # alignment: x must be 16-byte aligned, ld a multiple of 8
    assert lib.dfp4_quantize(vp(8), 4, 64, 64, _t(16, 16, 16, 4, 64), vp(0)) == -3
    assert lib.dfp4_quantize(vp(16), 4, 64, 68, _t(16, 16, 16, 4, 64), vp(0)) == -3
    # dtype
    assert lib.dfp4_dequantize(_t(16, 16, 16, 4, 64), vp(16), 7, 64, vp(0)) == -4
    assert lib.dfp4_gemm(_t(16, 16, 16, 4, 64), _t(16, 16, 16, 4, 64), vp(16), 9, 4, vp(0), 0, vp(0)) == -4
    # gemm: mismatched K, ldc < N, null output
    assert lib.dfp4_gemm(_t(16, 16, 16, 4, 64), _t(16, 16, 16, 4, 96), vp(16), 0, 4, vp(0), 0, vp(0)) == -2
    assert lib.dfp4_gemm(_t(16, 16, 16, 4, 64), _t(16, 16, 16, 8, 64), vp(16), 0, 4, vp(0), 0, vp(0)) == -2
    assert lib.dfp4_gemm(_t(16, 16, 16, 4, 64), _t(16, 16, 16, 4, 64), vp(0), 0, 4, vp(0), 0, vp(0)) == -1
    # empty problems succeed as no-ops
    assert lib.dfp4_quantize(vp(0), 0, 64, 64, _t(0, 0, 0, 0, 64), vp(0)) == 0
    assert lib.dfp4_gemm(_t(0, 0, 0, 0, 64), _t(16, 16, 16, 4, 64), vp(0), 0, 4, vp(0), 0, vp(0)) == 0
    assert lib.dfp4_formatbook(vp(0)) == -1


def test_binding_refuses_to_run_without_the_library(monkeypatch):
    monkeypatch.setattr(dfp4, "_lib", None)
    monkeypatch.setattr(dfp4, "_LIB_PATH", "/nonexistent/libdfp4.so")
    with pytest.raises(dfp4.Dfp4Error):
        dfp4.load()


def test_header_compiles_as_c99(tmp_path):
    # the boundary is a C ABI: the public header must be plain C
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no C compiler")
    header = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include", "dfp4.h")
    src = tmp_path / "t.c"
    src.write_text('#include "%s"\nint main(void) { return dfp4_strerror(0) == 0; }\n' % header)
    subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror", "-c", str(src), "-o",
                    str(tmp_path / "t.o")], check=True)


def test_argument_errors_of_the_later_entry_points(lib):
    vp, sz = ctypes.c_void_p, ctypes.c_size_t
    q = _t(16, 16, 16, 64, 64)
    # MSE and transposing quantizers: same checks as dfp4_quantize; the transposing one needs rows % 32 == 0
    assert lib.dfp4_quantize_mse(vp(16), 4, 48, 48, _t(16, 16, 16, 4, 48), vp(0)) == -2
    assert lib.dfp4_quantize_mse(vp(0), 4, 64, 64, _t(16, 16, 16, 4, 64), vp(0)) == -1
    assert lib.dfp4_quantize_t(vp(16), 48, 64, 64, _t(16, 16, 16, 64, 48), vp(0)) == -2
    assert lib.dfp4_quantize_t(vp(16), 64, 64, 64, _t(16, 16, 16, 64, 32), vp(0)) == -2
    assert lib.dfp4_quantize_t(vp(8), 64, 64, 64, q, vp(0)) == -3
    assert lib.mxfp4_quantize_t(vp(16), 64, 64, 64, _t(0, 0, 16, 64, 64), vp(0)) == -1
    # requantizing GEMM: N must be a multiple of 32, the output shape [M, N], a workspace is required
    a, w = _t(16, 16, 16, 64, 64), _t(16, 16, 16, 48, 64)
    assert lib.dfp4_gemm_requant(a, w, _t(16, 16, 16, 64, 48), vp(256), sz(1 << 30), vp(0)) == -2
    w = _t(16, 16, 16, 64, 64)
    assert lib.dfp4_gemm_requant(a, w, _t(16, 16, 16, 64, 32), vp(256), sz(1 << 30), vp(0)) == -2
    assert lib.dfp4_gemm_requant(a, w, _t(0, 16, 16, 64, 64), vp(256), sz(1 << 30), vp(0)) == -1
    assert lib.dfp4_gemm_requant(a, w, q, vp(0), sz(0), vp(0)) == -5
    assert lib.dfp4_gemm_requant_workspace_bytes(64, 64, 64) > lib.dfp4_gemm_workspace_bytes(64, 64, 64)
    # native family: packed sizes, workspace and alignment checks
    need = lib.dfp4_native_packed_bytes(64, 64)
    assert need > 0 and lib.dfp4_native_packed_bytes(0, 64) == 0
    assert lib.dfp4_native_pack(a, vp(256), sz(need - 1), vp(0)) == -5
    assert lib.dfp4_native_pack(a, vp(128), sz(need), vp(0)) == -3
    assert lib.dfp4_native_pack(_t(16, 0, 16, 64, 64), vp(256), sz(need), vp(0)) == -1
    assert lib.mxfp4_native_pack(_t(16, 0, 16, 64, 48), vp(256), sz(need), vp(0)) == -2
    assert lib.dfp4_quantize_native(vp(16), 64, 64, 64, vp(256), sz(need - 1), vp(0)) == -5
    assert lib.dfp4_quantize_native(vp(16), 64, 64, 32, vp(256), sz(need), vp(0)) == -2
    assert lib.dfp4_gemm_native(a, w, vp(16), 0, 64, vp(256), sz(need), vp(0)) == -5          # two operands do not fit
    assert lib.dfp4_gemm_native(a, _t(16, 16, 16, 64, 96), vp(16), 0, 64, vp(256), sz(1 << 30), vp(0)) == -2
    assert lib.dfp4_gemm_native(a, w, vp(16), 3, 64, vp(256), sz(1 << 30), vp(0)) == -4
    assert lib.dfp4_gemm_native_packed_w(a, vp(0), 64, vp(16), 0, 64, vp(256), sz(1 << 30), vp(0)) == -1
    assert lib.dfp4_gemm_native_packed(vp(256), 64, vp(256), 64, 48, vp(16), 0, 64, vp(0), sz(0), vp(0)) == -2
    assert lib.dfp4_gemm_native_packed(vp(256), 64, vp(128), 64, 64, vp(16), 0, 64, vp(0), sz(0), vp(0)) == -3
    assert lib.dfp4_gemm_native_packed(vp(256), 0, vp(256), 64, 64, vp(16), 0, 64, vp(0), sz(0), vp(0)) == 0


def test_gemm_noalloc_argument_errors(lib):
    vp = ctypes.c_void_p
    # a product whose workspace exceeds the library's fixed scratch array is refused before anything else
    big_a, big_w = _t(16, 16, 16, 2048, 14336), _t(16, 16, 16, 4096, 14336)
    assert lib.dfp4_gemm_workspace_bytes(2048, 4096, 14336) > (64 << 20)
    assert lib.dfp4_gemm_noalloc(big_a, big_w, vp(16), 0, 4096, vp(0)) == -5
    assert b"workspace" in lib.dfp4_strerror(-5)
    # more than the scratch array only as one of a batch: the single product needs none and is not refused for it (its null
    # output is found next)
    assert lib.dfp4_gemm_workspace_bytes(4141, 518, 12576) > (64 << 20) and lib.dfp4_gemm_path(4141, 518, 12576, 1, 0) > 0
    assert lib.dfp4_gemm_noalloc(_t(16, 16, 16, 4141, 12576), _t(16, 16, 16, 518, 12576), vp(0), 0, 518, vp(0)) == -1
    # the other checks are those of dfp4_gemm
    assert lib.dfp4_gemm_noalloc(_t(16, 16, 16, 4, 64), _t(16, 16, 16, 4, 96), vp(16), 0, 4, vp(0)) == -2
    assert lib.dfp4_gemm_noalloc(_t(16, 16, 16, 4, 64), _t(16, 16, 16, 4, 64), vp(16), 9, 4, vp(0)) == -4
    assert lib.dfp4_gemm_noalloc(_t(16, 16, 16, 4, 64), _t(16, 16, 16, 4, 64), vp(0), 0, 4, vp(0)) == -1
    assert lib.dfp4_gemm_noalloc(_t(0, 0, 0, 0, 64), _t(16, 16, 16, 4, 64), vp(0), 0, 4, vp(0)) == 0


def test_block_size_entry_points_argument_errors(lib):
    vp, sz = ctypes.c_void_p, ctypes.c_size_t
    q = _t(16, 16, 16, 4, 64)
    assert lib.dfp4_quantize_block(vp(16), 4, 64, 64, 8, q, vp(0)) == -2          # block size not 16 / 32 / 64
    assert lib.dfp4_quantize_block(vp(16), 4, 96, 96, 64, _t(16, 16, 16, 4, 96), vp(0)) == -2   # K % 64
    assert lib.dfp4_quantize_block(vp(0), 4, 64, 64, 16, q, vp(0)) == -1
    assert lib.dfp4_quantize_block(vp(16), 0, 64, 64, 16, _t(0, 0, 0, 0, 64), vp(0)) == 0
    assert lib.dfp4_dequantize_block(q, 48, vp(16), 0, 64, vp(0)) == -2
    assert lib.dfp4_dequantize_block(q, 16, vp(16), 5, 64, vp(0)) == -4
    assert lib.dfp4_gemm_blocks(q, 16, _t(16, 16, 16, 4, 96), 16, vp(16), 0, 4, vp(0), sz(0), vp(0)) == -2
    assert lib.dfp4_gemm_blocks(q, 16, q, 24, vp(16), 0, 4, vp(0), sz(0), vp(0)) == -2
    assert lib.dfp4_gemm_blocks(q, 16, q, 16, vp(0), 0, 4, vp(0), sz(0), vp(0)) == -1


def test_gemm_requant_batched_argument_errors(lib):
    vp, sz = ctypes.c_void_p, ctypes.c_size_t
    a, w = _t(16, 16, 16, 64, 64), _t(16, 16, 16, 64, 64)
    assert lib.dfp4_gemm_requant_batched(a, w, _t(16, 16, 16, 64, 64), 2, 64, 64, vp(256), sz(1 << 30), vp(0)) == -2   # out.rows != batch * M
    assert lib.dfp4_gemm_requant_batched(a, w, _t(16, 16, 16, 128, 64), 2, 64, 64, vp(0), sz(0), vp(0)) == -5
    assert lib.dfp4_gemm_requant_batched(a, w, _t(16, 16, 16, 128, 64), -1, 64, 64, vp(256), sz(1 << 30), vp(0)) == -2
    assert lib.dfp4_gemm_requant_batched(a, w, _t(16, 16, 16, 0, 64), 0, 64, 64, vp(0), sz(0), vp(0)) == 0


def test_gemm_prepared_refuses_a_weight_beyond_its_limit(lib):
    # rows * K / 2 < 2^31 for W (dfp4_gemm_prepare refuses such a W): also where A has few rows
    vp, sz = ctypes.c_void_p, ctypes.c_size_t
    big = _t(256, 256, 256, 1 << 18, 16384)
    assert lib.dfp4_gemm_prepare(big, 1, vp(256), sz(1 << 62), vp(0)) == -2
    for rows in (1, 64, 256, 300):
        a = _t(256, 256, 256, rows, 16384)
        assert lib.dfp4_gemm_prepared(a, vp(256), big, vp(256), vp(256), 0, 1 << 18, vp(256), sz(1 << 40), vp(0)) == -2


@pytest.mark.parametrize("M,N,K,batch,prepared,large", [
    # microseconds of the large kernel (with its prepass unless prepared) and of the best shape of gemm_f8_kernel; the line is that of the int8
    # kernels before them, and the large kernel is the faster one of three that it does not get
    (2048, 4096, 14336, 1, 0, True),       # 101, 190
    (1536, 4096, 14336, 1, 0, True),       # 84, 174
    (2048, 2048, 14336, 1, 0, True),       # 72, 124
    (2048, 4096, 11008, 1, 0, True),       # 81, 146
    (1024, 14336, 4096, 1, 0, True),       # 61, 109
    (3067, 1281, 14464, 1, 0, True),       # 83, 198
    (4096, 4096, 4096, 1, 0, True),        # 55, 114
    (512, 14336, 4096, 1, 1, True),        # 23, 57
    (2048, 4096, 4096, 1, 0, False),       # 40, 59
    (777, 3001, 2080, 1, 0, False),        # 33, 24
    (512, 4096, 14336, 1, 0, False),       # 70, 101
    (1024, 1024, 4096, 1, 0, False),       # 56, 18
    (2048, 128, 2048, 128, 0, False),      # 308, 153
    (2048, 2048, 128, 128, 0, False),      # 567, 360
    (400, 2759, 6592, 1, 1, False),        # 34, 44
    (64, 28672, 16384, 1, 0, False), (1, 32, 32, 1, 0, False), (700, 700, 16416, 1, 1, False)])     # the only kernel
def test_gemm_path_of_sizes(lib, M, N, K, batch, prepared, large):
    path = lib.dfp4_gemm_path(M, N, K, batch, prepared)
    assert 0 <= path <= 7 and (path == 0) == large


def test_gemm_path_of_short_k_and_of_errors(lib):
    # K of one iteration: small tiles while they are few (4.7 against 8 microseconds), the one-iteration form beyond
    assert dfp4.gemm_path(1, 256, 128) == 1 and dfp4.gemm_path(60, 700, 64) == 1
    assert dfp4.gemm_path(2048, 4096, 128) == 7 and dfp4.gemm_path(1, 2048, 128, batch=128) == 7
    assert dfp4.gemm_path(2048, 4096, 160) != 7
    for bad in ((0, 4, 32, 1), (4, 0, 32, 1), (4, 4, 33, 1), (4, 4, 32, 0), (4, 4, -32, 1)):
        assert lib.dfp4_gemm_path(*bad, 0) == -2


def test_a_native_module_that_does_not_load_says_why(monkeypatch):
    import sys
    import paper_2501_01144_amd as package
    monkeypatch.setattr(dfp4, "_lib", None)
    monkeypatch.setattr(dfp4, "_native", None)
    monkeypatch.delattr(package, "_binding", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2501_01144_amd._binding", None)
    with pytest.raises(dfp4.Dfp4Error, match="halted"):                # the import system's own words
        dfp4.load()


# --------------------------------------------------------------------------
# Main loop of gemm_native_kernel, from its generator: what its entry executes for a number of iterations.
# --------------------------------------------------------------------------
@pytest.mark.parametrize("fp6,ta", [(False, 4), (True, 4), (False, 2), (True, 2)])
@pytest.mark.parametrize("iters", [1, 2, 3, 4, 5, 64])
def test_native_loop_first_loads_no_more_than_there_is(fp6, ta, iters):
    spec = importlib.util.spec_from_file_location("gen_native_loop", os.path.join(os.path.dirname(dfp4.__file__), "csrc", "gen_native_loop.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    f = gen.Fmt(fp6, ta)
    lines = gen.main_loop(f)
    loads, steps, pending, scc, at = 0, 0, None, False, 0
    while "s_barrier" not in lines[at]:
        op, *args = lines[at].replace(",", " ").split()
        at += 1
        if op.startswith("global_load_lds"):
            loads += 1
        elif op == "v_add_u32" and args[0] == args[2] == gen.vr(gen.VOFF):
            steps += 1                                       # to the next step's operands
        elif op == "s_waitcnt":
            pending = int(re.search(r"vmcnt\((\d+)\)", args[0]).group(1))
        elif op == "s_cmp_eq_u32" and args[0] == "%[iters]":
            scc = iters == int(args[1])
        elif op == "s_branch" or op == "s_cbranch_scc1" and scc:
            at = lines.index(args[0][:-1] + ":", at if args[0][-1] == "f" else 0)
    slots = min(iters, f.slots)
    assert loads == 2 * slots * f.per_step and steps == 2 * slots
    # the first iteration's loads, of two steps, have landed at the barrier; where the fill was cut short all have, since the loop counts
    # on f.slots iterations of them
    assert pending == (0 if iters < f.slots else (f.slots - 1) * 2 * f.per_step)


@pytest.mark.parametrize("M,N,K,ranges", [
    # microseconds (FP6, fp32) whole / in 2 ranges of K / in 4
    (231, 5376, 6048, 2),         # 24.1, 21.2
    (1024, 1216, 6176, 2),        # 25.4, 22.2, 23.5
    (361, 2048, 3936, 4),         # 15.7, 14.3, 13.1
    (65, 4096, 2560, 4),          # 11.9, 11.1, 10.0
    (512, 4096, 14336, 4),        # 46.7, 36.1, 33.9
    (256, 1024, 4096, 4),         # 15.8, 13.0, 11.6
    (512, 4096, 4096, 1),         # 17.4, 20.4, 22.8
    (461, 4940, 2368, 1),         # 13.4, 19.1
    (3136, 767, 1280, 1),         # 10.9, 20.9
    (2048, 14336, 4096, 1), (64, 64, 480, 1)])
def test_native_k_is_split_where_it_pays(lib, M, N, K, ranges):
    # the room asked for is enough for either format and type of the results; these sizes are FP6's to choose
    lib.dfp4_gemm_native_splitk_bytes.restype = ctypes.c_size_t
    need = lib.dfp4_gemm_native_splitk_bytes(ctypes.c_int64(M), ctypes.c_int64(N), ctypes.c_int64(K))
    assert need == (-(-ranges * M * N * 4 // 256) * 256 if ranges > 1 else 0)
