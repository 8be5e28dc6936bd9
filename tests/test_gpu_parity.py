"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on
the same seeded inputs.  Quantizer outputs (codes, dialect ids, exponent
bytes) must match bit for bit; dequantization is exact; the GEMM must satisfy
|out - ref| <= 1e-5 * sum_k |A^[m,k]| |W^[n,k]| with ref the float64 product of
the oracle's dequantized operands."""
import numpy as np
import pytest
import torch

from oracle import dfp4_oracle as O
from oracle import mxfp4_oracle as MX
from paper_2501_01144_amd import dfp4, synth

pytestmark = pytest.mark.gpu
GEMM_RTOL = 1e-5


@pytest.fixture(scope="module", autouse=True)
def _library():
    assert torch.cuda.is_available(), "GPU tests need a device"
    dfp4.load()


def _dev(x):
    return x.cuda()


def _np(t):
    return t.cpu().numpy()


def _assert_quant_equal(q, ref, what):
    codes, dialect, expo = ref
    got_e, got_d, got_c = _np(q.exponent), _np(q.dialect), _np(q.codes)
    assert np.array_equal(got_e, expo), f"{what}: exponent bytes differ at {np.argwhere(got_e != expo)[:4]}"
    assert np.array_equal(got_d, dialect), f"{what}: dialect ids differ at {np.argwhere(got_d != dialect)[:4]}"
    assert np.array_equal(got_c, codes), f"{what}: codes differ at {np.argwhere(got_c != codes)[:4]}"


def _check_quantize(x_bf16, what):
    print(f"quantize parity: {what} shape={tuple(x_bf16.shape)}", flush=True)
    q = dfp4.quantize(_dev(x_bf16))
    torch.cuda.synchronize()
    _assert_quant_equal(q, O.dfp4_quantize(synth.to_f64(x_bf16)), what)
    qm = dfp4.mxfp4_quantize(_dev(x_bf16))
    torch.cuda.synchronize()
    codes, expo = MX.mxfp4_quantize(synth.to_f64(x_bf16))
    assert np.array_equal(_np(qm.exponent), expo), f"{what}: mx exponent"
    assert np.array_equal(_np(qm.codes), codes), f"{what}: mx codes at {np.argwhere(_np(qm.codes) != codes)[:4]}"
    return q, qm


# --------------------------------------------------------------------------
# quantizer
# --------------------------------------------------------------------------
def test_quantize_single_linear_activation():
    a, _ = synth.single_linear(seed=0)
    _check_quantize(a, "config1 A")


@pytest.mark.parametrize("rows,K", [(1, 32), (3, 96), (5, 2048), (65, 64), (127, 4096), (1000, 1056)])
def test_quantize_ragged_shapes(rows, K):
    # sizes that end inside a wavefront's 64-block group and inside a 16-block load
    _check_quantize(synth.student_t(rows, K, 3.0, seed=rows + K), f"t3 {rows}x{K}")


def test_quantize_every_bf16_value():
    x = synth.all_bf16_bit_patterns()                       # [2040, 32]: one block per row
    _check_quantize(x, "all finite bf16 patterns")
    # each value also as a lone element next to a larger block maximum
    g = torch.Generator().manual_seed(1)
    y = x[torch.randperm(x.shape[0], generator=g)].reshape(-1, 64)
    _check_quantize(y, "all finite bf16 patterns, shuffled pairs of rows")


def test_quantize_degenerate_blocks():
    x = torch.zeros(8, 128, dtype=torch.bfloat16)
    x[1, 5] = -0.0
    x[2, 40] = 1.0                                          # single nonzero
    x[3, :32] = 7.875                                       # rounded maximum 8.0
    x[3, 32:64] = 7.75
    x[4, 64:96] = torch.tensor(2.0 ** -133).to(torch.bfloat16)   # smallest subnormal
    x[5, :] = torch.tensor(3.3895e38).to(torch.bfloat16)    # largest finite
    x[6, ::3] = -1.5
    x[7, 96:] = torch.linspace(-8, 8, 32).to(torch.bfloat16)
    _check_quantize(x, "degenerate blocks")


def test_quantize_wide_dynamic_range_and_ties():
    g = torch.Generator().manual_seed(4)
    x = torch.randn(256, 512, generator=g) * torch.exp2(torch.randint(-120, 120, (256, 16), generator=g)
                                                        .repeat_interleave(32, dim=1).float())
    _check_quantize(x.to(torch.bfloat16), "wide range")
    ties = (torch.randint(-64, 64, (256, 512), generator=g).float() / 8).to(torch.bfloat16)
    _check_quantize(ties, "multiples of 1/8 (every rounding tie)")


def test_quantize_strided_rows():
    base = synth.student_t(64, 1024, 3.0, seed=9)
    view = base[:, 128:128 + 512]                           # ld = 1024, K = 512
    q = dfp4.quantize(_dev(base)[:, 128:128 + 512])
    torch.cuda.synchronize()
    _assert_quant_equal(q, O.dfp4_quantize(synth.to_f64(view.contiguous())), "strided")


def test_quantize_streaming_tensor_sampled_rows():
    # full-size streaming tensor in the benchmark's launch configuration;
    # the oracle checks a seeded sample of rows
    x = synth.student_t(8192, 4096, 3.0, seed=3)
    q = dfp4.quantize(_dev(x))
    qm = dfp4.mxfp4_quantize(_dev(x))
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(0).choice(8192, 96, replace=False))
    rows = np.concatenate([rows, [0, 8191]])
    ref = O.dfp4_quantize(synth.to_f64(x[rows]))
    assert np.array_equal(_np(q.codes)[rows], ref[0])
    assert np.array_equal(_np(q.dialect)[rows], ref[1])
    assert np.array_equal(_np(q.exponent)[rows], ref[2])
    refm = MX.mxfp4_quantize(synth.to_f64(x[rows]))
    assert np.array_equal(_np(qm.codes)[rows], refm[0])
    assert np.array_equal(_np(qm.exponent)[rows], refm[1])
    # properties that hold at any size: ids in range, exponent = max exponent field - 2
    assert int(q.dialect.max()) <= 15
    amax = x.abs().view(8192, -1, 32).amax(dim=2).float()
    _, ex = torch.frexp(amax)                               # amax = m * 2^ex, m in [0.5, 1)
    want = torch.where(amax == 0, torch.zeros_like(ex), torch.clamp(ex - 1 - 2 + 127, min=0)).to(torch.uint8)
    assert torch.equal(q.exponent.cpu(), want)


def test_quantize_second_streaming_tensor_sampled_rows():
    # 4096 x 14336 Student-t tensor (448 blocks per row) in the benchmark's launch configuration
    x = synth.student_t(4096, 14336, 3.0, seed=4)
    print("quantize parity: 4096x14336 sampled rows", flush=True)
    q = dfp4.quantize(_dev(x))
    qm = dfp4.mxfp4_quantize(_dev(x))
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(1).choice(4096, 48, replace=False))
    rows = np.concatenate([rows, [0, 4095]])
    ref = O.dfp4_quantize(synth.to_f64(x[rows]))
    assert np.array_equal(_np(q.codes)[rows], ref[0])
    assert np.array_equal(_np(q.dialect)[rows], ref[1])
    assert np.array_equal(_np(q.exponent)[rows], ref[2])
    refm = MX.mxfp4_quantize(synth.to_f64(x[rows]))
    assert np.array_equal(_np(qm.codes)[rows], refm[0])
    assert np.array_equal(_np(qm.exponent)[rows], refm[1])
    assert int(q.dialect.max()) <= 15
    amax = x.abs().view(4096, -1, 32).amax(dim=2).float()
    _, ex = torch.frexp(amax)
    want = torch.where(amax == 0, torch.zeros_like(ex), torch.clamp(ex - 1 - 2 + 127, min=0)).to(torch.uint8)
    assert torch.equal(q.exponent.cpu(), want)


# --------------------------------------------------------------------------
# dequantizer
# --------------------------------------------------------------------------
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_dequantize_exact(dtype):
    x = torch.cat([synth.student_t(37, 1088, 3.0, seed=12),
                   synth.all_bf16_bit_patterns().reshape(-1, 1088)])
    xf = synth.to_f64(x)
    q = dfp4.quantize(_dev(x))
    y = dfp4.dequantize(q, dtype)
    torch.cuda.synchronize()
    ref = O.dfp4_dequantize(*O.dfp4_quantize(xf))
    got = y.cpu().to(torch.float64).numpy()
    assert np.array_equal(got, ref)
    assert np.array_equal(np.signbit(got), np.signbit(ref))
    qm = dfp4.mxfp4_quantize(_dev(x))
    ym = dfp4.mxfp4_dequantize(qm, dtype)
    torch.cuda.synchronize()
    assert np.array_equal(ym.cpu().to(torch.float64).numpy(), MX.mxfp4_dequantize(*MX.mxfp4_quantize(xf)))


def test_dequantize_strided_output():
    x = synth.gaussian(16, 256, 1.0, seed=5)
    q = dfp4.quantize(_dev(x))
    buf = torch.full((16, 512), 99.0, dtype=torch.float32, device="cuda")
    dfp4.dequantize(q, out=buf[:, 64:64 + 256])
    torch.cuda.synchronize()
    ref = O.dfp4_dequantize(*O.dfp4_quantize(synth.to_f64(x)))
    assert np.array_equal(buf[:, 64:320].cpu().double().numpy(), ref)
    assert (buf[:, :64] == 99).all() and (buf[:, 320:] == 99).all()


# --------------------------------------------------------------------------
# GEMM
# --------------------------------------------------------------------------
def _gemm_ref(a_f64, w_f64, mx=False):
    if mx:
        ad = MX.mxfp4_dequantize(*MX.mxfp4_quantize(a_f64))
        wd = MX.mxfp4_dequantize(*MX.mxfp4_quantize(w_f64))
    else:
        ad = O.dfp4_dequantize(*O.dfp4_quantize(a_f64))
        wd = O.dfp4_dequantize(*O.dfp4_quantize(w_f64))
    return ad @ wd.T, np.abs(ad) @ np.abs(wd).T


def _assert_gemm_close(got, ref, absdot, what, bf16=False):
    got = got.cpu().to(torch.float64).numpy()
    if bf16:
        want = torch.from_numpy(ref).to(torch.bfloat16).to(torch.float64).numpy()
        ulp = np.exp2(np.floor(np.log2(np.maximum(np.abs(want), 1e-300))) - 7)
        assert (np.abs(got - want) <= ulp + GEMM_RTOL * absdot).all(), what
        return
    err = np.abs(got - ref)
    bad = err > GEMM_RTOL * absdot
    assert not bad.any(), f"{what}: {bad.sum()} outputs off, worst {np.max(err / np.maximum(absdot, 1e-300)):.3e}"


def test_gemm_single_linear_full():
    a, w = synth.single_linear(seed=0)
    print("gemm parity: config1 32x4096x4096", flush=True)
    out = dfp4.gemm(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    _assert_gemm_close(out, ref, absdot, "config1")
    outm = dfp4.mxfp4_gemm(dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w)))
    torch.cuda.synchronize()
    refm, absm = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
    _assert_gemm_close(outm, refm, absm, "config1 mxfp4")


@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (70, 200, 160), (129, 257, 96), (300, 130, 1024)])
def test_gemm_ragged_shapes(M, N, K):
    print(f"gemm parity: ragged {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 100), 50.0, 1.0, seed=M)
    w = synth.student_t(N, K, 3.0, seed=N)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    out = dfp4.gemm(qa, qw)
    torch.cuda.synchronize()
    _assert_gemm_close(out, ref, absdot, "f32")
    outb = dfp4.gemm(qa, qw, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    _assert_gemm_close(outb, ref, absdot, "bf16", bf16=True)
    # leading dimension larger than N, surroundings untouched
    buf = torch.full((M, N + 24), -7.0, dtype=torch.float32, device="cuda")
    dfp4.gemm(qa, qw, out=buf[:, 8:8 + N])
    torch.cuda.synchronize()
    _assert_gemm_close(buf[:, 8:8 + N], ref, absdot, "ldc")
    assert (buf[:, :8] == -7).all() and (buf[:, 8 + N:] == -7).all()


def test_gemm_wide_exponent_spread():
    # blocks whose exponents differ by tens of binades along K
    g = torch.Generator().manual_seed(6)
    scale = torch.exp2(torch.randint(-30, 30, (96, 8), generator=g).repeat_interleave(32, dim=1).float())
    a = (torch.randn(96, 256, generator=g) * scale).to(torch.bfloat16)
    w = (torch.randn(160, 256, generator=g) * scale[:1]).to(torch.bfloat16)
    out = dfp4.gemm(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    _assert_gemm_close(out, ref, absdot, "wide spread")


def test_gemm_batched():
    B, M, N, K = 3, 80, 144, 128
    a = synth.gaussian_outlier_channels(B * M, K, 2, 30.0, 1.0, seed=31)
    w = synth.gaussian_outlier_channels(B * N, K, 2, 30.0, 1.0, seed=32)
    out = dfp4.gemm_batched(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)), B, M, N)
    torch.cuda.synchronize()
    for b in range(B):
        ref, absdot = _gemm_ref(synth.to_f64(a[b * M:(b + 1) * M]), synth.to_f64(w[b * N:(b + 1) * N]))
        _assert_gemm_close(out[b], ref, absdot, f"batch {b}")


def test_gemm_mlp_prefill_sampled_outputs():
    # LLaMA-3-8B gate projection at full size, in the benchmark's launch
    # configuration; the oracle computes a seeded sample of rows x columns
    ops = synth.llama3_8b_mlp(seed=2)
    x, w = ops["x"], ops["w_gate"]
    print("gemm parity: 2048x14336x4096 sampled", flush=True)
    out = dfp4.gemm(dfp4.quantize(_dev(x)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    rng = np.random.default_rng(1)
    rows = np.sort(rng.choice(x.shape[0], 24, replace=False))
    cols = np.sort(rng.choice(w.shape[0], 192, replace=False))
    ref, absdot = _gemm_ref(synth.to_f64(x[rows]), synth.to_f64(w[cols]))
    _assert_gemm_close(out[rows][:, cols], ref, absdot, "mlp gate sampled")
    # down projection, K = 14336
    h, wd = ops["h"], ops["w_down"]
    out = dfp4.gemm(dfp4.quantize(_dev(h)), dfp4.quantize(_dev(wd)))
    torch.cuda.synchronize()
    cols = np.sort(rng.choice(wd.shape[0], 64, replace=False))
    ref, absdot = _gemm_ref(synth.to_f64(h[rows]), synth.to_f64(wd[cols]))
    _assert_gemm_close(out[rows][:, cols], ref, absdot, "mlp down sampled")


def test_gemm_mlp_prefill_bf16_sampled_outputs():
    # bf16 output of a full-size GEMM (full tiles store two adjacent columns per lane)
    ops = synth.llama3_8b_mlp(seed=2)
    x, w = ops["x"], ops["w_up"]
    print("gemm parity: 2048x14336x4096 bf16 sampled", flush=True)
    out = dfp4.gemm(dfp4.quantize(_dev(x)), dfp4.quantize(_dev(w)), dtype=torch.bfloat16)
    torch.cuda.synchronize()
    rng = np.random.default_rng(2)
    rows = np.sort(rng.choice(x.shape[0], 24, replace=False))
    cols = np.sort(rng.choice(w.shape[0], 192, replace=False))
    ref, absdot = _gemm_ref(synth.to_f64(x[rows]), synth.to_f64(w[cols]))
    _assert_gemm_close(out[rows][:, cols], ref, absdot, "mlp up bf16 sampled", bf16=True)


def test_gemm_some_tiles_declined():
    # rows 520..539 carry block exponents spread over tens of binades, so the second 512-row
    # tile goes to the per-block-flush fallback while the first one takes the fast path
    g = torch.Generator().manual_seed(9)
    M, N, K = 600, 300, 512
    a = torch.randn(M, K, generator=g)
    scale = torch.exp2(torch.randint(-25, 25, (20, K // 32), generator=g).repeat_interleave(32, dim=1).float())
    a[520:540] *= scale
    a = a.to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g) * 0.02).to(torch.bfloat16)
    print("gemm parity: 600x300x512 with declined tiles", flush=True)
    out = dfp4.gemm(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    _assert_gemm_close(out, ref, absdot, "mixed fast and declined tiles")


def test_gemm_llama2_down_projection_sampled_outputs():
    # LLaMA-2-7B down projection at M = 4096: K = 11008 is 344 blocks (not a multiple of 16)
    g = synth.llama2_7b_linears(seed=4)
    h, w = g["h"], g["w_down"]
    print("gemm parity: 4096x4096x11008 sampled", flush=True)
    out = dfp4.gemm(dfp4.quantize(_dev(h)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    rng = np.random.default_rng(4)
    rows = np.sort(rng.choice(h.shape[0], 16, replace=False))
    cols = np.sort(rng.choice(w.shape[0], 96, replace=False))
    ref, absdot = _gemm_ref(synth.to_f64(h[rows]), synth.to_f64(w[cols]))
    _assert_gemm_close(out[rows][:, cols], ref, absdot, "llama2 down sampled")


@pytest.mark.parametrize("name,N", [("w_qkv", 12288), ("w_o", 4096), ("w_gate", 11008)])
def test_gemm_llama2_linears_sampled_outputs(name, N):
    # the other LLaMA-2-7B linears at M = 4096, K = 4096, full size, sampled outputs
    g = synth.llama2_7b_linears(seed=4)
    x, w = g["x"], g[name]
    assert w.shape[0] == N
    print(f"gemm parity: 4096x{N}x4096 ({name}) sampled", flush=True)
    out = dfp4.gemm(dfp4.quantize(_dev(x)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    rng = np.random.default_rng(40 + N)
    rows = np.sort(np.concatenate([rng.choice(x.shape[0], 14, replace=False), [0, x.shape[0] - 1]]))
    cols = np.sort(np.concatenate([rng.choice(N, 94, replace=False), [0, N - 1]]))
    ref, absdot = _gemm_ref(synth.to_f64(x[rows]), synth.to_f64(w[cols]))
    _assert_gemm_close(out[rows][:, cols], ref, absdot, f"llama2 {name} sampled")


def test_gemm_attention_full_batch_first_and_last_head():
    # both attention products at the full batch of 4 x 32 = 128 heads; the oracle checks
    # sampled outputs of the first and the last head (the largest batch offsets)
    B, H, S, D = 4, 32, 2048, 128
    bh = B * H
    ops = synth.attention_operands(seed=5, B=B, H=H, S=S, D=D)
    q, k, vt = ops["q"], ops["k"], ops["vt"]
    print("gemm parity: attention 128 heads Q K^T", flush=True)
    out = dfp4.gemm_batched(dfp4.quantize(_dev(q.reshape(bh * S, D))), dfp4.quantize(_dev(k.reshape(bh * S, D))), bh, S, S)
    torch.cuda.synchronize()
    rng = np.random.default_rng(50)
    rows = np.sort(np.concatenate([rng.choice(S, 14, replace=False), [0, S - 1]]))
    cols = np.sort(np.concatenate([rng.choice(S, 126, replace=False), [0, S - 1]]))
    for hd in (0, 77, bh - 1):
        ref, absdot = _gemm_ref(synth.to_f64(q[hd][rows]), synth.to_f64(k[hd][cols]))
        _assert_gemm_close(out[hd][rows][:, cols], ref, absdot, f"QK^T head {hd}")
    del out
    print("gemm parity: attention 128 heads P V", flush=True)
    # P: softmax rows, generated per head to bound host memory; only the checked heads are kept
    qp = dfp4.empty_qtensor(bh * S, S, torch.device("cuda:0"))
    keep = {}
    for hd in range(bh):
        p = synth.softmax_rows(S, S, seed=5000 + hd)
        part = dfp4.quantize(_dev(p))
        qp.codes[hd * S:(hd + 1) * S] = part.codes
        qp.dialect[hd * S:(hd + 1) * S] = part.dialect
        qp.exponent[hd * S:(hd + 1) * S] = part.exponent
        if hd in (0, bh - 1):
            keep[hd] = p
    out = dfp4.gemm_batched(qp, dfp4.quantize(_dev(vt.reshape(bh * D, S))), bh, S, D)
    torch.cuda.synchronize()
    for hd in (0, bh - 1):
        ref, absdot = _gemm_ref(synth.to_f64(keep[hd][rows]), synth.to_f64(vt[hd]))
        _assert_gemm_close(out[hd][rows], ref, absdot, f"PV head {hd}")


def test_gemm_attention_shapes_batched_sampled():
    # attention matmuls at the real sequence length and head size, 4 of the 128 heads:
    # Q K^T (K = 128, blocks along the head dimension) and P V (K = 2048, blocks along the sequence)
    B, H, S, D = 1, 4, 2048, 128
    ops = synth.attention_operands(seed=5, B=B, H=H, S=S, D=D)
    q, k, vt = ops["q"], ops["k"], ops["vt"]
    print("gemm parity: attention 4 heads Q K^T", flush=True)
    out = dfp4.gemm_batched(dfp4.quantize(_dev(q.reshape(H * S, D))), dfp4.quantize(_dev(k.reshape(H * S, D))), H, S, S)
    torch.cuda.synchronize()
    rng = np.random.default_rng(5)
    rows = np.sort(rng.choice(S, 16, replace=False))
    cols = np.sort(rng.choice(S, 128, replace=False))
    for hd in (0, 3):
        ref, absdot = _gemm_ref(synth.to_f64(q[hd][rows]), synth.to_f64(k[hd][cols]))
        _assert_gemm_close(out[hd][rows][:, cols], ref, absdot, f"QK^T head {hd}")
    print("gemm parity: attention 4 heads P V", flush=True)
    p = synth.softmax_rows(H * S, S, seed=55)
    out = dfp4.gemm_batched(dfp4.quantize(_dev(p)), dfp4.quantize(_dev(vt.reshape(H * D, S))), H, S, D)
    torch.cuda.synchronize()
    for hd in (1, 2):
        ref, absdot = _gemm_ref(synth.to_f64(p[hd * S:(hd + 1) * S][rows]), synth.to_f64(vt[hd]))
        _assert_gemm_close(out[hd][rows], ref, absdot, f"PV head {hd}")


@pytest.mark.parametrize("M,N,K", [(5, 40, 64), (33, 100, 4096), (64, 96, 256), (16, 4096, 14336)])
def test_gemm_few_rows(M, N, K):
    # decode shapes (M <= 64) take the W-streaming kernel: per-block exponent pairs in fp32
    print(f"gemm parity: few rows {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 200), 50.0, 1.0, seed=100 + M)
    w = synth.gaussian(N, K, 0.02, seed=200 + N)
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    out = dfp4.gemm(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    _assert_gemm_close(out, ref, absdot, "few rows f32")
    outb = dfp4.gemm(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)), dtype=torch.bfloat16)
    torch.cuda.synchronize()
    _assert_gemm_close(outb, ref, absdot, "few rows bf16", bf16=True)
    refm, absm = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
    outm = dfp4.mxfp4_gemm(dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w)))
    torch.cuda.synchronize()
    _assert_gemm_close(outm, refm, absm, "few rows mxfp4")


@pytest.mark.parametrize("scale,K,exact", [(30.0, 4096, True), (2.0 ** 13, 512, False)])
def test_gemm_few_rows_both_forms_of_the_tile(scale, K, exact):
    # Nothing prepared, at most 64 rows: a tile whose exponents allow it is summed exactly in int32 (one
    # rounding of the exact sum, checked here to half an ulp); a tile with outliers 13 binades above the
    # rest cannot be and takes one fp32 term per block (held to the usual tolerance).
    M, N = 32, 96
    print(f"gemm parity: few rows {M}x{N}x{K}, outliers x{scale}, exact={exact}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, 4, scale, 1.0, seed=901)
    w = synth.gaussian(N, K, 0.02, seed=902)
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    out = dfp4.gemm(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    _assert_gemm_close(out, ref, absdot, "few rows, both forms")
    if exact:
        err = np.abs(out.cpu().double().numpy() - ref)
        assert (err <= np.abs(ref) * 2.0 ** -24 + 1e-300).all(), "more than one rounding of the exact sum"


def test_gemm_very_long_k_is_summed_exactly():
    # K beyond the large kernel's range (more than 512 blocks): gemm_f8_kernel, exact while the sum fits int32
    M, N, K = 70, 64, 32 * 520
    print(f"gemm parity: long K {M}x{N}x{K}", flush=True)
    a = synth.gaussian(M, K, 1.0, seed=71)
    w = synth.gaussian(N, K, 0.02, seed=72)
    out = dfp4.gemm(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    _assert_gemm_close(out, ref, absdot, "long K")
    assert (np.abs(out.cpu().double().numpy() - ref) <= np.abs(ref) * 2.0 ** -24 + 1e-300).all()


def test_gemm_batched_with_split_k():
    # few tiles per problem and a long K: the K ranges of every batch entry are summed separately
    B, M, N, K = 2, 100, 200, 2048
    print(f"gemm parity: batched split K {B}x{M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(B * M, K, 8, 50.0, 1.0, seed=81)
    w = synth.gaussian(B * N, K, 0.02, seed=82)
    out = dfp4.gemm_batched(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)), B, M, N)
    torch.cuda.synchronize()
    for b in range(B):
        ref, absdot = _gemm_ref(synth.to_f64(a[b * M:(b + 1) * M]), synth.to_f64(w[b * N:(b + 1) * N]))
        _assert_gemm_close(out[b], ref, absdot, f"batch {b}")


# --------------------------------------------------------------------------
# offline quantizer with MSE-based dialect selection
# --------------------------------------------------------------------------
def _check_quantize_mse(x_bf16, what):
    print(f"quantize_mse parity: {what} shape={tuple(x_bf16.shape)}", flush=True)
    q = dfp4.quantize_mse(_dev(x_bf16))
    torch.cuda.synchronize()
    _assert_quant_equal(q, O.dfp4_quantize_mse(synth.to_f64(x_bf16)), what)
    return q


@pytest.mark.parametrize("rows,K", [(1, 32), (7, 96), (33, 4096), (257, 1056)])
def test_quantize_mse_shapes(rows, K):
    _check_quantize_mse(synth.student_t(rows, K, 3.0, seed=rows + K), "student-t")
    _check_quantize_mse(synth.gaussian(rows, K, 0.02, seed=rows), "weights")


def test_quantize_mse_every_bf16_value_and_ties():
    _check_quantize_mse(synth.all_bf16_bit_patterns(), "all finite bf16 values")
    g = torch.Generator().manual_seed(12)
    grid = (torch.randint(-64, 64, (64, 256), generator=g).float() / 8.0).to(torch.bfloat16)   # many equal errors
    _check_quantize_mse(grid, "multiples of 1/8")
    scale = torch.exp2(torch.randint(-120, 120, (64, 8), generator=g).repeat_interleave(32, dim=1).float())
    _check_quantize_mse((torch.randn(64, 256, generator=g) * scale).to(torch.bfloat16), "wide range")
    _check_quantize_mse(torch.zeros(4, 64, dtype=torch.bfloat16), "zeros")


def test_gemm_with_mse_quantized_weights():
    M, N, K = 96, 160, 512
    a = synth.gaussian_outlier_channels(M, K, 4, 50.0, 1.0, seed=91)
    w = synth.gaussian(N, K, 0.02, seed=92)
    out = dfp4.gemm(dfp4.quantize(_dev(a)), dfp4.quantize_mse(_dev(w)))
    torch.cuda.synchronize()
    ad = O.dfp4_dequantize(*O.dfp4_quantize(synth.to_f64(a)))
    wd = O.dfp4_dequantize(*O.dfp4_quantize_mse(synth.to_f64(w)))
    _assert_gemm_close(out, ad @ wd.T, np.abs(ad) @ np.abs(wd).T, "mse weights")


# --------------------------------------------------------------------------
# transposing quantizer (blocks along the rows of the input)
# --------------------------------------------------------------------------
@pytest.mark.parametrize("rows,cols", [(32, 8), (96, 72), (2048, 128), (160, 264), (4096, 64)])
def test_quantize_transposed(rows, cols):
    print(f"quantize_t parity: {rows}x{cols}", flush=True)
    x = synth.gaussian_outlier_channels(rows, cols, max(1, cols // 64), 30.0, 1.0, seed=rows + cols)
    xt = synth.to_f64(x).T.copy()
    q = dfp4.quantize_t(_dev(x))
    torch.cuda.synchronize()
    assert (q.rows, q.K) == (cols, rows)
    _assert_quant_equal(q, O.dfp4_quantize(xt), "transposed")
    qm = dfp4.mxfp4_quantize_t(_dev(x))
    torch.cuda.synchronize()
    codes, expo = MX.mxfp4_quantize(xt)
    assert np.array_equal(_np(qm.exponent), expo) and np.array_equal(_np(qm.codes), codes)


def test_quantize_transposed_strided_input_and_pv_product():
    # V stored [S, D] inside a wider buffer; P V with V quantized along the sequence by the
    # transposing quantizer equals the product with an explicitly transposed V
    S, D = 256, 64
    buf = synth.gaussian(S, D + 16, 1.0, seed=77).cuda()
    v = buf[:, 8:8 + D]
    qv = dfp4.quantize_t(v)
    torch.cuda.synchronize()
    vt = synth.to_f64(v.cpu()).T.copy()
    _assert_quant_equal(qv, O.dfp4_quantize(vt), "strided transposed")
    p = synth.softmax_rows(96, S, seed=78)
    out = dfp4.gemm(dfp4.quantize(_dev(p)), qv)
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(p), vt)
    _assert_gemm_close(out, ref, absdot, "P V")


# --------------------------------------------------------------------------
# GEMM on operands prepared ahead (dfp4_gemm_prepare / dfp4_gemm_prepared)
# --------------------------------------------------------------------------
@pytest.mark.parametrize("M,N,K,why", [(600, 352, 512, "whole tiles"), (100, 256, 4096, "split K"),
                                       (2048, 1024, 2048, "many tiles"), (33, 100, 4096, "few rows"),
                                       (70, 200, 160, "ragged")])
def test_gemm_prepared_matches_oracle_and_gemm(M, N, K, why):
    print(f"gemm_prepared parity: {why} {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 200), 50.0, 1.0, seed=500 + M)
    w = synth.gaussian(N, K, 0.02, seed=600 + N)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    want = dfp4.gemm(qa, qw)
    # the same prepared A serves several products in a row (its arrival counters return to zero)
    for rep in range(3):
        out = dfp4.gemm_prepared(pa, pw)
        torch.cuda.synchronize()
        _assert_gemm_close(out, ref, absdot, f"prepared {why} rep {rep}")
        if M > 64:
            assert torch.equal(out.view(torch.int32), want.view(torch.int32)), "prepared and plain GEMM differ"
        else:
            # few rows: the prepared form takes the exact scheme (one rounding of the exact sum),
            # the plain call adds one fp32 term per block
            assert (np.abs(out.cpu().double().numpy() - ref) <= np.abs(ref) * 2.0 ** -23 + 1e-300).all()
    outb = dfp4.gemm_prepared(pa, pw, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    _assert_gemm_close(outb, ref, absdot, f"prepared {why} bf16", bf16=True)
    assert dfp4.gemm_declined_tiles(pa) == 0
    # MXFP4
    qam, qwm = dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w))
    outm = dfp4.gemm_prepared(dfp4.gemm_prepare(qam, weight=False, mx=True), dfp4.gemm_prepare(qwm, weight=True, mx=True))
    torch.cuda.synchronize()
    refm, absm = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
    _assert_gemm_close(outm, refm, absm, f"prepared mxfp4 {why}")


@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (5, 40, 64), (33, 100, 4096), (64, 96, 256), (32, 4096, 4096),
                                   (16, 14336, 4096), (16, 4096, 14336)])
def test_gemm_prepared_few_rows(M, N, K):
    # decode shapes on prepared operands: the few-rows kernel with exact int32 sums
    print(f"gemm_prepared parity: few rows {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 200), 50.0, 1.0, seed=700 + M)
    w = synth.gaussian(N, K, 0.02, seed=800 + N)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    for dtype in (torch.float32, torch.bfloat16):
        out = dfp4.gemm_prepared(pa, pw, dtype=dtype)
        torch.cuda.synchronize()
        _assert_gemm_close(out, ref, absdot, f"few rows prepared {dtype}", bf16=dtype == torch.bfloat16)
        if dtype == torch.float32:
            assert (np.abs(out.cpu().double().numpy() - ref) <= np.abs(ref) * 2.0 ** -23 + 1e-300).all()
    assert dfp4.gemm_declined_tiles(pa) == 0
    qam, qwm = dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w))
    outm = dfp4.gemm_prepared(dfp4.gemm_prepare(qam, weight=False, mx=True), dfp4.gemm_prepare(qwm, weight=True, mx=True))
    torch.cuda.synchronize()
    refm, absm = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
    _assert_gemm_close(outm, refm, absm, "few rows prepared mxfp4")


def test_gemm_prepared_few_rows_wide_exponents():
    # classes on both operands, absent class sums, and spreads the exact scheme declines
    # (spreads are those of the drawn powers of two; block maxima of Gaussian data add about one binade)
    for case, (sa, sw) in enumerate([(5, 2), (9, 0), (0, 9), (30, 30)]):
        g = torch.Generator().manual_seed(900 + case)
        M, N, K = 40, 200, 512           # 16 blocks: class sum 2 in every block stays within the int32 bound
        def operand(rows, spread, std):
            x = torch.randn(rows, K, generator=g) * std
            sh = torch.randint(0, spread + 1, (rows, K // 32, 1), generator=g)
            if case == 1 or case == 2:
                sh = torch.where(sh >= 4, torch.full_like(sh, 9), torch.zeros_like(sh))    # classes 0 and 2 only
            return (x.view(rows, K // 32, 32) * torch.exp2(sh.float())).view(rows, K).to(torch.bfloat16)
        a, w = operand(M, sa, 1.0), operand(N, sw, 0.02)
        qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
        pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
        out = dfp4.gemm_prepared(pa, pw)
        torch.cuda.synchronize()
        ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
        _assert_gemm_close(out, ref, absdot, f"few rows prepared, spreads {sa}/{sw}")
        assert (dfp4.gemm_declined_tiles(pa) > 0) == (case == 3)


def test_gemm_prepared_declined_tiles_are_counted():
    # second 512-row tile: block exponents spread over tens of binades -> per-block fp32 path,
    # computed by the workgroup that finds it; the first tile takes the exact path
    g = torch.Generator().manual_seed(19)
    M, N, K = 700, 300, 512
    a = torch.randn(M, K, generator=g)
    scale = torch.exp2(torch.randint(-25, 25, (20, K // 32), generator=g).repeat_interleave(32, dim=1).float())
    a[520:540] *= scale
    a = a.to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g) * 0.02).to(torch.bfloat16)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    out = dfp4.gemm_prepared(pa, pw)
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    _assert_gemm_close(out, ref, absdot, "prepared, mixed exact and declined tiles")
    assert dfp4.gemm_declined_tiles(pa) == 3              # the three column tiles of the second row tile


@pytest.mark.parametrize("spread_a,spread_w,K,expect_declined", [
    (0, 7, 1024, False), (7, 0, 1024, False), (3, 7, 1024, False),
    (4, 4, 512, False),      # class 1 on both sides: visits of class sum 2, 16 blocks stay within the int32 bound
    (4, 4, 1024, True),      # the same over 32 blocks could overflow int32 in the worst case
    (7, 7, 1024, True), (0, 13, 1024, True)])
def test_gemm_prepared_classes_on_both_operands(spread_a, spread_w, K, expect_declined):
    # block exponents spread over `spread` binades along K on either operand: the exact path takes
    # every pair (class of A, class of W) whose sum stays within the classes kept; beyond that the
    # tile is computed block by block in fp32.  Either way the result meets the oracle.
    M, N = 520, 260
    g = torch.Generator().manual_seed(100 + 16 * spread_a + spread_w)
    def operand(rows, spread, std):
        x = torch.randn(rows, K, generator=g) * std
        # every block max lands in the same binade, then a per-block power of two spreads them
        x = x.view(rows, K // 32, 32)
        x[:, :, 0] = 3.0 * std * torch.sign(x[:, :, 0] + 1e-9)
        x = torch.clamp(x, -3.0 * std, 3.0 * std)
        sh = torch.randint(0, spread + 1, (rows, K // 32, 1), generator=g)
        sh[:, 0] = 0
        sh[:, 1] = spread
        return (x * torch.exp2(sh.float())).view(rows, K).to(torch.bfloat16)
    a, w = operand(M, spread_a, 1.0), operand(N, spread_w, 0.02)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    ea, ew = qa.exponent.int(), qw.exponent.int()
    assert int((ea.max(dim=1).values - ea.min(dim=1).values).max()) == spread_a
    assert int((ew.max(dim=1).values - ew.min(dim=1).values).max()) == spread_w
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    out = dfp4.gemm_prepared(pa, pw)
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    _assert_gemm_close(out, ref, absdot, f"spread A {spread_a} W {spread_w}")
    assert (dfp4.gemm_declined_tiles(pa) > 0) == expect_declined
    if not expect_declined:
        # exact path: one rounding of the exact sum
        got = out.cpu().double().numpy()
        assert (np.abs(got - ref) <= np.abs(ref) * 2.0 ** -23 + 1e-300).all()


def test_gemm_prepared_shared_activation_full_size():
    # LLaMA-3-8B gate and up projections on one prepared activation, then the down projection
    # (K split between workgroups), sampled outputs against the oracle
    ops = synth.llama3_8b_mlp(seed=2)
    x, h = ops["x"], ops["h"]
    print("gemm_prepared parity: 2048x14336x4096 (gate, up) and 2048x4096x14336 (down) sampled", flush=True)
    px = dfp4.gemm_prepare(dfp4.quantize(_dev(x)), weight=False)
    rng = np.random.default_rng(7)
    rows = np.sort(rng.choice(x.shape[0], 16, replace=False))
    for name in ("w_gate", "w_up"):
        w = ops[name]
        pw = dfp4.gemm_prepare(dfp4.quantize(_dev(w)), weight=True)
        out = dfp4.gemm_prepared(px, pw)
        torch.cuda.synchronize()
        cols = np.sort(rng.choice(w.shape[0], 128, replace=False))
        ref, absdot = _gemm_ref(synth.to_f64(x[rows]), synth.to_f64(w[cols]))
        _assert_gemm_close(out[rows][:, cols], ref, absdot, f"prepared {name} sampled")
    ph = dfp4.gemm_prepare(dfp4.quantize(_dev(h)), weight=False)
    pw = dfp4.gemm_prepare(dfp4.quantize(_dev(ops["w_down"])), weight=True)
    for rep in range(2):
        out = dfp4.gemm_prepared(ph, pw)
        torch.cuda.synchronize()
        cols = np.sort(rng.choice(4096, 64, replace=False))
        ref, absdot = _gemm_ref(synth.to_f64(h[rows]), synth.to_f64(ops["w_down"][cols]))
        _assert_gemm_close(out[rows][:, cols], ref, absdot, f"prepared down sampled rep {rep}")
    assert dfp4.gemm_declined_tiles(px) == 0 and dfp4.gemm_declined_tiles(ph) == 0


# --------------------------------------------------------------------------
# GEMM with requantizing epilogue
# --------------------------------------------------------------------------
def _requant_ref(a_bf16, w_bf16, mx=False):
    a64, w64 = synth.to_f64(a_bf16), synth.to_f64(w_bf16)
    if mx:
        prod = MX.mxfp4_dequantize(*MX.mxfp4_quantize(a64)) @ MX.mxfp4_dequantize(*MX.mxfp4_quantize(w64)).T
        return MX.mxfp4_quantize(O.round_to_bf16(prod))
    return O.dfp4_gemm_requant(O.dfp4_quantize(a64), O.dfp4_quantize(w64))


@pytest.mark.parametrize("M,N,K", [(600, 352, 512), (512, 128, 64), (130, 96, 1024)])
def test_gemm_requant_fused_tiles_bit_exact(M, N, K):
    # enough tiles that K is not split and moderate exponent spreads: every tile takes the
    # single-accumulator kernel, whose sums are exact, so the quantized result must equal the
    # oracle's bit for bit
    print(f"gemm_requant parity: {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 128), 50.0, 1.0, seed=300 + M)
    w = synth.gaussian(N, K, 0.02, seed=400 + N)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    q = dfp4.gemm_requant(qa, qw)
    torch.cuda.synchronize()
    _assert_quant_equal(q, _requant_ref(a, w), "requant")
    qm = dfp4.mxfp4_gemm_requant(dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w)))
    torch.cuda.synchronize()
    codes, expo = _requant_ref(a, w, mx=True)
    assert np.array_equal(_np(qm.exponent), expo) and np.array_equal(_np(qm.codes), codes)


def test_gemm_requant_full_size_sampled_rows():
    ops = synth.llama3_8b_mlp(seed=2)
    x, w = ops["x"], ops["w_gate"]
    print("gemm_requant parity: 2048x14336x4096 sampled rows", flush=True)
    q = dfp4.gemm_requant(dfp4.quantize(_dev(x)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    rows = np.sort(np.random.default_rng(6).choice(x.shape[0], 6, replace=False))
    codes, dialect, expo = _requant_ref(x[rows], w)
    assert np.array_equal(_np(q.exponent)[rows], expo)
    assert np.array_equal(_np(q.dialect)[rows], dialect)
    assert np.array_equal(_np(q.codes)[rows], codes)


def test_gemm_requant_split_k_bit_exact():
    # few tiles: K is split between workgroups whose exact int32 partial tiles are added before the
    # single conversion, so the requantized result must equal the oracle's bit for bit
    M, N, K = 100, 256, 4096
    print(f"gemm_requant parity: split K {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, 20, 50.0, 1.0, seed=77)
    w = synth.gaussian(N, K, 0.02, seed=78)
    q = dfp4.gemm_requant(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)))
    torch.cuda.synchronize()
    _assert_quant_equal(q, _requant_ref(a, w), "requant split K")


# Both tile heights (3000 x 3296: 156 tiles of 256 x 256), whose waves stage their rows in two halves or at once, edges in both directions.
@pytest.mark.parametrize("M,N,K", [(3000, 3296, 256), (1000, 1120, 192)])
@pytest.mark.parametrize("mx", [False, True])
def test_gemm_requant_equals_the_quantized_product(M, N, K, mx):
    print(f"gemm_requant against quantize(gemm): {M}x{N}x{K}, mx {mx}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M)
    quant = dfp4.mxfp4_quantize if mx else dfp4.quantize
    qa, qw = (quant(torch.randn(r, K, generator=g, device="cuda").to(torch.bfloat16)) for r in (M, N))
    # sums of such blocks are exact, so that both round the same number
    want = quant((dfp4.mxfp4_gemm if mx else dfp4.gemm)(qa, qw, dtype=torch.bfloat16))
    q = (dfp4.mxfp4_gemm_requant if mx else dfp4.gemm_requant)(qa, qw)
    torch.cuda.synchronize()
    assert torch.equal(q.codes, want.codes) and torch.equal(q.exponent, want.exponent)
    assert mx or torch.equal(q.dialect, want.dialect)


@pytest.mark.parametrize("B,M,N,K", [(3, 600, 352, 128), (5, 40, 64, 256), (2, 2048, 2048, 128)])
def test_gemm_requant_batched(B, M, N, K):
    # attention-like batches: every problem's quantized scores against the oracle, bit for bit where the
    # sums are exact (more than 64 rows), to the fp32-accumulation bar otherwise
    print(f"gemm_requant_batched parity: {B} x {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(B * M, K, 2, 30.0, 1.0, seed=310 + M)
    w = synth.gaussian_outlier_channels(B * N, K, 2, 30.0, 1.0, seed=311 + N)
    q = dfp4.gemm_requant_batched(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)), B, M, N)
    torch.cuda.synchronize()
    for b in (range(B) if M <= 600 else (0, B - 1)):
        rows = slice(b * M, (b + 1) * M) if M <= 600 else slice(b * M + 1000, b * M + 1032)
        ab = a[rows]
        wb = w[b * N:(b + 1) * N]
        if M > 64:
            codes, dialect, expo = _requant_ref(ab, wb)
            assert np.array_equal(_np(q.exponent)[rows], expo), f"problem {b}"
            assert np.array_equal(_np(q.dialect)[rows], dialect), f"problem {b}"
            assert np.array_equal(_np(q.codes)[rows], codes), f"problem {b}"
        else:
            ref, _ = _gemm_ref(synth.to_f64(ab), synth.to_f64(wb))
            codes, dialect, expo = O.dfp4_quantize(O.round_to_bf16(ref))
            same = np.array_equal(_np(q.codes)[rows], codes)
            # few rows accumulate in fp32: nearly all blocks reproduce the oracle's
            agree = (_np(q.exponent)[rows] == expo).mean()
            assert agree > 0.99 and (same or (_np(q.codes)[rows] == codes).mean() > 0.99)


def test_gemm_requant_handworked_block(golden_dir):
    # the hand-worked product of tests/golden (products on and just below a bf16 midpoint)
    import json, os
    g = json.load(open(os.path.join(golden_dir, "handworked_requant.json")))
    a = torch.zeros(1, 96)
    a[0, 0::32] = torch.tensor(g["a_blocks"])
    w = torch.zeros(32, 96)
    for j, row in enumerate(g["w_rows"]):
        w[j, 0::32] = torch.tensor(row)
    q = dfp4.gemm_requant(dfp4.quantize(_dev(a.to(torch.bfloat16))), dfp4.quantize(_dev(w.to(torch.bfloat16))))
    torch.cuda.synchronize()
    nib = _np(q.codes)[0]
    nib = np.stack([nib & 15, nib >> 4], axis=1).reshape(-1)
    assert int(q.exponent[0, 0]) == g["exponent_byte"] and int(q.dialect[0, 0]) == g["dialect"]
    assert list(nib[:8]) == g["codes"] and (nib[8:] == 0).all()


@pytest.mark.parametrize("M,N,K,why", [(16, 256, 512, "few rows"), (96, 160, 256, "declined tiles")])
def test_gemm_requant_fp32_accumulating_paths(M, N, K, why):
    # paths that add one fp32 term per block: the bf16 result may differ from the oracle's by one
    # bf16 ulp where the fp32 sum rounds across a bf16 midpoint.  Bar: every bf16 value within one
    # ulp of the oracle's, and every block whose 32 bf16 values all equal the oracle's carries the
    # oracle's exponent byte, dialect id and codes.
    print(f"gemm_requant parity: {why} {M}x{N}x{K}", flush=True)
    g = torch.Generator().manual_seed(M)
    a = torch.randn(M, K, generator=g)
    if why == "declined tiles":
        a = a * torch.exp2(torch.randint(-30, 30, (M, K // 32), generator=g).repeat_interleave(32, dim=1).float())
    a = a.to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g) * 0.02).to(torch.bfloat16)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    q = dfp4.gemm_requant(qa, qw)
    gb = dfp4.gemm(qa, qw, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    rb = O.round_to_bf16(ref)
    got = gb.cpu().double().numpy()
    ulp = np.exp2(np.floor(np.log2(np.maximum(np.abs(rb), 1e-300))) - 7)
    assert (np.abs(got - rb) <= ulp + GEMM_RTOL * absdot).all()
    same = (got == rb).reshape(M, N // 32, 32).all(axis=2)
    assert same.mean() > 0.5, "too few blocks reproduce the oracle's bf16 values to say anything"
    codes, dialect, expo = O.dfp4_quantize(rb)
    assert np.array_equal(_np(q.exponent)[same], expo[same])
    assert np.array_equal(_np(q.dialect)[same], dialect[same])
    assert np.array_equal(_np(q.codes).reshape(M, N // 32, 16)[same], codes.reshape(M, N // 32, 16)[same])
    # the blocks that differ are quantizations of the bf16 values the GPU did compute
    cg, dg, eg = O.dfp4_quantize(got)
    assert np.array_equal(_np(q.codes), cg) and np.array_equal(_np(q.dialect), dg) and np.array_equal(_np(q.exponent), eg)


# --------------------------------------------------------------------------
# MXFP4 on the block-scaled matrix instruction
# --------------------------------------------------------------------------
@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (70, 200, 160), (300, 130, 1056), (512, 512, 4096)])
def test_mxfp4_gemm_native(M, N, K):
    print(f"mxfp4_gemm_native parity: {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 100), 50.0, 1.0, seed=500 + M)
    w = synth.student_t(N, K, 3.0, seed=600 + N)
    qa, qw = dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w))
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
    out = dfp4.mxfp4_gemm_native(qa, qw)
    torch.cuda.synchronize()
    _assert_gemm_close(out, ref, absdot, "native f32")
    outb = dfp4.mxfp4_gemm_native(qa, qw, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    _assert_gemm_close(outb, ref, absdot, "native bf16", bf16=True)


def test_mxfp4_gemm_native_wide_exponents_and_full_size_sample():
    g = torch.Generator().manual_seed(16)
    scale = torch.exp2(torch.randint(-40, 40, (96, 8), generator=g).repeat_interleave(32, dim=1).float())
    a = (torch.randn(96, 256, generator=g) * scale).to(torch.bfloat16)
    w = (torch.randn(160, 256, generator=g) * scale[:1]).to(torch.bfloat16)
    out = dfp4.mxfp4_gemm_native(dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w)))
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
    _assert_gemm_close(out, ref, absdot, "native wide")
    ops = synth.llama3_8b_mlp(seed=2)
    x, wg = ops["x"], ops["w_gate"]
    out = dfp4.mxfp4_gemm_native(dfp4.mxfp4_quantize(_dev(x)), dfp4.mxfp4_quantize(_dev(wg)))
    torch.cuda.synchronize()
    rng = np.random.default_rng(17)
    rows = np.sort(rng.choice(x.shape[0], 16, replace=False))
    cols = np.sort(rng.choice(wg.shape[0], 128, replace=False))
    ref, absdot = _gemm_ref(synth.to_f64(x[rows]), synth.to_f64(wg[cols]), mx=True)
    _assert_gemm_close(out[rows][:, cols], ref, absdot, "native full size sampled")


@pytest.mark.parametrize("M,N,K", [(1, 1, 32), (70, 200, 160), (300, 130, 1056), (512, 512, 4096)])
def test_dfp4_gemm_native(M, N, K):
    # DialectFP4 operands repacked to FP6 E2M3 (exact) on the block-scaled matrix instruction
    print(f"dfp4_gemm_native parity: {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 100), 50.0, 1.0, seed=700 + M)
    w = synth.student_t(N, K, 3.0, seed=800 + N)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    out = dfp4.gemm_native(qa, qw)
    torch.cuda.synchronize()
    _assert_gemm_close(out, ref, absdot, "native fp6 f32")
    outb = dfp4.gemm_native(qa, qw, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    _assert_gemm_close(outb, ref, absdot, "native fp6 bf16", bf16=True)


def test_dfp4_gemm_native_all_dialects_wide_exponents_and_full_size_sample():
    # every dialect and every index occurs; block exponents spread over tens of binades
    g = torch.Generator().manual_seed(18)
    scale = torch.exp2(torch.randint(-40, 40, (128, 16), generator=g).repeat_interleave(32, dim=1).float())
    a = (torch.randn(128, 512, generator=g) * scale).to(torch.bfloat16)
    w = (torch.randn(160, 512, generator=g) * scale[:1]).to(torch.bfloat16)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize_mse(_dev(w))
    assert len(torch.unique(qa.dialect)) == 16
    out = dfp4.gemm_native(qa, qw)
    torch.cuda.synchronize()
    ad = O.dfp4_dequantize(*O.dfp4_quantize(synth.to_f64(a)))
    wd = O.dfp4_dequantize(*O.dfp4_quantize_mse(synth.to_f64(w)))
    _assert_gemm_close(out, ad @ wd.T, np.abs(ad) @ np.abs(wd).T, "native fp6 wide")
    ops = synth.llama3_8b_mlp(seed=2)
    x, wg = ops["x"], ops["w_gate"]
    out = dfp4.gemm_native(dfp4.quantize(_dev(x)), dfp4.quantize(_dev(wg)))
    torch.cuda.synchronize()
    rng = np.random.default_rng(19)
    rows = np.sort(rng.choice(x.shape[0], 16, replace=False))
    cols = np.sort(rng.choice(wg.shape[0], 128, replace=False))
    ref, absdot = _gemm_ref(synth.to_f64(x[rows]), synth.to_f64(wg[cols]))
    _assert_gemm_close(out[rows][:, cols], ref, absdot, "native fp6 full size sampled")


def test_gemm_native_with_prepacked_weights():
    # weights arranged once in the instruction's register order; results identical to the call
    # that packs both operands
    M, N, K = 300, 520, 1056
    a = synth.gaussian_outlier_channels(M, K, 8, 50.0, 1.0, seed=901)
    w = synth.gaussian(N, K, 0.02, seed=902)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    wp = dfp4.native_pack(qw)
    out = dfp4.gemm_native_packed_w(qa, wp)
    both = dfp4.gemm_native(qa, qw)
    both_packed = dfp4.gemm_native_packed(dfp4.native_pack(qa), wp)
    torch.cuda.synchronize()
    assert torch.equal(out, both) and torch.equal(both_packed, both)
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    _assert_gemm_close(out, ref, absdot, "prepacked fp6")
    qam, qwm = dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w))
    outm = dfp4.gemm_native_packed_w(qam, dfp4.native_pack(qwm, mx=True), dtype=torch.bfloat16)
    torch.cuda.synchronize()
    refm, absm = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
    _assert_gemm_close(outm, refm, absm, "prepacked fp4 bf16", bf16=True)


def test_gemm_random_edge_shapes_all_paths():
    # seeded sweep over awkward shapes (sizes around the tile boundaries, odd block counts) and three
    # input recipes; every GEMM path against the oracle, the requantizing one against its composition
    rng = np.random.default_rng(2024)
    for it in range(14):
        M = int(rng.choice([1, 31, 33, 65, 127, 129, 257, 300, 513, 700]))
        N = int(rng.choice([1, 7, 33, 96, 130, 256, 257, 520]))
        KB = int(rng.choice([1, 3, 8, 15, 17, 33, 65]))
        K, kind = KB * 32, int(rng.integers(0, 3))
        print(f"gemm sweep {it}: {M}x{N}x{K} recipe {kind}", flush=True)
        g = torch.Generator().manual_seed(int(rng.integers(1 << 30)))
        a = torch.randn(M, K, generator=g)
        if kind == 1:
            a[:, rng.integers(0, K, max(1, K // 100))] *= 50
        if kind == 2:
            a = a * torch.exp2(torch.randint(-12, 12, (M, KB), generator=g).repeat_interleave(32, dim=1).float())
        a = a.to(torch.bfloat16)
        w = (torch.randn(N, K, generator=g) * 0.02).to(torch.bfloat16)
        ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
        qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
        _assert_gemm_close(dfp4.gemm(qa, qw), ref, absdot, f"exact path {M}x{N}x{K}")
        _assert_gemm_close(dfp4.gemm_native(qa, qw), ref, absdot, f"native path {M}x{N}x{K}")
        if N % 32 == 0:
            rq = dfp4.gemm_requant(qa, qw)
            want = dfp4.quantize(dfp4.gemm(qa, qw, dtype=torch.bfloat16))
            torch.cuda.synchronize()
            assert torch.equal(rq.codes, want.codes) and torch.equal(rq.dialect, want.dialect)
            assert torch.equal(rq.exponent, want.exponent)
        refm, absm = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
        qam, qwm = dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w))
        _assert_gemm_close(dfp4.mxfp4_gemm(qam, qwm), refm, absm, f"mx exact path {M}x{N}x{K}")
        _assert_gemm_close(dfp4.mxfp4_gemm_native(qam, qwm), refm, absm, f"mx native path {M}x{N}x{K}")


@pytest.mark.parametrize("rows,K", [(1, 32), (70, 160), (300, 1056), (513, 4096), (64, 14336)])
def test_quantize_native_equals_quantize_then_pack(rows, K):
    # the quantizer that writes the matrix instruction's FP6 operand directly: byte-identical to
    # dfp4_quantize + dfp4_native_pack (both buffers start as zeros: the fused kernel leaves the
    # layout's padding rows untouched), also from a strided input
    print(f"quantize_native parity: {rows}x{K}", flush=True)
    x = synth.gaussian_outlier_channels(rows, K, max(1, K // 100), 50.0, 1.0, seed=rows + K).cuda()
    n = int(dfp4.load().dfp4_native_packed_bytes(rows, K))
    want = dfp4.native_pack(dfp4.quantize(x), buf=torch.zeros(n, dtype=torch.uint8, device="cuda"))
    got = dfp4.quantize_native(x)
    torch.cuda.synchronize()
    assert torch.equal(got.buf, want.buf), int((got.buf != want.buf).sum())
    wide = torch.zeros(rows, K + 64, dtype=torch.bfloat16, device="cuda")
    wide[:, 32:32 + K] = x
    got2 = dfp4.quantize_native(wide[:, 32:32 + K])
    torch.cuda.synchronize()
    assert torch.equal(got2.buf, want.buf)
    # and it multiplies to the oracle's product
    w = synth.gaussian(96, K, 0.02, seed=K)
    out = dfp4.gemm_native_packed(got, dfp4.native_pack(dfp4.quantize(_dev(w))))
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(x.cpu()), synth.to_f64(w))
    _assert_gemm_close(out, ref, absdot, "quantize_native product")


# --------------------------------------------------------------------------
# value cache with a high-precision residual chunk (Appendix C)
# --------------------------------------------------------------------------
def test_value_cache_appends_match_quantizing_the_transpose():
    from paper_2501_01144_amd.kvcache import ValueCache
    D, cap = 64, 256
    v = synth.gaussian_outlier_channels(200, D, 2, 30.0, 1.0, seed=41)
    cache = ValueCache(D, cap, "cuda")
    pos = 0
    for step in (1, 5, 26, 1, 64, 31, 40, 32):          # odd sizes: chunks complete at different points
        cache.append(v[pos:pos + step].cuda())
        pos += step
        torch.cuda.synchronize()
        assert cache.n_tokens == pos and cache.n_quantized == pos // 32 * 32
        nq = cache.n_quantized
        if nq:
            codes, dialect, expo = O.dfp4_quantize(synth.to_f64(v[:nq]).T.copy())
            assert np.array_equal(_np(cache.q.codes)[:, :nq // 2], codes)
            assert np.array_equal(_np(cache.q.dialect)[:, :nq // 32], dialect)
            assert np.array_equal(_np(cache.q.exponent)[:, :nq // 32], expo)
        assert not _np(cache.q.codes)[:, nq // 2:].any()                      # later blocks untouched
        assert torch.equal(cache.residual_values().cpu(), v[nq:pos])
    # P V over the whole capacity with zero-padded probabilities = product over the quantized tokens
    nq = cache.n_quantized
    p = torch.zeros(4, cap, dtype=torch.bfloat16)
    p[:, :nq] = synth.softmax_rows(4, nq, seed=42)
    out = dfp4.gemm(dfp4.quantize(_dev(p)), cache.q)
    torch.cuda.synchronize()
    ref, absdot = _gemm_ref(synth.to_f64(p[:, :nq]), synth.to_f64(v[:nq]).T.copy())
    _assert_gemm_close(out, ref, absdot, "P V through the cache")


# --------------------------------------------------------------------------
# blocks of 64
# --------------------------------------------------------------------------
@pytest.mark.parametrize("rows,K", [(1, 64), (7, 192), (33, 4096), (257, 1088)])
def test_quantize_block64(rows, K):
    print(f"quantize_b64 parity: {rows}x{K}", flush=True)
    for x in (synth.student_t(rows, K, 3.0, seed=rows + K),
              synth.gaussian_outlier_channels(rows, K, max(1, K // 100), 50.0, 1.0, seed=rows)):
        q = dfp4.quantize_b64(_dev(x))
        torch.cuda.synchronize()
        _assert_quant_equal(q, O.dfp4_quantize_block64(synth.to_f64(x)), "block 64")
    # strided input, and the result multiplies like any other quantized tensor
    wide = torch.zeros(rows, K + 64, dtype=torch.bfloat16, device="cuda")
    wide[:, 32:32 + K] = x.cuda()
    q2 = dfp4.quantize_b64(wide[:, 32:32 + K])
    torch.cuda.synchronize()
    _assert_quant_equal(q2, O.dfp4_quantize_block64(synth.to_f64(x)), "block 64 strided")
    w = synth.gaussian(40, K, 0.02, seed=K)
    out = dfp4.gemm(q, dfp4.quantize_b64(_dev(w)))
    torch.cuda.synchronize()
    ad = O.dfp4_dequantize(*O.dfp4_quantize_block64(synth.to_f64(x)))
    wd = O.dfp4_dequantize(*O.dfp4_quantize_block64(synth.to_f64(w)))
    _assert_gemm_close(out, ad @ wd.T, np.abs(ad) @ np.abs(wd).T, "block 64 product")


@pytest.mark.parametrize("M,N,K", [(5, 40, 64), (16, 4096, 4096), (33, 100, 1056), (64, 96, 256)])
def test_gemm_native_few_rows(M, N, K):
    # decode shapes on the block-scaled instruction: 32 W rows per workgroup, 16 waves share K
    print(f"native few rows parity: {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 200), 50.0, 1.0, seed=110 + M)
    w = synth.gaussian(N, K, 0.02, seed=210 + N)
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    wp = dfp4.native_pack(dfp4.quantize(_dev(w)))
    out = dfp4.gemm_native_packed(dfp4.quantize_native(_dev(a)), wp)
    torch.cuda.synchronize()
    _assert_gemm_close(out, ref, absdot, "native few rows f32")
    outb = dfp4.gemm_native(dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w)), dtype=torch.bfloat16)
    torch.cuda.synchronize()
    _assert_gemm_close(outb, ref, absdot, "native few rows bf16", bf16=True)
    refm, absm = _gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True)
    outm = dfp4.mxfp4_gemm_native(dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w)))
    torch.cuda.synchronize()
    _assert_gemm_close(outm, refm, absm, "native few rows mxfp4")


@pytest.mark.parametrize("M,N,K", [(1, 33, 3072), (32, 64, 3104), (33, 31, 3104), (32, 40, 4128), (64, 65, 4128), (7, 20, 16416)])
def test_gemm_native_few_rows_steps_of_a_wave(M, N, K):
    # three, four and five steps to a wave and many, waves without any, one and two row tiles, both formats
    print(f"native few rows, steps of a wave: {M}x{N}x{K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + K)
    x = torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16)
    w = (torch.randn(N, K, generator=g, device="cuda") * 0.02).to(torch.bfloat16)
    for mx, quant, back in ((False, dfp4.quantize, dfp4.dequantize), (True, dfp4.mxfp4_quantize, dfp4.mxfp4_dequantize)):
        qa, qw = quant(x), quant(w)
        da, dw = back(qa).double(), back(qw).double()
        out = dfp4.gemm_native_packed(dfp4.native_pack(qa, mx=mx), dfp4.native_pack(qw, mx=mx))
        torch.cuda.synchronize()
        assert bool(((out.double() - da @ dw.T).abs() <= GEMM_RTOL * (da.abs() @ dw.abs().T)).all())


# --------------------------------------------------------------------------
# blocks of 16 and mixed block sizes (Section 4.2, Table 3)
# --------------------------------------------------------------------------
@pytest.mark.parametrize("rows,K", [(1, 32), (7, 96), (33, 4096), (257, 1056), (2048, 4096)])
def test_quantize_and_dequantize_block16(rows, K):
    print(f"quantize parity: blocks of 16, {rows}x{K}", flush=True)
    x = torch.cat([synth.student_t(rows, K, 3.0, seed=60 + rows)[: rows - rows // 2],
                   synth.gaussian_outlier_channels(rows // 2, K, max(1, K // 100), 50.0, 1.0, seed=61 + rows)])
    q = dfp4.quantize_block(_dev(x), 16)
    torch.cuda.synchronize()
    assert q.dialect.shape == (rows, K // 16) and q.exponent.shape == (rows, K // 16)
    ref = O.dfp4_quantize_block16(synth.to_f64(x))
    _assert_quant_equal(q, ref, "block16")
    for dtype in (torch.float32, torch.bfloat16):
        back = dfp4.dequantize_block(q, 16, dtype=dtype)
        torch.cuda.synchronize()
        assert np.array_equal(back.cpu().double().numpy(), O.dfp4_dequantize_block(*ref, 16))
    # block sizes 32 and 64 through the same entry point
    _assert_quant_equal(dfp4.quantize_block(_dev(x), 32), O.dfp4_quantize(synth.to_f64(x)), "block32 via quantize_block")
    if K % 64 == 0:
        _assert_quant_equal(dfp4.quantize_block(_dev(x), 64), O.dfp4_quantize_block64(synth.to_f64(x)), "block64")


def test_quantize_block16_every_bf16_value_and_strided_rows():
    vals = synth.all_bf16_bit_patterns()                     # [2040, 32]: two blocks of 16 per row
    q = dfp4.quantize_block(_dev(vals), 16)
    torch.cuda.synchronize()
    _assert_quant_equal(q, O.dfp4_quantize_block16(synth.to_f64(vals)), "every bf16 value, blocks of 16")
    base = synth.gaussian_outlier_channels(70, 1024, 4, 30.0, 1.0, seed=67)
    qs = dfp4.quantize_block(_dev(base)[:, 128:128 + 512], 16)
    torch.cuda.synchronize()
    _assert_quant_equal(qs, O.dfp4_quantize_block16(synth.to_f64(base[:, 128:128 + 512].contiguous())), "strided, blocks of 16")


@pytest.mark.parametrize("M,N,K,ba,bw", [(70, 200, 160, 16, 16), (129, 257, 1024, 16, 32), (300, 130, 512, 32, 16),
                                         (64, 96, 256, 16, 64), (512, 256, 4096, 16, 16), (100, 100, 256, 64, 32)])
def test_gemm_mixed_block_sizes(M, N, K, ba, bw):
    print(f"gemm parity: blocks {ba} x {bw}, {M}x{N}x{K}", flush=True)
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 100), 50.0, 1.0, seed=70 + M)
    w = synth.gaussian(N, K, 0.02, seed=71 + N)
    qa, qw = dfp4.quantize_block(_dev(a), ba), dfp4.quantize_block(_dev(w), bw)
    def oracle_q(x, b):
        x = synth.to_f64(x)
        return (O.dfp4_quantize_block16(x), 16) if b == 16 else ((O.dfp4_quantize_block64(x) if b == 64 else O.dfp4_quantize(x)), 32)
    (ra, la), (rw, lw) = oracle_q(a, ba), oracle_q(w, bw)
    ad, wd = O.dfp4_dequantize_block(*ra, la), O.dfp4_dequantize_block(*rw, lw)
    ref, absdot = O.dfp4_gemm_blocks(ra, la, rw, lw), np.abs(ad) @ np.abs(wd).T
    for dtype in (torch.float32, torch.bfloat16):
        out = dfp4.gemm_blocks(qa, ba, qw, bw, dtype=dtype)
        torch.cuda.synchronize()
        _assert_gemm_close(out, ref, absdot, f"blocks {ba}x{bw} {dtype}", bf16=dtype == torch.bfloat16)


# --------------------------------------------------------------------------
# GEMM that expands both operands inside the kernel, at sizes that end inside a tile, inside a group of 4 blocks and
# inside a wave's share of K (every tile shape: test_gemm_direct_every_shape)
# --------------------------------------------------------------------------
@pytest.mark.parametrize("M,N,K,spread", [
    (1, 33, 32, 0), (33, 31, 96, 0), (31, 1000, 4128, 0), (64, 65, 16384, 0),      # 32 x 32
    (65, 2100, 1056, 0), (190, 2000, 512, 0), (513, 3001, 2080, 0),                # 32 x 32 and 64 x 64
    (300, 2049, 16416, 0),                                                         # 128 x 128, K in two shares
    (1500, 4000, 1120, 0),                                                         # 256 x 128
    (40, 70, 512, 7), (130, 900, 512, 7), (777, 1300, 1024, 5),                    # classes on both operands
    (40, 70, 1056, 30), (200, 1030, 544, 30), (513, 3001, 2080, 30)])              # tiles summed in fp32, block by block
def test_gemm_direct_shapes(M, N, K, spread):
    print(f"gemm direct: {M}x{N}x{K}, exponents over {spread} binades", flush=True)
    g = torch.Generator().manual_seed(M + N + K)
    def operand(rows, std):
        x = torch.randn(rows, K // 32, 32, generator=g) * std
        if spread:
            x *= torch.exp2(torch.randint(0, spread + 1, (rows, K // 32, 1), generator=g).float())
        return x.view(rows, K).to(torch.bfloat16)
    a, w = operand(M, 1.0), operand(N, 0.02)
    if not spread:
        a[:, :: max(2, K // 8)] *= 50.0                          # outlier channels
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    ref, absdot = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    out = dfp4.gemm(qa, qw)
    torch.cuda.synchronize()
    _assert_gemm_close(out, ref, absdot, "direct f32")
    if not spread:
        # one rounding of the exact sum (the float64 reference itself is exact at these sizes)
        assert (np.abs(out.cpu().double().numpy() - ref) <= np.abs(ref) * 2.0 ** -24 + 1e-300).all()
    out = dfp4.gemm(qa, qw, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    _assert_gemm_close(out, ref, absdot, "direct bf16", bf16=True)
    outm = dfp4.mxfp4_gemm(dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w)))
    torch.cuda.synchronize()
    _assert_gemm_close(outm, *_gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True), "direct mxfp4")


@pytest.mark.parametrize("M,N,K", [(256, 300, 512), (257, 300, 512), (400, 2000, 1056), (1100, 1030, 2048)])
def test_gemm_prepared_direct_shapes(M, N, K):
    # prepared operands, few tiles: the references and masks of the prepared form, expansion in the kernel
    a = synth.gaussian_outlier_channels(M, K, max(1, K // 100), 50.0, 1.0, seed=M)
    w = synth.gaussian(N, K, 0.02, seed=N)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    ref, _ = _gemm_ref(synth.to_f64(a), synth.to_f64(w))
    out = dfp4.gemm_prepared(pa, pw)
    torch.cuda.synchronize()
    assert (np.abs(out.cpu().double().numpy() - ref) <= np.abs(ref) * 2.0 ** -24 + 1e-300).all()
    assert dfp4.gemm_declined_tiles(pa) == 0


@pytest.mark.parametrize("batch,M,N,K,spread", [
    (1, 129, 131, 32, 0), (1, 1000, 520, 96, 0), (2, 300, 1030, 64, 0), (3, 257, 129, 128, 0), (1, 2000, 2049, 128, 0),
    (2, 300, 520, 128, 5), (1, 130, 1030, 96, 9), (2, 257, 260, 128, 30), (1, 200, 300, 160, 0)])
def test_gemm_short_k(batch, M, N, K, spread):
    # K of at most four blocks (one iteration of the direct kernel), and one block more; both operands have classes
    print(f"gemm short K: {batch} x {M}x{N}x{K}, exponents over {spread} binades", flush=True)
    g = torch.Generator().manual_seed(M + N + K)
    def operand(rows, std):
        x = torch.randn(rows, K // 32, 32, generator=g) * std
        if spread:
            x *= torch.exp2(torch.randint(0, spread + 1, (rows, K // 32, 1), generator=g).float())
        else:
            x[:, 0, 3] = torch.where(x[:, 0, 3] < 0, -40.0, 40.0) * std    # 3 to 6 binades above the others: class 1 at most
        return x.view(rows, K).to(torch.bfloat16)
    a, w = operand(batch * M, 1.0), operand(batch * N, 0.02)
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    for dtype in (torch.float32, torch.bfloat16):
        out = dfp4.gemm_batched(qa, qw, batch, M, N, dtype=dtype)
        torch.cuda.synchronize()
        out = out.reshape(batch, M, N)
        for b in range(batch):
            ref, absdot = _gemm_ref(synth.to_f64(a[b * M:(b + 1) * M]), synth.to_f64(w[b * N:(b + 1) * N]))
            _assert_gemm_close(out[b], ref, absdot, f"short K {dtype}", bf16=dtype == torch.bfloat16)
            if not spread and dtype == torch.float32:         # one rounding of the exact sum
                assert (np.abs(out[b].cpu().double().numpy() - ref) <= np.abs(ref) * 2.0 ** -24 + 1e-300).all()
    if batch == 1:
        pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
        _assert_gemm_close(dfp4.gemm_prepared(pa, pw), ref, absdot, "short K prepared")
        outm = dfp4.mxfp4_gemm(dfp4.mxfp4_quantize(_dev(a)), dfp4.mxfp4_quantize(_dev(w)))
        _assert_gemm_close(outm, *_gemm_ref(synth.to_f64(a), synth.to_f64(w), mx=True), "short K mxfp4")


def test_gemm_direct_rows_beyond_one_launch():
    # more rows than 65535 tiles of 32: the product is cut into launches; every output is the exact sum
    M, N, K = 65535 * 32 + 700, 5, 32
    print(f"gemm direct: {M}x{N}x{K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    qa = dfp4.quantize(torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16))
    qw = dfp4.quantize(torch.randn(N, K, generator=g, device="cuda").to(torch.bfloat16))
    a, w = dfp4.dequantize(qa, torch.float32).double(), dfp4.dequantize(qw, torch.float32).double()
    want = torch.zeros(M, N, dtype=torch.float64, device="cuda")     # sums of at most 32 products: exact in float64
    for k in range(K):
        want += a[:, k:k + 1] * w[:, k]
    assert torch.equal(dfp4.gemm(qa, qw), want.float())
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    assert torch.equal(dfp4.gemm_prepared(pa, pw), want.float())


def test_gemm_prepared_few_rows_counts_declined_tiles_for_any_n():
    # more columns than 65535 tiles of 32, in one launch; blocks 20 binades apart in a row of A decline every tile
    M, N, K = 4, 65535 * 32 + 700, 64
    print(f"gemm prepared: {M}x{N}x{K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(5)
    a, w = torch.randn(M, K, generator=g, device="cuda"), torch.randn(N, K, generator=g, device="cuda")
    a[1, :32] *= 2.0 ** 20
    qa, qw = dfp4.quantize(a.to(torch.bfloat16)), dfp4.quantize(w.to(torch.bfloat16))
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    out = dfp4.gemm_prepared(pa, pw)
    a, w = dfp4.dequantize(qa, torch.float32).double(), dfp4.dequantize(qw, torch.float32).double()
    ref, absdot = torch.zeros_like(out, dtype=torch.float64), torch.zeros_like(out, dtype=torch.float64)
    for k in range(K):
        term = a[:, k:k + 1] * w[:, k]
        ref += term
        absdot += term.abs()
    assert bool(((out.double() - ref).abs() <= GEMM_RTOL * absdot).all())
    assert dfp4.gemm_declined_tiles(pa) in [(N + n - 1) // n for n in (32, 64, 128)]      # every tile of one row of tiles


def test_gemm_direct_k_beyond_2_to_24():
    # fewer than 512 rows are addressed with 32-bit offsets; whole numbers whose sums fp32 holds: every output is exact
    M, N, K = 3, 2, 2 ** 24 + 64
    print(f"gemm direct: {M}x{N}x{K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(4)
    def operand(rows):
        x = torch.zeros(rows, K, device="cuda")
        x[:, ::32 * 997] = torch.randint(-6, 7, x[:, ::32 * 997].shape, generator=g, device="cuda").float()
        x[:, -1] = 3.0
        return dfp4.quantize(x.to(torch.bfloat16))
    qa, qw = operand(M), operand(N)
    a, w = dfp4.dequantize(qa, torch.float32).double(), dfp4.dequantize(qw, torch.float32).double()
    assert torch.equal(dfp4.gemm(qa, qw), torch.stack([(a * w[n]).sum(1) for n in range(N)], 1).float())


@pytest.mark.parametrize("rows,K", [(1, 32), (33, 96), (256, 64), (257, 320)])
def test_quantize_native_writes_the_whole_buffer(rows, K):
    # padding rows, the missing block of an odd K / 32 and the slack behind either array leave as zeros
    x = synth.student_t(rows, K, 3.0, seed=rows + K).cuda()
    n = int(dfp4.load().dfp4_native_packed_bytes(rows, K))
    want = dfp4.native_pack(dfp4.quantize(x), buf=torch.zeros(n, dtype=torch.uint8, device="cuda"))
    dirty = torch.full((n + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    dfp4.quantize_native(x, buf=dirty)
    torch.cuda.synchronize()
    assert torch.equal(dirty[:n], want.buf) and bool((dirty[n:] == 0xA5).all())


@pytest.mark.parametrize("rows,cols,skip", [(32, 8, 0), (96, 72, 4), (128, 64, 0), (160, 136, 12)])
def test_quantize_t_tile_edges_and_code_alignment(rows, cols, skip):
    # part tiles of 128 x 64, and codes that are only 4-byte aligned (16-byte stores are not taken)
    x = synth.student_t(rows, cols, 3.0, seed=rows + cols)
    n = cols * rows // 2
    buf = torch.full((skip + n + 16,), 0xA5, dtype=torch.uint8, device="cuda")
    meta = [torch.empty((cols, rows // 32), dtype=torch.uint8, device="cuda") for _ in range(2)]
    q = dfp4.quantize_t(_dev(x), out=dfp4.QTensor(buf[skip:skip + n].view(cols, rows // 2), *meta, cols, rows))
    torch.cuda.synchronize()
    _assert_quant_equal(q, O.dfp4_quantize(synth.to_f64(x).T.copy()), f"quantize_t {rows}x{cols} + {skip}")
    assert bool((buf[:skip] == 0xA5).all()) and bool((buf[skip + n:] == 0xA5).all())


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("rows,K", [(1, 32), (1, 2016), (2, 1024), (5, 416), (257, 64), (1, 224), (3, 96), (1023, 32768), (1031, 32736)])
def test_dequantize_around_64_blocks(rows, K, dtype):
    # 1, 63, 64, 65 and 514 blocks, 7 and 9, and either side of 2^20: a wave takes 8 (fp32), 16 or 64; contiguous and strided
    x = synth.student_t(rows, K, 3.0, seed=rows + K)
    q = dfp4.quantize(_dev(x))
    ref = O.dfp4_dequantize(*O.dfp4_quantize(synth.to_f64(x)))
    wide = torch.full((rows, K + 32), 7.0, dtype=dtype, device="cuda")
    y = dfp4.dequantize(q, dtype)
    dfp4.dequantize(q, out=wide[:, 16:16 + K])
    torch.cuda.synchronize()
    assert np.array_equal(y.cpu().double().numpy(), ref)
    assert np.array_equal(wide[:, 16:16 + K].cpu().double().numpy(), ref)
    assert bool((wide[:, :16] == 7).all()) and bool((wide[:, 16 + K:] == 7).all())


# --------------------------------------------------------------------------
# int32 sums are decided by the classes that meet in a block, not by the largest class of each operand
# --------------------------------------------------------------------------
def _lifted(rows, K, std, blocks, by, g, every=1):
    """Positive values whose blocks share one exponent, except `blocks` of every `every`-th row, lifted by 2^by (sums of
    products of lifted blocks pass 2^24 units: added one block at a time in fp32 they would be rounded)."""
    x = 0.5 + 7.0 * torch.rand(rows, K // 32, 32, generator=g)
    x[:, :, 3] = 7.0
    x[::every, blocks] *= 2.0 ** by
    return (x.view(rows, K) * std).to(torch.bfloat16)


@pytest.mark.parametrize("M,N,K,n_a,n_w,meet,by_a,by_w", [
    (16, 300, 4096, 20, 40, 10, 7, 7), (40, 70, 4192, 20, 40, 9, 6, 7),           # decode; K / 32 not a multiple of 4
    (16, 300, 11008, 10, 6, 4, 7, 7), (200, 300, 14336, 8, 6, 3, 7, 7),
    (128, 2049, 14336, 8, 6, 3, 7, 7), (700, 1030, 4096, 20, 30, 7, 7, 7),
    (300, 2049, 16480, 9, 9, 6, 7, 7),                                            # K beyond the prepared form
    (1500, 4000, 1120, 20, 22, 7, 7, 7), (652, 3397, 1184, 20, 22, 7, 7, 7),
    (16, 300, 1024, 2, 4, 0, 11, 7), (200, 300, 1056, 2, 6, 0, 9, 6), (300, 520, 128, 1, 1, 0, 10, 9),
    (300, 520, 96, 1, 1, 0, 10, 9), (40, 70, 64, 1, 1, 0, 9, 11)])                # classes 2 and 1 (and 2) that never meet
def test_gemm_exact_where_few_high_blocks_meet(M, N, K, n_a, n_w, meet, by_a, by_w):
    # A and W hold a few blocks far above the others, `meet` of them the same.  The exact sum fits int32 by the blocks that
    # meet (asserted), although not by the largest class of either operand
    print(f"gemm, few high blocks: {M}x{N}x{K}", flush=True)
    KB, ca, cw = K // 32, by_a // 4, by_w // 4
    g = torch.Generator().manual_seed(M + N + K)
    order = torch.randperm(KB, generator=g)
    in_a, in_w = order[:n_a], order[n_a - meet:n_a - meet + n_w]
    a, w = _lifted(M, K, 1.0, in_a, by_a, g, every=2), _lifted(N, K, 0.0625, in_w, by_w, g)
    both = 16 ** cw + 16 ** (ca + cw)                    # half the rows of A stay low
    weight = KB - n_a - n_w + meet + (n_a - meet) * (1 + 16 ** ca) + (n_w - meet) * 16 ** cw + meet * both
    assert weight <= (2 ** 31 - 1) // (32 * 120 * 120) and (ca + cw <= 2 or not meet)
    assert ca + cw > 2 or min((KB - n_a + n_a * 16 ** ca) * 16 ** cw, (KB - n_w + n_w * 16 ** cw) * 16 ** ca) > 4660
    qa, qw = dfp4.quantize(_dev(a)), dfp4.quantize(_dev(w))
    ref, _ = _gemm_ref(synth.to_f64(a), synth.to_f64(w))

    def assert_exact(out, what):                         # one rounding of the exact sum (float64 holds it)
        torch.cuda.synchronize()
        bad = np.abs(out.cpu().double().numpy() - ref) > np.abs(ref) * 2.0 ** -24
        assert not bad.any(), f"{what}: {bad.sum()} of {bad.size} outputs are not one rounding of the exact sum"
    assert_exact(dfp4.gemm(qa, qw), "plain")
    assert_exact(dfp4.gemm_batched(qa, qw, 1, M, N)[0], "batched")
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    assert_exact(dfp4.gemm_prepared(pa, pw), "prepared")
    if pa.buf is not None:
        assert dfp4.gemm_declined_tiles(pa) == 0


def test_dequantize_fp32_stores_whole_lines():
    # the same tensor to fp32 moves 1.8 times the bytes of bf16; stores of half lines that bypass the caches took 4.5 times
    # as long, whole lines take 2.0 times
    q = dfp4.quantize(synth.student_t(8192, 4096, 3.0, seed=0).cuda())

    def us(dtype):
        y, best = torch.empty(8192, 4096, dtype=dtype, device="cuda"), float("inf")
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            for _ in range(20):
                dfp4.dequantize(q, out=y)
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end) / 20 * 1e3)
        return best
    t32, t16 = us(torch.float32), us(torch.bfloat16)
    print(f"dequantize 8192x4096: fp32 {t32:.1f} us, bf16 {t16:.1f} us", flush=True)
    assert t32 < 3 * t16


def test_calls_go_to_the_current_stream():
    # the handle that a call gets is that of torch's current stream, also of a side stream and of a capturing one
    assert (dfp4._stream().value or 0) == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    a, w = synth.gaussian(33, 512, 1.0, seed=1).cuda(), synth.gaussian(65, 512, 0.02, seed=2).cuda()
    want = dfp4.gemm(dfp4.quantize(a), dfp4.quantize(w))
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        assert dfp4._stream().value == side.cuda_stream
        out = dfp4.gemm(dfp4.quantize(a), dfp4.quantize(w))
    side.synchronize()
    assert torch.equal(out, want)
    graph, qa, qw = torch.cuda.CUDAGraph(), dfp4.quantize(a), dfp4.quantize(w)
    out.zero_()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        dfp4.gemm(dfp4.quantize(a, out=qa), qw, out=out)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want)


def test_dequantize_small_tensors_take_waves():
    # 1024 blocks are latency: with a wave for 64 of them they took 1.6 times (fp32) and 1.3 times as long as 32 blocks
    # on top of a launch; with a wave for each 8 or 16 nearly as long
    def us(rows, dtype):
        q = dfp4.quantize(synth.gaussian(rows, 1024, 1.0, seed=rows).cuda())
        y, stream, graph = torch.empty(rows, 1024, dtype=dtype, device="cuda"), torch.cuda.Stream(), torch.cuda.CUDAGraph()
        with torch.cuda.stream(stream):
            dfp4.dequantize(q, out=y)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(50):
                dfp4.dequantize(q, out=y)
        best = float("inf")
        for _ in range(5):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            graph.replay()
            end.record()
            torch.cuda.synchronize()
            best = min(best, start.elapsed_time(end) / 50 * 1e3)
        return best
    one, many = us(1, torch.float32), us(32, torch.float32)
    print(f"dequantize to fp32: 32 blocks {one:.2f} us, 1024 blocks {many:.2f} us", flush=True)
    assert many < 1.25 * one


# --------------------------------------------------------------------------
# Every kernel that the size rule selects, plain and prepared, exact and with declined tiles.  References: the dequantized
# operands multiplied in float64 (the quantizers have tests of their own), which holds these sums exactly.
# --------------------------------------------------------------------------
def _path_operands(M, N, K, wide):
    """Outlier channels on A, a few high blocks on both operands; `wide`: rows of A beyond what int32 sums can take."""
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    def operand(rows, std, high):
        x = (torch.randn(rows, K // 32, 32, generator=g, device="cuda").clamp(-3.9, 3.9)) * std
        x[:, :, 3] = 4.5 * std
        x[:, :, 5] *= 0.1
        if K >= 512:
            x[:, high] *= 2.0 ** 5                                    # class 1
        return x
    a, w = operand(M, 1.0, 3), operand(N, 0.0625, 7)
    if wide:
        for r in (M // 3, M - 1):
            a[r, -1] *= 2.0 ** 24 if K >= 64 else 1.0
    qa, qw = (dfp4.quantize(x.view(x.shape[0], K).to(torch.bfloat16)) for x in (a, w))
    da, dw = dfp4.dequantize(qa, torch.float32).double(), dfp4.dequantize(qw, torch.float32).double()
    return qa, qw, da @ dw.T, da.abs() @ dw.abs().T


def _check_outputs(out, ref, absdot, exact_rows, what):
    torch.cuda.synchronize()
    err = (out.double() - ref).abs()
    if out.dtype == torch.bfloat16:
        want = ref.to(torch.bfloat16).double()
        ulp = torch.exp2(torch.floor(torch.log2(want.abs().clamp_min(1e-300))) - 7)
        assert bool(((out.double() - want).abs() <= ulp + GEMM_RTOL * absdot).all()), what
        return
    assert bool((err <= GEMM_RTOL * absdot).all()), what
    assert bool((err[exact_rows] <= ref[exact_rows].abs() * 2.0 ** -24).all()), what + ": not one rounding of the exact sum"


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("M,N,K,path", [
    (31, 1000, 4128, 1), (36, 7898, 1344, 2), (190, 2000, 512, 3), (777, 3001, 2080, 4), (652, 3397, 544, 5),
    (1500, 4000, 1120, 6), (1000, 2049, 96, 7), (300, 2049, 16416, 4)])
def test_gemm_direct_every_shape(M, N, K, path, wide):
    assert dfp4.gemm_path(M, N, K) == dfp4.gemm_path(M, N, K, prepared=True) == path
    print(f"gemm_f8_kernel, path {path}: {M}x{N}x{K}, declined tiles {wide}", flush=True)
    rows = [32, 64, 64, 128, 128, 256, 128][path - 1]
    tile_rows = torch.arange(M, device="cuda") // rows
    exact = (tile_rows != M // 3 // rows) & (tile_rows != (M - 1) // rows) if wide else torch.ones(M, dtype=torch.bool, device="cuda")
    qa, qw, ref, absdot = _path_operands(M, N, K, wide)
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    # prepared operands of more than 256 rows are taken or declined by 512 x 128 outputs
    exact_p = exact if M <= 256 or K > 16384 or not wide else (torch.arange(M, device="cuda") // 512 != M // 3 // 512) & (torch.arange(M, device="cuda") // 512 != (M - 1) // 512)
    for dtype in (torch.float32, torch.bfloat16):
        _check_outputs(dfp4.gemm(qa, qw, dtype=dtype), ref, absdot, exact, f"plain {dtype}")
        _check_outputs(dfp4.gemm_prepared(pa, pw, dtype=dtype), ref, absdot, exact_p, f"prepared {dtype}")
    if pa.buf is not None:
        assert (dfp4.gemm_declined_tiles(pa) > 0) == wide


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("M,N,K,prepared", [
    (1552, 5664, 160, True), (518, 6686, 2848, True), (1188, 2211, 9472, True), (2338, 396, 16032, True),    # K whole, in 2, 4 and 8 shares
    (2320, 5408, 448, False), (793, 4639, 4896, False), (845, 2333, 11104, False)])                          # K whole, in 2 and 4
def test_gemm_large_kernel_outputs(M, N, K, prepared, wide):
    # ragged results of the large kernel in both types, with classes on W and with declined tiles
    assert dfp4.gemm_path(M, N, K, prepared=prepared) == 0
    print(f"the large kernel: {M}x{N}x{K}, prepared {prepared}, declined tiles {wide}", flush=True)
    tile_rows = torch.arange(M, device="cuda") // 512
    exact = (tile_rows != M // 3 // 512) & (tile_rows != (M - 1) // 512) if wide else torch.ones(M, dtype=torch.bool, device="cuda")
    qa, qw, ref, absdot = _path_operands(M, N, K, wide)
    if prepared:
        pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    for dtype in (torch.float32, torch.bfloat16):
        out = dfp4.gemm_prepared(pa, pw, dtype=dtype) if prepared else dfp4.gemm(qa, qw, dtype=dtype)
        _check_outputs(out, ref, absdot, exact, f"{dtype}")
    if prepared:
        bad = len({M // 3 // 512, (M - 1) // 512}) * -(-N // 128)                  # tiles, counted by both products
        assert dfp4.gemm_declined_tiles(pa) == (2 * bad if wide else 0)


def test_gemm_prepared_and_plain_agree_across_kernels():
    # equal sizes through different kernels: the same bits wherever both sum exactly
    for M, N, K in ((1552, 5664, 160), (1188, 2211, 9472)):
        assert dfp4.gemm_path(M, N, K) > 0 and dfp4.gemm_path(M, N, K, prepared=True) == 0
        qa, qw, _, _ = _path_operands(M, N, K, False)
        pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
        for dtype, bits in ((torch.float32, torch.int32), (torch.bfloat16, torch.int16)):
            assert torch.equal(dfp4.gemm(qa, qw, dtype=dtype).view(bits), dfp4.gemm_prepared(pa, pw, dtype=dtype).view(bits)), (M, N, K)


# --------------------------------------------------------------------------
# Products sum in fp32 where norms of the rows show that no partial sum rounds, in int32 elsewhere: inputs on either side
# of that rule, in the large kernel and in every shape of the one that expands its operands.  Both are exact, so the bound is one rounding of the float64 product (2^-24; 2^-149 where that is subnormal).
# --------------------------------------------------------------------------
@pytest.mark.parametrize("M,N,K,prepared,path", [
    (1552, 5664, 160, True, 0), (518, 6686, 2848, True, 0), (2320, 5408, 448, False, 0), (845, 2333, 11104, False, 0),
    (31, 1000, 4128, False, 1), (36, 7898, 1344, True, 2), (190, 2000, 512, True, 3), (777, 3001, 2080, False, 4),
    (652, 3397, 544, False, 5), (1500, 4000, 1120, False, 6), (1000, 2049, 96, False, 7)])
@pytest.mark.parametrize("kind", ["plain", "outliers", "massive", "zero blocks", "tiny", "huge", "spread rows", "all zero"])
def test_gemm_exact_sums(M, N, K, prepared, path, kind):
    assert dfp4.gemm_path(M, N, K, prepared=prepared) == path
    print(f"gemm, exact sums: {M}x{N}x{K}, prepared {prepared}, {kind}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K + len(kind))
    a, w = torch.randn(M, K, generator=g, device="cuda"), torch.randn(N, K, generator=g, device="cuda") * 0.02
    if kind == "outliers":                                            # channels on both operands
        a[:, torch.randperm(K, generator=g, device="cuda")[:max(1, K // 200)]] *= 50
        w[:, torch.randperm(K, generator=g, device="cuda")[:2]] *= 20
    elif kind == "massive":                                           # single elements: past 2^24 units in some tiles, not in others
        for i, r in enumerate(range(3, M, 97)):
            a[r, (r * 37) % K] = 2.0 ** (4 + i % 6)
    elif kind == "zero blocks":
        a[::3, :64] = 0
        a[M // 2] = 0
        w[:, 96:128] = 0
    elif kind == "tiny":                                              # references below what the fp32 sums take, in some tiles
        a[: M // 2] *= 2.0 ** -70
        w[N // 2:] *= 2.0 ** -40
    elif kind == "huge":
        a[: M // 2] *= 2.0 ** 60
        w[N // 2:] *= 2.0 ** 55
    elif kind == "spread rows":                                       # every row its own power of two
        a *= torch.exp2(torch.randint(-20, 20, (M, 1), generator=g, device="cuda").float())
    elif kind == "all zero":
        a.zero_()
    qa, qw = dfp4.quantize(a.to(torch.bfloat16)), dfp4.quantize(w.to(torch.bfloat16))
    ref = dfp4.dequantize(qa).double() @ dfp4.dequantize(qw).double().T
    if prepared:
        out = dfp4.gemm_prepared(dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True))
    else:
        out = dfp4.gemm(qa, qw)
    torch.cuda.synchronize()
    assert bool(((out.double() - ref).abs() <= (ref.abs() * 2.0 ** -24).clamp_min(2.0 ** -149)).all())
    if kind == "all zero":
        assert not bool(out.view(torch.int32).any())                  # +0


@pytest.mark.parametrize("top", [190, 191, 193, 198, 199])
def test_gemm_few_rows_high_exponents(top):
    # One block 18 binades or more above the rest of its row: too far for fp32 sums and for int32, whatever its exponent byte
    # (from 191 on its square is no float), so the tiles are counted as declined.
    M, N, K = 40, 200, 512
    print(f"few rows, exponent byte {top}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(top)
    a = torch.randn(M, K // 32, 32, generator=g, device="cuda").clamp(-3.9, 3.9)
    a[:, :, 3] = 4.5                                                  # exponent byte 127
    a[7] *= 2.0 ** 45                                                 # 172
    a[7, 5] *= 2.0 ** (top - 172)
    w = torch.randn(N, K, generator=g, device="cuda") * 0.02
    qa, qw = dfp4.quantize(a.view(M, K).to(torch.bfloat16)), dfp4.quantize(w.to(torch.bfloat16))
    assert qa.exponent[7, 5] == top and qa.exponent[7, 4] == 172
    pa, pw = dfp4.gemm_prepare(qa, weight=False), dfp4.gemm_prepare(qw, weight=True)
    da, dw = dfp4.dequantize(qa).double(), dfp4.dequantize(qw).double()
    out = dfp4.gemm_prepared(pa, pw)
    torch.cuda.synchronize()
    assert bool(((out.double() - da @ dw.T).abs() <= GEMM_RTOL * (da.abs() @ dw.abs().T)).all())
    assert dfp4.gemm_declined_tiles(pa) > 0


@pytest.mark.parametrize("rows,K", [(32768, 4096), (32767, 4096), (4101, 32736)])     # 2^22 blocks, below, and more in a ragged shape
@pytest.mark.parametrize("mx", [False, True])
def test_quantize_large_tensors_like_their_parts(rows, K, mx):
    # tensors larger than the last cache are streamed past the caches; their parts, quantized alone, are not
    print(f"quantize streamed: {rows}x{K}, mx {mx}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(rows)
    x = torch.randn(rows, K, generator=g, device="cuda", dtype=torch.bfloat16)
    quant = dfp4.mxfp4_quantize if mx else dfp4.quantize
    q = quant(x)
    for lo in list(range(0, rows, rows // 7)) + [rows - 5]:
        hi = min(rows, lo + 512)
        part = quant(x[lo:hi])
        assert torch.equal(q.codes[lo:hi], part.codes) and torch.equal(q.exponent[lo:hi], part.exponent)
        assert mx or torch.equal(q.dialect[lo:hi], part.dialect)


# --------------------------------------------------------------------------
# The rule for fp32 sums at its limit: absolute products of an output that add up to 2^24 units all but a few thousandths, most of it
# one product (of two blocks 8 binades above the rest) beside products of one unit in the same pair of blocks, in other steps and in
# other shares of K.  Every output is a whole number of units, so there is one right answer, bit for bit.  `over`: sums beyond 2^24 units
# that int32 holds, rounded once.
# --------------------------------------------------------------------------
def _limit_operand(rows, K, mx, over, weight, g):
    """Quantized operand, and its elements as whole numbers of units.  Rows whose numbers agree modulo 5 have their high blocks in the
    same places."""
    KB, dev = K // 32, "cuda"
    book = torch.tensor(dfp4.formatbook(), device=dev)
    r = torch.arange(rows, device=dev)
    sign = torch.randint(0, 2, (rows, KB, 32), generator=g, device=dev)
    idx = torch.ones(rows, KB, 32, dtype=torch.long, device=dev)                  # u = 1
    dial = torch.full((rows, KB), 7, device=dev) if mx else torch.randint(0, 16, (rows, KB), generator=g, device=dev)
    delta = torch.zeros(rows, KB, dtype=torch.long, device=dev)
    if not weight:
        idx[torch.randint(0, 16, (rows, KB, 32), generator=g, device=dev) == 0] = 0          # odd and even sums
    if over:
        n = min(KB - 1, 16)
        for i in range(n):                                                        # A 8 binades up, W not: products of 15 * 15 * 2^8
            kb = i * KB // n
            idx[:, kb], sign[:, kb] = 7, 0
            dial[:, kb] = 7 if mx else i % 2                                      # largest magnitude 15, or 12
            delta[:, kb] = 0 if weight else 8
    else:
        p = torch.tensor([0, KB // 2, KB - 1, 1, 2 * KB // 3], device=dev)[r % 5]
        for kb, up, elements, d in ((p, 8, (3,), 1), ((p + 1) % KB, 7, (0, 17, 31), 8)):
            idx[r, kb] = 0
            delta[r, kb] = up
            dial[r, kb] = 7 if mx else d                                          # largest magnitude 15, 11 or 12
            for e in elements if mx else elements[-1:]:
                idx[r, kb, e] = 7
                sign[r, kb, e] = (r % 2 if weight and up == 7 else 0)             # the second product taken away in every other column
    u = book[dial].gather(2, idx)
    whole = u * (1 - 2 * sign) << delta.unsqueeze(-1)
    code = ((sign << 3) | idx).view(rows, K // 2, 2)
    return dfp4.QTensor((code[..., 0] | (code[..., 1] << 4)).to(torch.uint8), None if mx else dial.to(torch.uint8),
                        (delta + (118 if weight else 121)).to(torch.uint8), rows, K), whole.view(rows, K).double()


@pytest.mark.parametrize("M,N,K,prepared,path", [
    (1552, 5664, 160, True, 0), (518, 6686, 2848, True, 0), (2338, 396, 16032, True, 0), (845, 2333, 11104, False, 0),     # K whole, in 2, 8 and 4 shares
    (31, 1000, 4128, False, 1), (36, 7898, 1344, True, 2), (190, 2000, 512, True, 3), (777, 3001, 2080, False, 4),
    (300, 2049, 16416, False, 4), (652, 3397, 544, False, 5), (1500, 4000, 1120, True, 6), (1500, 4000, 1120, False, 6), (1000, 2049, 96, False, 7)])
@pytest.mark.parametrize("mx", [False, True])
@pytest.mark.parametrize("over", [False, True])
def test_gemm_exact_sums_at_the_limit(M, N, K, prepared, path, mx, over):
    assert dfp4.gemm_path(M, N, K, prepared=prepared) == path
    print(f"gemm, sums at the limit: {M}x{N}x{K}, prepared {prepared}, mx {mx}, over {over}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K + M)
    (qa, a), (qw, w) = _limit_operand(M, K, mx, over, False, g), _limit_operand(N, K, mx, over, True, g)
    units, most = a @ w.T, float((a.abs() @ w.abs().T).max())
    if over:
        assert K < 512 or most > 2.0 ** 24
    else:
        assert 0.98 * 2 ** 24 < most and float(a.square().sum(1).max()) < 0.9998 * 2 ** 24
        assert K < 512 or float(units.abs().min()) < 2 ** 23 and bool((units[units.abs() > 2 ** 23].long() & 1).any())
    if prepared:
        out = dfp4.gemm_prepared(dfp4.gemm_prepare(qa, weight=False, mx=mx), dfp4.gemm_prepare(qw, weight=True, mx=mx))
    else:
        out = (dfp4.mxfp4_gemm if mx else dfp4.gemm)(qa, qw)
    torch.cuda.synchronize()
    assert torch.equal(out, (units * 2.0 ** (118 + 121 - 256)).float())


@pytest.mark.parametrize("M,N,K", [(1552, 5664, 160), (518, 6686, 2848), (2338, 396, 16032), (2304, 4096, 4096)])
@pytest.mark.parametrize("mx", [False, True])
def test_gemm_exact_sums_with_a_large_product(M, N, K, mx):
    # One product of 2^23 units beside units: below 2^24 in all, and yet the block-scaled instruction drops the last bit of its sum where
    # both factors are the smallest magnitude (a subnormal FP6 or FP4 number) of blocks 23 binades up.
    assert dfp4.gemm_path(M, N, K, prepared=True) == 0
    print(f"gemm, one product of 2^23 units: {M}x{N}x{K}, mx {mx}", flush=True)
    g, KB = torch.Generator(device="cuda").manual_seed(K + M), K // 32
    def operand(rows, up, base):
        idx = (torch.rand(rows, KB, 32, generator=g, device="cuda") < 0.2).long()  # u = 1 or 0
        sign = torch.randint(0, 2, idx.shape, generator=g, device="cuda")
        delta, kb = torch.zeros(rows, KB, dtype=torch.long, device="cuda"), KB - 2
        idx[:, kb], idx[:, kb, 5], delta[:, kb] = 0, 1, up
        dial = torch.randint(0, 16, (rows, KB), generator=g, device="cuda")        # index 1 is u = 1 in all
        whole = idx * (1 - 2 * sign) << delta.unsqueeze(-1)
        code = ((sign << 3) | idx).view(rows, K // 2, 2)
        return dfp4.QTensor((code[..., 0] | (code[..., 1] << 4)).to(torch.uint8), None if mx else dial.to(torch.uint8),
                            (delta + base).to(torch.uint8), rows, K), whole.view(rows, K).double()
    (qa, a), (qw, w) = operand(M, 11, 121), operand(N, 12, 118)
    units = a @ w.T
    assert float((a.abs() @ w.abs().T).max()) < 2 ** 24 and bool((units.long() & 1).any())
    out = dfp4.gemm_prepared(dfp4.gemm_prepare(qa, weight=False, mx=mx), dfp4.gemm_prepare(qw, weight=True, mx=mx))
    torch.cuda.synchronize()
    assert torch.equal(out, (units * 2.0 ** (118 + 121 - 256)).float())


def _rows_of_any_alignment(M, N, first, more, dtype):
    """[M, N] inside a larger buffer, `first` columns into rows of N + more, and what is true of the buffer when nothing beside it was written"""
    buf = torch.full((M + 512, N + more), 12345.0, dtype=dtype, device="cuda")
    out = buf[256:256 + M, first:first + N]

    def untouched():
        out.fill_(12345.0)
        return bool((buf == torch.full((), 12345.0, dtype=dtype, device="cuda")).all())
    return out, untouched


def _native_rows(M, N, ranges):
    """rows of a workgroup's tile in gemm_native_kernel"""
    tiles = -(-M // 256) * -(-N // 256)
    return 128 if tiles * ranges * 2 <= torch.cuda.get_device_properties(0).multi_processor_count or M <= 128 else 256


# Fewer iterations than the loop of gemm_native_kernel keeps on their way, odd numbers of steps, both tile heights, K in two and four ranges,
# tiles of an XCD in rectangles (2048 x 1024, 4000 x 4096), edges, and results at every alignment of their rows: nothing beside them is written.
@pytest.mark.parametrize("M,N,K,rows,ranges", [
    (65, 257, 32, 128, 1), (128, 300, 64, 128, 1), (129, 256, 96, 128, 1), (200, 513, 160, 128, 1), (257, 264, 192, 128, 1), (300, 1024, 224, 128, 1),
    (256, 256, 256, 128, 1), (400, 700, 288, 128, 1), (1030, 520, 416, 128, 1), (2048, 1024, 544, 128, 1), (4096, 2048, 96, 128, 1),
    (100, 1000, 8224, 128, 4), (300, 5000, 12064, 128, 2),
    (1552, 5664, 32, 256, 1), (4000, 4096, 96, 256, 1), (1552, 5664, 160, 256, 1), (2338, 4001, 224, 256, 1), (2304, 3849, 416, 256, 1),
    (4100, 2055, 544, 256, 1)])
@pytest.mark.parametrize("first,more", [(0, 0), (8, 8), (2, 4), (1, 3)])
@pytest.mark.parametrize("mx", [False, True])
def test_gemm_native_loop_and_results(M, N, K, rows, ranges, first, more, mx):
    need = int(dfp4.load().dfp4_gemm_native_splitk_bytes(M, N, K))
    assert need == (-(-ranges * M * N * 4 // 256) * 256 if ranges > 1 else 0) and _native_rows(M, N, ranges) == rows
    print(f"gemm native: {M}x{N}x{K}, {first} columns into rows of {N + more}, mx {mx}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K + M)
    x, w = (torch.randn(r, K, generator=g, device="cuda").to(torch.bfloat16) for r in (M, N))
    quant, back = (dfp4.mxfp4_quantize, dfp4.mxfp4_dequantize) if mx else (dfp4.quantize, dfp4.dequantize)
    qa, qw = quant(x), quant(w)
    a, b = dfp4.native_pack(qa, mx=mx), dfp4.native_pack(qw, mx=mx)
    da, dw = back(qa).double(), back(qw).double()
    ref, absdot = da @ dw.T, da.abs() @ dw.abs().T
    for dtype in (torch.float32, torch.bfloat16):
        out, untouched = _rows_of_any_alignment(M, N, first, more, dtype)
        dfp4.gemm_native_packed(a, b, out=out)
        torch.cuda.synchronize()
        err = (out.double() - ref).abs()
        assert bool((err <= GEMM_RTOL * absdot + (ref.abs() * 2.0 ** -8 if dtype == torch.bfloat16 else 0)).all())
        assert untouched()


# The same epilogue after exact sums: both tile heights, whole and with K split, there with the tiles of an XCD in rectangles.
@pytest.mark.parametrize("M,N,K,rows,split", [(1552, 5664, 160, 256, False), (2338, 4001, 544, 256, False), (3968, 4096, 96, 256, False),
                                              (1000, 2000, 14336, 128, True), (2000, 2041, 8192, 128, True), (2048, 4096, 8224, 128, False)])
@pytest.mark.parametrize("first,more", [(0, 0), (2, 4), (1, 3)])
@pytest.mark.parametrize("mx", [False, True])
def test_gemm_exact_results_of_any_alignment(M, N, K, rows, split, first, more, mx):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    across, down = -(-N // 256), -(-M // rows)
    assert dfp4.gemm_path(M, N, K, prepared=True) == 0 and _native_rows(M, N, 1) == rows
    assert (int(dfp4.load().dfp4_gemm_prepared_workspace_bytes(M, N, K)) > 0) == split
    if split:                                                # a power of two of columns, eight rectangles, all workgroups at once
        assert across & (across - 1) == 0 and down % 8 == 0 and across * down * 2 <= cus
    print(f"gemm, exact: {M}x{N}x{K}, {first} columns into rows of {N + more}, mx {mx}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(K + M)
    quant, back = (dfp4.mxfp4_quantize, dfp4.mxfp4_dequantize) if mx else (dfp4.quantize, dfp4.dequantize)
    qa, qw = (quant(torch.randn(r, K, generator=g, device="cuda").to(torch.bfloat16)) for r in (M, N))
    a, b = dfp4.gemm_prepare(qa, weight=False, mx=mx), dfp4.gemm_prepare(qw, weight=True, mx=mx)
    ref = back(qa).double() @ back(qw).double().T            # exact: whole numbers of units below 2^24, as fp32 holds them
    assert dfp4.gemm_declined_tiles(a) == 0
    for dtype in (torch.float32, torch.bfloat16):
        out, untouched = _rows_of_any_alignment(M, N, first, more, dtype)
        dfp4.gemm_prepared(a, b, out=out)
        torch.cuda.synchronize()
        assert torch.equal(out, ref.float().to(dtype)) and torch.equal(ref.float().double(), ref)
        assert untouched()
    assert dfp4.gemm_declined_tiles(a) == 0


# K is split where that pays: 128 x 4096 x 4096 took as long in four ranges as whole.
@pytest.mark.parametrize("M,N,K", [(128, 4096, 4096), (256, 1024, 4096), (512, 4096, 14336)])
def test_gemm_native_split_k_pays(M, N, K):
    lib = dfp4.load()
    a, b = (dfp4.native_pack(dfp4.quantize(torch.randn(r, K, device="cuda").to(torch.bfloat16))) for r in (M, N))
    need = int(lib.dfp4_gemm_native_splitk_bytes(M, N, K))
    assert need > 0
    room = torch.empty(need, dtype=torch.uint8, device="cuda")
    out = torch.empty(M, N, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    times = {"split": [], "whole": []}
    for rep in range(12):
        for k, (ptr, size) in {"split": (room.data_ptr(), need), "whole": (None, 0)}.items():
            first, last = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            first.record()
            for _ in range(20):
                assert lib.dfp4_gemm_native_packed(a.buf.data_ptr(), M, b.buf.data_ptr(), N, K, out.data_ptr(), 0, N, ptr, size, stream) == 0
            last.record()
            last.synchronize()
            times[k].append(first.elapsed_time(last) * 50)
    us = {k: float(np.median(v[2:])) for k, v in times.items()}
    print(f"gemm native {M}x{N}x{K} fp32, us: {us}", flush=True)
    assert us["split"] < 0.88 * us["whole"], us


# Results into rows of any alignment go out 16 bytes a lane: they took 1.3 times as long as aligned ones where a lane stored one or two elements.
def test_gemm_native_results_of_any_alignment_take_as_long():
    M, N, K = 4992, 4864, 32
    a, b = (dfp4.native_pack(dfp4.quantize(torch.randn(r, K, device="cuda").to(torch.bfloat16))) for r in (M, N))
    rows = torch.empty(M, N + 16, dtype=torch.bfloat16, device="cuda")
    outs = {"16 bytes": rows[:, :N], "2 bytes": torch.empty(M, N + 3, dtype=torch.bfloat16, device="cuda")[:, 1:N + 1],
            "4 bytes": torch.empty(M, N + 2, dtype=torch.bfloat16, device="cuda")[:, :N]}
    times = {k: [] for k in outs}
    for rep in range(12):
        for k, out in outs.items():
            first, last = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            first.record()
            for _ in range(20):
                dfp4.gemm_native_packed(a, b, out=out)
            last.record()
            last.synchronize()
            times[k].append(first.elapsed_time(last) * 50)
    us = {k: float(np.median(v[2:])) for k, v in times.items()}
    print(f"gemm native {M}x{N}x{K} bf16, us by alignment of the rows: {us}", flush=True)
    assert max(us.values()) < 1.2 * us["16 bytes"], us


# --------------------------------------------------------------------------
# Calls that allocate their result raise what torch.empty raises.
# --------------------------------------------------------------------------
def test_calls_that_allocate_raise_out_of_memory():
    rows = 1 << 20
    print("results of 4 TiB", flush=True)
    q = dfp4.quantize(torch.ones(rows, 32, dtype=torch.bfloat16, device="cuda"))
    assert 4 * rows * rows > torch.cuda.get_device_properties(0).total_memory
    a, w, packed = dfp4.gemm_prepare(q, weight=False), dfp4.gemm_prepare(q, weight=True), dfp4.native_pack(q)
    for call in (lambda: dfp4.gemm(q, q), lambda: dfp4.gemm_prepared(a, w), lambda: dfp4.gemm_native_packed(packed, packed),
                 lambda: dfp4.gemm_batched(q, q, 1, rows, rows), lambda: dfp4.gemm_native_packed_w(q, packed)):
        with pytest.raises(torch.OutOfMemoryError):
            call()


# --------------------------------------------------------------------------
# gemm_f8_kernel, inputs with outliers on which the first, cheap norms give no proof: a second look at the codes does, of W alone
# ("channels"), of A too ("A"), or not at all ("neither").
# --------------------------------------------------------------------------
def _outlier_operands(M, N, K, kind, batch=1):
    g = torch.Generator(device="cuda").manual_seed(M + K + len(kind))
    fa, fw = {"plain": (1, 1), "channels": (50, 40), "A": (400, 1), "neither": (4000, 100)}[kind]
    def operand(rows, std, factor):
        x = torch.randn(rows, K, generator=g, device="cuda") * std
        x[:, torch.randperm(K, generator=g, device="cuda")[:max(1, K // 200)]] *= factor
        return dfp4.quantize(x.to(torch.bfloat16).repeat(batch, 1))
    return operand(M, 1.0, fa), operand(N, 0.02, fw)


@pytest.mark.parametrize("M,N,K,path", [
    (31, 1000, 4128, 1), (36, 7898, 1344, 2), (190, 2000, 512, 3), (777, 3001, 2080, 4), (300, 2049, 16416, 4), (652, 3397, 544, 5), (1500, 4000, 1120, 6),
    (1000, 2049, 96, 7), (1000, 2049, 128, 7)])
@pytest.mark.parametrize("kind", ["channels", "A", "neither"])
def test_gemm_second_look(M, N, K, path, kind):
    assert dfp4.gemm_path(M, N, K) == path
    print(f"gemm, second look: {M}x{N}x{K}, {kind}", flush=True)
    qa, qw = _outlier_operands(M, N, K, kind)
    da, dw = dfp4.dequantize(qa).double(), dfp4.dequantize(qw).double()
    ref, absdot = da @ dw.T, da.abs() @ dw.abs().T
    out = dfp4.gemm(qa, qw)
    torch.cuda.synchronize()
    err = (out.double() - ref).abs()
    assert bool((err <= GEMM_RTOL * absdot).all())
    if kind != "neither" and K < 8192:                                # proven, or within int32 sums
        assert bool((err <= ref.abs() * 2.0 ** -24).all())


@pytest.mark.parametrize("M,N,K,batch", [(32, 4096, 4096, 1), (300, 4096, 4096, 1), (777, 3001, 2080, 1), (1500, 4000, 1120, 1), (1024, 128, 2048, 64)])
def test_gemm_outlier_channels_cost_little(M, N, K, batch):
    # A second look is part of a product's time (1.1 to 1.4 times), the same product a second time in int32 is not (2.3 to 5.3)
    print(f"gemm, time with outlier channels: {M}x{N}x{K}, batch {batch}", flush=True)
    def timed(kind):
        qa, qw = _outlier_operands(M, N, K, kind, batch)
        out = torch.empty(batch, M, N, device="cuda")
        times = []
        for _ in range(7):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            dfp4.gemm_batched(qa, qw, batch, M, N, out=out)
            torch.cuda._sleep(1000000)                                # the calls are enqueued meanwhile
            start.record()
            for _ in range(20):
                dfp4.gemm_batched(qa, qw, batch, M, N, out=out)
            end.record()
            end.synchronize()
            times.append(start.elapsed_time(end) * 1e3 / 20)
        return sorted(times)[3]
    plain, channels = timed("plain"), timed("channels")
    print(f"{plain:.1f} us, with channels {channels:.1f} us", flush=True)
    assert channels < 1.75 * plain
