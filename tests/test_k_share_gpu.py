"""K shared out: over slices of workgroups (with more rows than the few-row kernel takes, so that the slices
run), and over the waves of a small tile (64x64 and 128x128_s3 from 2 KB of K on), whose four stage buffers
wrap, whose partial last K tile is zeroed by hand and whose two groups of waves join their sums in LDS."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2512_23424_amd import binding as B
from paper_2512_23424_amd import inputs as I
from tests import _harness as H

pytestmark = pytest.mark.gpu
NORMS = [I.NORM_NONE, I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_RMSNORM, I.NORM_LOGSUMEXP]
DIST = {"X": ("normal", 0.0, 1.0), "b": ("uniform", -0.5, 0.5), "gamma": ("normal", 1.0, 0.1), "beta": ("normal", 0.0, 0.1)}


def _workload(dt, M, K, N, act, norm, out=None):
    scale = dict(alpha=1.0 / K ** 0.5) if dt == I.F8E4M3 else {}
    w_std = 1.0 if dt == I.F8E4M3 else 1.0 / K ** 0.5
    return I.Workload(name=f"share{act}{norm}", M=M, K=K, N=N, in_dtype=dt, out_dtype=out if out is not None else I.BF16 if dt == I.F8E4M3 else dt,
                      act=act, norm=norm, post_scale=1.5, clamp_lo=-0.5, clamp_hi=0.75, eps=1e-5, dist=dict(DIST, W=("normal", 0.0, w_std)), **scale)


def _params(w, d, out, aux, flags=0):
    return B.make_params(d["X"], d["W"], out, alpha=w.alpha, post_scale=w.post_scale, clamp_lo=w.clamp_lo, clamp_hi=w.clamp_hi, eps=w.eps,
                         gamma=d["gamma"], beta=d["beta"], aux_out=aux, flags=flags)


@pytest.mark.parametrize("dt", [I.BF16, I.F16, I.F8E4M3])
@pytest.mark.parametrize("act,norm", [(I.ACT_GELU_TANH, I.NORM_NONE), (I.ACT_RELU, I.NORM_SOFTMAX), (I.ACT_CLAMP, I.NORM_LOGSUMEXP),
                                      (I.ACT_NONE, I.NORM_LAYERNORM), (I.ACT_SILU, I.NORM_RMSNORM)])
def test_k_slices_of_16_and_8_bit_operands(dt, act, norm):
    for M, flags in ((72, 0), (16, 1 << 8)):           # (the forced 64x64 tile keeps few rows on it)
        w = _workload(dt, M, 4096, 1032, act, norm)
        t = I.generate(w)
        d = {k: H.to_device(v) for k, v in t.items()}
        aux = torch.empty(M, device="cuda") if norm == I.NORM_LOGSUMEXP else None
        p = _params(w, d, torch.empty(M, w.N, dtype=H.tdtype(w.out_dtype), device="cuda"), aux, flags)
        assert not B.fge_few_rows(False, act, norm, p) and B.fge_fused_k_slices(act, norm, p) == 8
        ref, raux = H.oracle_chain(w, t)
        got, gaux = H.run_gpu(w, t, "fused", dev=d, flags=flags)
        H.check(w, got, gaux, ref, raux, f"k slices M={M}")
        again, _ = H.run_gpu(w, t, "fused", dev=d, flags=flags)
        assert np.array_equal(got, again)


@pytest.mark.parametrize("dt", [I.BF16, I.F16, I.F8E4M3])
@pytest.mark.parametrize("norm", NORMS)
def test_gated_products_in_k_slices(dt, norm):
    w = _workload(dt, 72, 4096, 1032, I.ACT_SILU, norm)
    t = I.generate_gated(w)
    d = {k: H.to_device(v) for k, v in t.items()}
    out = torch.full((w.M, w.N), float("nan"), dtype=H.tdtype(w.out_dtype), device="cuda")
    aux = torch.full((w.M,), float("nan"), device="cuda") if norm == I.NORM_LOGSUMEXP else None
    p = _params(w, d, out, aux)
    assert not B.fge_few_rows(True, w.act, norm, p) and B.fge_gated_tile_name(w.act, norm, p) == "partial_products_then_gate"
    n = B.fge_gated_workspace_bytes(True, w.act, norm, p)
    assert n >= 2 * 8 * w.M * w.N * 4                   # eight slices of either product
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    p.workspace, p.workspace_bytes = ws.data_ptr(), n
    B.fused_gated_gemm_epilogue(d["X"], d["W"], d["W2"], d["b"], d["b2"], w.act, norm, p, out)
    torch.cuda.synchronize()
    f = {k: I.as_f64(v) for k, v in t.items()}
    ref, raux = O.gated_chain(f["X"], f["W"], f["W2"], f["b"], f["b2"], f["gamma"], f["beta"], alpha=w.alpha, post_scale=w.post_scale,
                              act=w.act, clamp_lo=w.clamp_lo, clamp_hi=w.clamp_hi, norm=norm, eps=w.eps)
    H.check(w, H.to_host_f64(out), None if aux is None else H.to_host_f64(aux), ref, raux, "gated k slices")


@pytest.mark.parametrize("M", [24, 72])                 # the few-row kernel and its row kernel; the slices' kernels
def test_capture_and_replay(M):
    w = _workload(I.BF16, M, 4096, 1024, I.ACT_SILU, I.NORM_RMSNORM)
    t = I.generate(w)
    d = {k: H.to_device(v) for k, v in t.items()}
    want, _ = H.run_gpu(w, t, "fused", dev=d)
    out = torch.full((M, w.N), float("nan"), dtype=torch.bfloat16, device="cuda")
    p = _params(w, d, out, None)
    assert B.fge_few_rows(False, w.act, w.norm, p) == (M <= 64) and B.fge_fused_k_slices(w.act, w.norm, p) == 8
    ws = torch.empty(B.fge_workspace_bytes(True, w.act, w.norm, p), dtype=torch.uint8, device="cuda")
    p.workspace, p.workspace_bytes = ws.data_ptr(), ws.numel()
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        B.fused_gemm_epilogue(d["X"], d["W"], d["b"], w.act, w.norm, p, out, stream=side)
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(H.to_host_f64(out), want)


@pytest.mark.parametrize("dt,out", [(I.BF16, I.F32), (I.F16, I.F16), (I.F8E4M3, I.F32), (I.F8E4M3, I.BF16)])
@pytest.mark.parametrize("tile,M", [(0, 200), (10, 300)])
def test_exact_sums_over_every_phase_of_the_stage_buffers(dt, out, tile, M):
    """Whole and partial last K tiles for every remainder of the tile count by four, ordinary launch and - 128x128_s3,
    logsumexp, which leaves the values - the one-kernel and the two-pass form."""
    unit, tile_k = (16, 128) if dt == I.F8E4M3 else (8, 64)
    forms = [(I.NORM_NONE, 0)] + ([(I.NORM_LOGSUMEXP, 0), (I.NORM_LOGSUMEXP, B.FLAG_TWO_PASS)] if tile == 10 else [(I.NORM_LOGSUMEXP, 0)])
    for tiles in (16, 17, 18, 19, 20):
        for K in (tiles * tile_k, tiles * tile_k + unit, (tiles + 1) * tile_k - unit):
            w = I.Workload(name="phase", M=M, K=K, N=392, in_dtype=dt, out_dtype=out, alpha=2.0 ** -6,
                           dist={"X": ("int", -1, 1), "W": ("int", -1, 1), "b": ("int", -2, 2)})
            t = I.generate(w)
            d = {k: H.to_device(v) for k, v in t.items()}
            ref, _ = H.oracle_chain(w, t)
            exact = ref.astype(np.float16).astype(np.float64) if out == I.F16 else I.as_f64(I.f64_to_bf16_bits(ref)) if out == I.BF16 else ref
            for norm, flags in forms:
                wn = I.scaled(w, norm=norm)
                got, gaux = H.run_gpu(wn, t, "fused", dev=d, flags=flags | (tile + 1) << 8 | B.FLAG_NO_SPLIT_K)
                assert np.array_equal(got, exact), f"K={K} norm {norm} flags {flags}: {int((got != exact).sum())} mismatches"
                if norm == I.NORM_LOGSUMEXP:
                    m = ref.max(axis=1)
                    lse = m + np.log(np.exp(ref - m[:, None]).sum(axis=1))
                    assert np.abs(gaux - lse).max() <= 1e-5 * np.abs(lse).max()     # fp32 exponentials and sums


@pytest.mark.parametrize("norm", NORMS)
def test_fp32_instruction_with_results_of_any_width(norm):
    """FGE_FLAG_IEEE_FP32 over odd widths: direct stores, parked rows, whole rows of the one tile that exists there."""
    for M, K, N in ((300, 272, 515), (500, 1000, 61), (260, 512, 2051)):
        w = _workload(I.F32, M, K, N, I.ACT_SILU, norm)
        t = I.generate(w)
        d = {k: H.to_device(v) for k, v in t.items()}
        aux = torch.empty(M, device="cuda") if norm == I.NORM_LOGSUMEXP else None
        p = _params(w, d, torch.empty(M, N, device="cuda"), aux, B.FLAG_IEEE_FP32)
        assert B.fge_tile_name(True, w.act, norm, p) == "repacked_operands"
        ref, raux = H.oracle_chain(w, t)
        got, gaux = H.run_gpu(w, t, "fused", dev=d, flags=B.FLAG_IEEE_FP32)
        H.check(w, got, gaux, ref, raux, "fp32 instruction, any width")
        assert H.C.max_rel_err(got, ref) <= 2e-5       # (without the flag the split product's 2^-16.5 per term)
