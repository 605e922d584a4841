"""Products of at most 64 rows: whole sums per workgroup, the K tiles shared out over its waves,
results of any width.  Exact integers over every phase of the wave rings (one tile per wave and less,
partial tiles, rings that wrap), then the row operations - inside the launch and as a second
kernel, which must agree bit for bit - against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2512_23424_amd import binding as B
from paper_2512_23424_amd import inputs as I
from tests import _harness as H

pytestmark = pytest.mark.gpu
NORMS = [I.NORM_NONE, I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_RMSNORM, I.NORM_LOGSUMEXP]


def _gated(w, d, flags=0):
    out = torch.full((w.M, w.N), float("nan"), dtype=H.tdtype(w.out_dtype), device="cuda")
    aux = torch.full((w.M,), float("nan"), device="cuda") if w.norm == I.NORM_LOGSUMEXP else None
    p = B.make_params(d["X"], d["W"], out, alpha=w.alpha, post_scale=w.post_scale, eps=w.eps, gamma=d["gamma"], beta=d["beta"],
                      aux_out=aux, flags=flags)
    n = B.fge_gated_workspace_bytes(True, w.act, w.norm, p)
    ws = torch.full((n // 4 + 64,), float("nan"), device="cuda")
    p.workspace, p.workspace_bytes = ws.data_ptr(), n
    B.fused_gated_gemm_epilogue(d["X"], d["W"], d["W2"], d["b"], d["b2"], w.act, w.norm, p, out)
    torch.cuda.synchronize()
    assert bool(torch.isnan(ws[(n + 3) // 4:]).all())
    return H.to_host_f64(out), None if aux is None else H.to_host_f64(aux)


@pytest.mark.parametrize("dt", [I.BF16, I.F16, I.F8E4M3])
@pytest.mark.parametrize("gated", [False, True])
def test_exact_sums_over_rows_columns_and_k_tiles(dt, gated):
    unit, tile_k = (16, 128) if dt == I.F8E4M3 else (8, 64)
    for M, N in ((1, 16), (16, 4104), (17, 8232), (32, 24), (33, 1032), (64, 8200)):
        for K in (8 * tile_k, 8 * tile_k + unit, 15 * tile_k - unit, 17 * tile_k, 41 * tile_k + 3 * unit):
            w = I.Workload(name="few", M=M, K=K, N=N if gated else N - (N % 3), in_dtype=dt, out_dtype=I.F32,
                           dist={"X": ("int", -2, 2), "W": ("int", -2, 2), "b": ("int", -3, 3)})
            t = I.generate_gated(w) if gated else I.generate(w)
            d = {k: H.to_device(v) for k, v in t.items()}
            if gated:
                f = {k: I.as_f64(v) for k, v in t.items()}
                ref, _ = O.gated_chain(f["X"], f["W"], f["W2"], f["b"], f["b2"], None, None, act=w.act, norm=w.norm, eps=w.eps)
                got, _ = _gated(w, d)
            else:
                ref, _ = H.oracle_chain(w, t)
                got, _ = H.run_gpu(w, t, "fused", dev=d)
            # sums stay below 2^24 and the gate's product of two is rounded once to fp32
            ref = ref.astype(np.float32).astype(np.float64)
            assert np.array_equal(got, ref), f"M={M} N={w.N} K={K}: {int((got != ref).sum())} mismatches"


@pytest.mark.parametrize("dt,out", [(I.BF16, I.BF16), (I.F16, I.F16), (I.F8E4M3, I.BF16), (I.BF16, I.F32)])
@pytest.mark.parametrize("norm", NORMS)
def test_row_operations_in_one_launch_and_in_two(dt, out, norm):
    """Widths: fewer workgroups than rows, odd ones, the widest row and the first too wide for the
    product's own workgroups, the widest of all, and (logsumexp) one wider still."""
    for M, K, N, act in ((64, 1032, 72, I.ACT_GELU_ERF), (5, 2048, 4099, I.ACT_SILU), (33, 1040, 1001, I.ACT_RELU), (18, 1024, 8192, I.ACT_SILU),
                         (3, 1024, 8200, I.ACT_GELU_TANH), (2, 1024, 16384, I.ACT_SILU), (18, 1024, 33001, I.ACT_NONE)):
        K = K // 16 * 16 if dt == I.F8E4M3 else K
        w = I.Workload(name=f"few{norm}", M=M, K=K, N=N, in_dtype=dt, out_dtype=out, act=act, norm=norm,
                       alpha=1.0 / K ** 0.5, post_scale=1.5, eps=1e-5,
                       dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, 1.0), "b": ("uniform", -0.5, 0.5),
                             "gamma": ("normal", 1.0, 0.1), "beta": ("normal", 0.0, 0.1)})
        t = I.generate(w)
        d = {k: H.to_device(v) for k, v in t.items()}
        ref, raux = H.oracle_chain(w, t)
        got, gaux = H.run_gpu(w, t, "fused", dev=d)
        H.check(w, got, gaux, ref, raux, f"one launch {M}x{K}x{N}")
        two, taux = H.run_gpu(w, t, "fused", dev=d, flags=B.FLAG_TWO_PASS)
        assert np.array_equal(got, two) and (gaux is None or np.array_equal(gaux, taux))
        if N % 8 == 0:
            t = I.generate_gated(w)
            d = {k: H.to_device(v) for k, v in t.items()}
            f = {k: I.as_f64(v) for k, v in t.items()}
            ref, raux = O.gated_chain(f["X"], f["W"], f["W2"], f["b"], f["b2"], f["gamma"], f["beta"], alpha=w.alpha,
                                      post_scale=w.post_scale, act=w.act, norm=w.norm, eps=w.eps)
            got, gaux = _gated(w, d)
            H.check(w, got, gaux, ref, raux, f"gated {M}x{K}x{N}")
            two, taux = _gated(w, d, B.FLAG_TWO_PASS)
            assert np.array_equal(got, two) and (gaux is None or np.array_equal(gaux, taux))


def test_strided_operands_and_an_odd_result_stride():
    M, K, N = 20, 1096, 515
    w = I.Workload(name="fewld", M=M, K=K, N=N, in_dtype=I.BF16, out_dtype=I.BF16, act=I.ACT_SILU, norm=I.NORM_SOFTMAX,
                   dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, 0.05), "b": None})
    t = I.generate(w)
    d = {k: H.to_device(v) for k, v in t.items()}
    ref, _ = H.oracle_chain(w, t)
    Xb = torch.full((M, K + 24), float("nan"), dtype=torch.bfloat16, device="cuda"); Xb[:, :K] = d["X"]
    Wb = torch.full((N, K + 8), float("nan"), dtype=torch.bfloat16, device="cuda"); Wb[:, :K] = d["W"]
    ob = torch.full((M, N + 2), float("nan"), dtype=torch.bfloat16, device="cuda")
    X, W, out = Xb[:, :K], Wb[:, :K], ob[:, :N]
    p = B.make_params(X, W, out)
    ws = torch.empty(B.fge_workspace_bytes(True, w.act, w.norm, p), dtype=torch.uint8, device="cuda")
    p.workspace, p.workspace_bytes = ws.data_ptr(), ws.numel()
    B.fused_gemm_epilogue(X, W, None, w.act, w.norm, p, out)
    torch.cuda.synchronize()
    H.check(w, H.to_host_f64(out), None, ref, None, "strided")
    assert bool(torch.isnan(ob[:, N:]).all())


@pytest.mark.parametrize("norm", [I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_RMSNORM, I.NORM_LOGSUMEXP])
def test_a_wait_that_runs_out_poisons_the_rows(norm):
    """The first workgroup keeps its mark back and every wait gives up after one poll: each row's
    workgroup waits in vain, the rows come back as NaN and the fault word is set."""
    w = I.Workload(name="fewexpire", M=8, K=1024, N=1024, in_dtype=I.BF16, out_dtype=I.BF16, act=I.ACT_SILU, norm=norm, eps=1e-5,
                   dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, 0.1), "b": None})
    t = I.generate(w)
    d = {k: H.to_device(v) for k, v in t.items()}
    got, gaux = H.run_gpu(w, t, "fused", dev=d, flags=B.FLAG_TEST_EXPIRE_WAIT, expect_fault=True)
    assert np.isnan(gaux if norm == I.NORM_LOGSUMEXP else got).all()
    ref, raux = H.oracle_chain(w, t)
    got, gaux = H.run_gpu(w, t, "fused", dev=d)
    H.check(w, got, gaux, ref, raux, "after an expired wait")


@pytest.mark.parametrize("dt", [I.BF16, I.F16, I.F8E4M3])
def test_sums_are_as_exact_as_those_of_k_slices(dt):
    """fp32 results over a long K against float64, beside the same call in K slices of 64x64 tiles (which the forced
    tile takes): the error is a matter of how long the chains of additions are, which is its square root - 512 values
    in either form at K = 8192; at 16384, where there are 16 slices and no more, 1024 against half a slice's 1024."""
    for M, K, N, longer in ((64, 8192, 2048, 1), (16, 8192, 1024, 1), (1, 16384, 1024, 2)):
        g = torch.Generator(device="cuda").manual_seed(3)
        tdt = {I.BF16: torch.bfloat16, I.F16: torch.float16, I.F8E4M3: torch.float8_e4m3fn}[dt]
        X = torch.randn(M, K, generator=g, device="cuda").to(tdt)
        W = torch.randn(N, K, generator=g, device="cuda").to(tdt)
        ref = X.double() @ W.double().T
        err = []
        for flags in (0, 1 << 8):
            out = torch.full((M, N), float("nan"), device="cuda")
            p = B.make_params(X, W, out, flags=flags)
            ws = torch.empty(B.fge_workspace_bytes(True, I.ACT_NONE, I.NORM_NONE, p), dtype=torch.uint8, device="cuda")
            p.workspace, p.workspace_bytes = ws.data_ptr(), ws.numel()
            B.fused_gemm_epilogue(X, W, None, I.ACT_NONE, I.NORM_NONE, p, out)
            torch.cuda.synchronize()
            err.append(float((out.double() - ref).norm() / ref.norm()))
        print(f"dt {dt} {M}x{K}x{N}: few-row {err[0]:.3e}, K slices {err[1]:.3e}", flush=True)
        assert err[0] <= 1.02 * longer ** 0.5 * err[1]                 # (2 %: the spread of either over seeds)
