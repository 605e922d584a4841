"""Results whose rows start and end at any element, stored by the tile kernels themselves (no row op,
logsumexp, rows one tile spans) or parked in fp32 and finished by one pass (softmax, LayerNorm,
RMSNorm over several tiles): widths around the tiles' edges and the stores' groups of eight, row
strides that are odd or leave padding, which must stay untouched."""
import numpy as np
import pytest
import torch

from paper_2512_23424_amd import binding as B
from paper_2512_23424_amd import inputs as I
from tests import _harness as H

pytestmark = pytest.mark.gpu


def _run(w, d, pad, flags=0):
    buf = torch.full((w.M, w.N + pad), float("nan"), dtype=H.tdtype(w.out_dtype), device="cuda")
    out = buf[:, :w.N]
    aux = torch.full((w.M,), float("nan"), device="cuda") if w.norm == I.NORM_LOGSUMEXP else None
    p = B.make_params(d["X"], d["W"], out, alpha=w.alpha, post_scale=w.post_scale, eps=w.eps, gamma=d["gamma"], beta=d["beta"],
                      aux_out=aux, flags=flags)
    assert B.fge_tile_name(True, w.act, w.norm, p) == "repacked_operands"
    ws = torch.empty(B.fge_workspace_bytes(True, w.act, w.norm, p), dtype=torch.uint8, device="cuda")
    p.workspace, p.workspace_bytes = ws.data_ptr(), ws.numel()
    B.fused_gemm_epilogue(d["X"], d["W"], d["b"], w.act, w.norm, p, out)
    torch.cuda.synchronize()
    assert pad == 0 or bool(torch.isnan(buf[:, w.N:]).all())
    return H.to_host_f64(out.contiguous()), None if aux is None else H.to_host_f64(aux)


@pytest.mark.parametrize("dt,out", [(I.BF16, I.BF16), (I.F16, I.F32), (I.F8E4M3, I.BF16), (I.F32, I.F32), (I.F32, I.BF16)])
@pytest.mark.parametrize("tile", [0, 2, 3, 9, 10])
def test_exact_values_at_the_edges_of_tiles_and_stores(dt, out, tile):
    if (tile == 9) != (dt == I.F32) and tile in (3, 9, 10):
        pytest.skip("no such tile for these operands")
    for M, N, pad in ((300, 511, 0), (517, 257, 3), (330, 520, 1), (301, 1029, 5), (400, 770, 0)):
        w = I.Workload(name="any", M=M, K=272, N=N, in_dtype=dt, out_dtype=out,
                       dist={"X": ("int", -2, 2), "W": ("int", -2, 2), "b": ("int", -3, 3)})
        t = I.generate(w)
        ref, _ = H.oracle_chain(w, t)
        ref = I.as_f64(I.f64_to_bf16_bits(ref)) if out == I.BF16 else ref
        got, _ = _run(w, {k: H.to_device(v) for k, v in t.items()}, pad, (tile + 1) << 8)
        assert np.array_equal(got, ref), f"M={M} N={N} pad={pad}: {int((got != ref).sum())} mismatches"


@pytest.mark.parametrize("dt,out", [(I.BF16, I.BF16), (I.F16, I.F16), (I.F8E4M3, I.BF16), (I.F32, I.F32)])
@pytest.mark.parametrize("norm", [I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_RMSNORM, I.NORM_LOGSUMEXP])
def test_row_operations_on_rows_of_any_width(dt, out, norm):
    for M, K, N, pad in ((700, 1024, 61, 0), (300, 272, 515, 2), (260, 1040, 1544, 3), (130, 272, 9001, 0)):
        w = I.Workload(name=f"any{norm}", M=M, K=K, N=N, in_dtype=dt, out_dtype=out, act=I.ACT_SILU, norm=norm,
                       alpha=1.0 / K ** 0.5, post_scale=1.5, eps=1e-5,
                       dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, 1.0), "b": ("uniform", -0.5, 0.5),
                             "gamma": ("normal", 1.0, 0.1), "beta": ("normal", 0.0, 0.1)})
        t = I.generate(w)
        d = {k: H.to_device(v) for k, v in t.items()}
        ref, raux = H.oracle_chain(w, t)
        got, gaux = _run(w, d, pad)
        H.check(w, got, gaux, ref, raux, f"any rows {M}x{K}x{N}+{pad}")


@pytest.mark.parametrize("norm", [I.NORM_NONE, I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_LOGSUMEXP])
def test_stage_entry_points_in_the_room_asked_for(norm):
    """Stage 1 alone leaves the final result of an odd width, bit for bit the one-call result, in a workspace
    of exactly the size asked for (none at all without a row op)."""
    for M, K, N in ((300, 1024, 2051), (70, 1001, 1001), (40, 1024, 2051)):
        w = I.Workload(name=f"stage{norm}", M=M, K=K, N=N, in_dtype=I.BF16, out_dtype=I.BF16, act=I.ACT_SILU, norm=norm, eps=1e-5,
                       dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, 1.0 / K ** 0.5), "b": None})
        d = {k: H.to_device(v) for k, v in I.generate(w).items()}
        want, waux = _run(w, d, 0)
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        aux = torch.full((M,), float("nan"), device="cuda") if norm == I.NORM_LOGSUMEXP else None
        p = B.make_params(d["X"], d["W"], out, eps=w.eps, aux_out=aux)
        n = B.fge_workspace_bytes(True, w.act, norm, p)
        ws = torch.full((n + 1024,), 0xA5, dtype=torch.uint8, device="cuda")
        if n:
            p.workspace, p.workspace_bytes = ws.data_ptr(), n
        B.fge_fused_tiles(d["X"], d["W"], None, w.act, norm, p, out)
        assert not B.fge_fused_needs_finish(w.act, norm, p)
        B.fge_fused_finish(w.act, norm, p, out)
        torch.cuda.synchronize()
        got = H.to_host_f64(out)
        assert bool((ws[n:] == 0xA5).all())
        if M > 64 and K % 8 == 0:
            assert np.array_equal(got, want) and (aux is None or np.array_equal(H.to_host_f64(aux), waux))
        else:                                          # (few rows, copied operands: the stages keep the element-granular product)
            assert np.isfinite(got).all() and np.abs(got - want).max() <= 2.0 ** -6 * np.abs(want).max()


def test_the_least_workspace_and_less():
    """Copied operands and the row statistics are all the direct form needs of the workspace; with a byte less the
    element-granular kernels run, with the fp32 rows those need."""
    M, K, N = 333, 2049, 515
    w = I.Workload(name="least", M=M, K=K, N=N, in_dtype=I.BF16, out_dtype=I.BF16, act=I.ACT_SILU, norm=I.NORM_LOGSUMEXP,
                   dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, 1.0 / K ** 0.5), "b": None})
    t = I.generate(w)
    d = {k: H.to_device(v) for k, v in t.items()}
    ref, raux = H.oracle_chain(w, t)
    whole, waux = _run(w, d, 0)
    up = lambda n: (n + 255) // 256 * 256
    # X and W in rows of 2056 values, W to 516 rows; statistics of nine 64-column tiles, two strips each
    least = up(M * 2056 * 2) + up(516 * 2056 * 2) + up(M * 18 * 8)
    for n, same in ((least, True), (least - 1, False)):
        out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
        aux = torch.full((M,), float("nan"), device="cuda")
        p = B.make_params(d["X"], d["W"], out, aux_out=aux)
        assert M * N * 4 < n < B.fge_workspace_bytes(True, w.act, w.norm, p)
        ws = torch.full((n + 1024,), 0xA5, dtype=torch.uint8, device="cuda")
        p.workspace, p.workspace_bytes = ws.data_ptr(), n
        B.fused_gemm_epilogue(d["X"], d["W"], None, w.act, w.norm, p, out)
        torch.cuda.synchronize()
        assert bool((ws[n:] == 0xA5).all())
        H.check(w, H.to_host_f64(out), H.to_host_f64(aux), ref, raux, f"{n} bytes")
        assert np.array_equal(H.to_host_f64(aux), waux) == same


@pytest.mark.parametrize("M", [7, 300])
@pytest.mark.parametrize("norm", [I.NORM_SOFTMAX, I.NORM_LOGSUMEXP])
def test_masked_columns_contribute_nothing(M, norm):
    """A bias of -inf masks columns, whole strips of a tile among them: probabilities of zero and a
    finite logsumexp, for few rows and for rows of odd width."""
    K, N = 1024, 2051
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn(M, K, generator=g, device="cuda").bfloat16()
    W = (torch.randn(N, K, generator=g, device="cuda") / K ** 0.5).bfloat16()
    b = torch.zeros(N, device="cuda")
    b[64:330] = b[1000:1016] = b[1800:] = float("-inf")
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda")
    aux = torch.full((M,), float("nan"), device="cuda") if norm == I.NORM_LOGSUMEXP else None
    p = B.make_params(X, W, out, aux_out=aux)
    ws = torch.empty(B.fge_workspace_bytes(True, I.ACT_NONE, norm, p), dtype=torch.uint8, device="cuda")
    p.workspace, p.workspace_bytes = ws.data_ptr(), ws.numel()
    B.fused_gemm_epilogue(X, W, b, I.ACT_NONE, norm, p, out)
    torch.cuda.synchronize()
    ref = X.double().cpu() @ W.double().cpu().T + b.double().cpu()
    if norm == I.NORM_LOGSUMEXP:
        assert torch.allclose(aux.double().cpu(), torch.logsumexp(ref, 1), rtol=1e-5)      # fp32 sums
        assert bool((out[:, 1800:] == float("-inf")).all())
    else:
        assert torch.allclose(out.double().cpu(), torch.softmax(ref, 1), rtol=2 ** -7, atol=1e-9)   # one bf16 rounding
        assert bool((out[:, 64:330] == 0).all())


@pytest.mark.parametrize("dt", [I.BF16, I.F8E4M3])
@pytest.mark.parametrize("norm", [I.NORM_NONE, I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_RMSNORM, I.NORM_LOGSUMEXP])
def test_columns_behind_whole_rounds_are_a_launch_of_their_own(dt, norm):
    """17 x 17 tiles of 256x256: 15 column tiles are a whole round, the other columns (259, the last ones alone in their tile)
    run in 128x128 tiles; the statistics of a row come from both."""
    K = 1032 if dt == I.BF16 else 2064
    w = I.Workload(name=f"tail{norm}", M=4300, K=K, N=4099, in_dtype=dt, out_dtype=I.BF16, act=I.ACT_SILU, norm=norm, eps=1e-5,
                   alpha=1.0 if dt == I.BF16 else K ** -0.5,
                   dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, K ** -0.5 if dt == I.BF16 else 1.0), "b": ("uniform", -0.5, 0.5),
                         "gamma": ("normal", 1.0, 0.1), "beta": ("normal", 0.0, 0.1)})
    t = I.generate(w)
    got, gaux = H.run_gpu(w, t, "fused")
    ref, raux = H.oracle_chain(w, t)
    H.check(w, got, gaux, ref, raux, "columns behind whole rounds")
