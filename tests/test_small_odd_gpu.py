"""Small products of odd extents (element-granular product: 32x32 tiles, 128 k at a time or all of a K of up to 32 or 64, shared out by four waves): exact integers
around the K tile and the waves' parts of it, around the output tile, and with strides."""
import numpy as np
import pytest
import torch

from paper_2512_23424_amd import binding as B
from paper_2512_23424_amd import inputs as I
from tests import _harness as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [I.F32, I.BF16, I.F16, I.F8E4M3])
def test_exact_sums(dt):
    for M, N in ((1, 33), (31, 31), (33, 65), (70, 97)):
        for K in (1, 3, 31, 32, 33, 63, 64, 65, 127, 129, 161, 255, 257, 429):
            w = I.Workload(name="odd", M=M, K=K, N=N, in_dtype=dt, out_dtype=I.F32, act=I.ACT_RELU,
                           dist={"X": ("int", -2, 2), "W": ("int", -2, 2), "b": ("int", -3, 3)})
            t = I.generate(w)
            ref, _ = H.oracle_chain(w, t)
            got, _ = H.run_gpu(w, t, "fused")
            assert np.array_equal(got, ref), f"K={K} M={M} N={N}: {int((got != ref).sum())} mismatches"


@pytest.mark.parametrize("norm", [I.NORM_SOFTMAX, I.NORM_LAYERNORM])
def test_fp32_precision(norm):
    """fp32 products and sums: the gate of the fp32 instruction."""
    w = I.Workload(name="odd32", M=365, K=429, N=33, act=I.ACT_SILU, norm=norm, eps=1e-5,
                   dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, 429 ** -0.5), "b": ("uniform", -0.5, 0.5),
                         "gamma": ("normal", 1.0, 0.1), "beta": ("normal", 0.0, 0.1)})
    t = I.generate(w)
    ref, raux = H.oracle_chain(w, t)
    got, gaux = H.run_gpu(w, t, "fused")
    assert B.fge_tile_name(True, w.act, norm, B.make_params(*(H.to_device(t[k]) for k in "XW"), H.to_device(got.astype(np.float32)))) == "generic32x32_scalar"
    assert H.C.max_rel_err(got, ref) <= 2e-5


@pytest.mark.parametrize("dt", [I.F32, I.BF16, I.F16])
@pytest.mark.parametrize("norm", [I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_RMSNORM, I.NORM_LOGSUMEXP])
def test_row_operations_of_odd_width(dt, norm):
    """fge_row_op on rows that start and end at any element: widths around the chunks of a lane, a wave and a workgroup, few rows and
    many, out of place and in place."""
    td = H.tdtype(dt)
    g = torch.Generator(device="cuda").manual_seed(3)
    for M, N in ((3, 1), (40, 63), (1030, 65), (40, 97), (1030, 193), (40, 319), (1030, 321), (5, 255), (1030, 257), (1030, 511), (1500, 513), (1030, 1029), (40, 1025), (40, 2049), (9, 4097), (5, 8191)):
        A = (torch.randn(M, N, generator=g, device="cuda") * 2).to(td)
        gamma = 1 + 0.1 * torch.randn(N + 3, generator=g, device="cuda")[:N]
        beta = 0.1 * torch.randn(N + 3, generator=g, device="cuda")[:N]
        x = A.double()
        raux = torch.logsumexp(x, 1)
        if norm == I.NORM_SOFTMAX:
            ref = torch.softmax(x, 1)
        elif norm == I.NORM_LAYERNORM:
            ref = (x - x.mean(1, keepdim=True)) / (x.var(1, unbiased=False, keepdim=True) + 1e-5).sqrt() * gamma.double() + beta.double()
        elif norm == I.NORM_RMSNORM:
            ref = x / ((x * x).mean(1, keepdim=True) + 1e-5).sqrt() * gamma.double()
        else:
            ref = x
        for inplace in (False, True):
            src = A.clone()
            out = src if inplace else torch.full_like(A, float("nan"))
            aux = torch.full((M,), float("nan"), device="cuda") if norm == I.NORM_LOGSUMEXP else None
            p = B.make_params(None, None, out, eps=1e-5, gamma=gamma, beta=beta, aux_out=aux)
            B.fge_row_op(src, norm, p, out)
            torch.cuda.synchronize()
            # one rounding to the result's type on top of fp32 arithmetic
            tol = {I.F32: 2e-5, I.BF16: 2.0 ** -8, I.F16: 2.0 ** -10}[dt]
            den = ref.abs().maximum(ref.abs().mean(1, keepdim=True))
            assert float(((out.double() - ref).abs() / den).max()) <= tol, (M, N, inplace)
            if aux is not None:
                assert float((aux.double() - raux).abs().max()) <= 1e-4


def test_more_rows_than_workgroups_of_four_waves():
    """2^24 rows of more columns than one wave takes: a workgroup of 256 per row would pass the 2^32 work items a launch may have."""
    M, N = 1 << 24, 2049
    if torch.cuda.mem_get_info()[0] < M * N * 2 + (4 << 30):
        pytest.skip("needs 73 GB of device memory")
    A = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
    A.fill_(0.5)
    rows = torch.tensor([0, 1, 12345, (1 << 23) + 7, M - 2, M - 1], device="cuda")
    A[rows] = (torch.randn(len(rows), N, generator=torch.Generator(device="cuda").manual_seed(5), device="cuda") * 2).to(torch.bfloat16)
    ref = torch.logsumexp(A[rows].double(), 1)
    aux = torch.full((M,), float("nan"), device="cuda")
    p = B.make_params(None, None, A, aux_out=aux)
    B.fge_row_op(A, I.NORM_LOGSUMEXP, p, A)
    torch.cuda.synchronize()
    assert float((aux[rows].double() - ref).abs().max()) <= 1e-4          # fp32 arithmetic on values near 10
    others = torch.ones(M, dtype=torch.bool, device="cuda")
    others[rows] = False
    assert float((aux[others] - (0.5 + float(np.log(N)))).abs().max()) <= 1e-4
    del A
    torch.cuda.empty_cache()


def test_no_row_op_in_place_leaves_every_byte():
    """Signalling NaNs included: there is nothing to write back."""
    A = torch.arange(-(1 << 15), 1 << 15, device="cuda").to(torch.int16)[:4 * 16381].reshape(4, 16381)[:, :4095].contiguous()
    A[1, 7] = 0x7F81                        # a signalling NaN in bf16 and in fp16
    out = A.clone().view(torch.bfloat16)
    B.fge_row_op(out, I.NORM_NONE, B.make_params(None, None, out), out)
    torch.cuda.synchronize()
    assert torch.equal(out.view(torch.int16), A)
