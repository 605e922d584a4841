"""Columns masked by the bias, for softmax and logsumexp, on every path that merges statistics of
parts of a row: strips and tiles that hold masked columns only must add nothing to the row, whatever
value masks them - the infinity, the lowest finite value of a type, a large negative number."""
import pytest
import torch

from paper_2512_23424_amd import binding as B
from paper_2512_23424_amd import inputs as I

pytestmark = pytest.mark.gpu
MASKS = [float("-inf"), torch.finfo(torch.float32).min, torch.finfo(torch.bfloat16).min, -1e38, -1e30, -1e20, -1e10, -5e9, -1e6]
DT = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "f8": torch.float8_e4m3fn}


def tile(t, flags=0):
    return ((t + 1) << 8) | flags


# (type of the operands, M, K, N, flags): what runs
FEW = [("bf16", 7, 1024, 2051, 0), ("f16", 40, 1032, 2048, 0), ("f8", 17, 1024, 4098, 0), ("bf16", 16, 1024, 1500, B.FLAG_TWO_PASS)]
ANY = [("bf16", 300, 1024, 2051, 0), ("f8", 300, 272, 2050, tile(3)), ("f32", 300, 272, 2051, 0), ("f32", 300, 272, 2051, B.FLAG_IEEE_FP32),
       ("f16", 300, 272, 2049, tile(10))]
ALIGNED = [("bf16", 300, 256, 2048, tile(0)), ("f32", 300, 256, 2048, tile(0)),                        # second pass
           ("bf16", 2000, 256, 2048, tile(3)), ("f8", 700, 1024, 2048, tile(2)), ("f16", 700, 1024, 2048, tile(10)),     # one kernel
           ("bf16", 700, 256, 2048, tile(7)), ("f32", 700, 256, 2048, tile(5)), ("f32", 700, 256, 2048, tile(9)),
           ("bf16", 300, 256, 448, tile(1)), ("f32", 300, 256, 448, tile(1)), ("f32", 4200, 64, 448, 0)]               # whole rows
SLICED = [("bf16", 70, 4096, 2048, 0), ("f32", 40, 4096, 2051, 0), ("f32", 20, 2048, 16381, 0), ("f32", 3, 64, 2051, 0)]


def call(dt, M, K, N, flags, norm, b):
    g = torch.Generator(device="cuda").manual_seed(5)
    X = torch.randn(M, K, generator=g, device="cuda").to(DT[dt])
    W = (torch.randn(N, K, generator=g, device="cuda") / (1.0 if dt == "f8" else K ** 0.5)).to(DT[dt])
    alpha = 1.0 / K ** 0.5 if dt == "f8" else 1.0
    out = torch.full((M, N), float("nan"), dtype=torch.bfloat16 if dt == "f8" else DT[dt], device="cuda")
    aux = torch.full((M,), float("nan"), device="cuda") if norm == I.NORM_LOGSUMEXP else None
    p = B.make_params(X, W, out, aux_out=aux, flags=flags, alpha=alpha)
    ws = torch.empty(max(16, B.fge_workspace_bytes(True, I.ACT_NONE, norm, p)), dtype=torch.uint8, device="cuda")
    p.workspace, p.workspace_bytes = ws.data_ptr(), ws.numel()
    B.fused_gemm_epilogue(X, W, b, I.ACT_NONE, norm, p, out)
    torch.cuda.synchronize()
    ref = alpha * (X.double().cpu() @ W.double().cpu().T) + b.double().cpu()
    return out.double().cpu(), None if aux is None else aux.double().cpu(), ref


@pytest.mark.parametrize("norm", [I.NORM_SOFTMAX, I.NORM_LOGSUMEXP])
@pytest.mark.parametrize("case", FEW + ANY + ALIGNED + SLICED, ids=lambda c: "-".join(map(str, c)))
def test_masks_of_any_size_contribute_nothing(case, norm):
    dt, M, K, N, flags = case
    for mask in MASKS:
        b = torch.zeros(N, device="cuda")
        masked = torch.zeros(N, dtype=torch.bool)
        for lo, hi in ((0, N // 2 + 7), (N - N // 4, N - N // 8), (N - 40, N)):      # whole strips and tiles, parts of others
            masked[lo:hi] = True
        b[masked.cuda()] = mask
        out, aux, ref = call(dt, M, K, N, flags, norm, b)
        if norm == I.NORM_LOGSUMEXP:
            # fp32 sums of values from fp32 operands split in two, or from E4M3 sums of 64 terms: 2^-16.5, about 2e-4
            tol = {"f32": 1e-4, "f8": 2e-3}.get(dt, 1e-5)
            assert torch.allclose(aux, torch.logsumexp(ref, 1), rtol=tol), f"mask {mask}"
        else:
            # values of magnitude 5 with these errors, and the rounding of the result
            tol = {"f32": 1e-3, "f8": 2e-2, "f16": 2 ** -9}.get(dt, 2 ** -7)
            assert torch.allclose(out, torch.softmax(ref, 1), rtol=tol, atol=1e-7), f"mask {mask}"
            assert bool((out[:, masked] == 0).all()), f"mask {mask}"


@pytest.mark.parametrize("case", [("bf16", 7, 1024, 1025, 0), ("f16", 17, 1024, 4097, 0), ("bf16", 7, 1024, 1025, B.FLAG_TWO_PASS),
                                  ("bf16", 300, 1024, 2049, 0), ("bf16", 300, 256, 2056, tile(0)), ("bf16", 2000, 256, 2056, tile(3)),
                                  ("f32", 300, 256, 448, tile(1)), ("f32", 4200, 64, 456, 0)], ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("norm", [I.NORM_SOFTMAX, I.NORM_LOGSUMEXP])
def test_a_nan_column_reaches_the_result(case, norm):
    """One NaN in a row makes its logsumexp and its probabilities NaN - alone in the last strip, or among
    masked columns that have no maximum of their own."""
    dt, M, K, N, flags = case
    for columns_masked, at in (([], N - 1), ([(N - 400, N)], N - 1), ([(0, 300)], 5)):
        b = torch.zeros(N, device="cuda")
        for lo, hi in columns_masked:
            b[lo:hi] = float("-inf")
        b[at] = float("nan")
        out, aux, _ = call(dt, M, K, N, flags, norm, b)
        assert bool(torch.isnan(out[:, at]).all())
        assert bool(torch.isnan(out if norm == I.NORM_SOFTMAX else aux).all()), f"masked {columns_masked}"
