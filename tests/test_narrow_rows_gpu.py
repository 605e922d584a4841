"""fp32 rows of up to 256 columns over K <= 64 in the narrow-K kernel (four waves of 64 columns across and 64 rows, or two and 128): widths
at the waves' edges, rows off the tiles, K off the staged width, every row op, fewer tiles than workgroups and several each."""
import numpy as np
import pytest

from paper_2512_23424_amd import inputs as I
from tests import _harness as H

pytestmark = pytest.mark.gpu
FLAG_PANEL = (4 + 1) << 8                   # FGE_FLAG_TILE(FGE_TILE_PANEL)
FLAG_64 = (0 + 1) << 8                      # FGE_FLAG_TILE(FGE_TILE_64x64)


@pytest.mark.parametrize("out", [I.F32, I.BF16])
@pytest.mark.parametrize("N", [64, 72, 128, 136, 192, 248, 256])
def test_exact_integers(N, out):
    for M, K in ((4097, 4), (5000, 60), (33000, 64)):
        w = I.Workload(name="narrow", M=M, K=K, N=N, in_dtype=I.F32, out_dtype=out, act=I.ACT_RELU,
                       dist={"X": ("int", -2, 2), "W": ("int", -2, 2), "b": ("int", -3, 3)})
        t = I.generate(w)
        ref, _ = H.oracle_chain(w, t)
        ref = I.as_f64(I.f64_to_bf16_bits(ref)) if out == I.BF16 else ref
        got, _ = H.run_gpu(w, t, "fused", flags=FLAG_PANEL)
        assert np.array_equal(got, ref), f"M={M} K={K}: {int((got != ref).sum())} mismatches"


@pytest.mark.parametrize("act", [I.ACT_GELU_ERF, I.ACT_CLAMP])
@pytest.mark.parametrize("norm", [I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_RMSNORM, I.NORM_LOGSUMEXP])
def test_row_operations(norm, act):
    """The choice of the library: some of these take the kernel, all are held to the same gate."""
    for M, K, N in ((4100, 64, 68), (4100, 36, 128), (9000, 20, 132), (33000, 64, 252), (40000, 48, 256), (140000, 44, 96)):
        w = I.Workload(name=f"narrow{norm}", M=M, K=K, N=N, act=act, norm=norm, post_scale=2.0, clamp_lo=-5.0, clamp_hi=5.0, eps=1e-5,
                       dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, K ** -0.5), "b": ("uniform", -0.5, 0.5),
                             "gamma": ("normal", 1.0, 0.1), "beta": ("normal", 0.0, 0.1)})
        t = I.generate(w)
        ref, raux = H.oracle_chain(w, t)
        got, gaux = H.run_gpu(w, t, "fused")
        H.check(w, got, gaux, ref, raux, "narrow rows")


@pytest.mark.parametrize("norm", [I.NORM_NONE, I.NORM_LAYERNORM])
@pytest.mark.parametrize("M,K,N", [(40000, 64, 252), (33000, 36, 192), (4100, 64, 128)])
def test_a_large_bias_costs_no_precision(norm, M, K, N):
    """A bias of 100 on every column and an uneven scale: the error is that of the general tiles, which add the bias once.  (Both errors are
    sums of the same kind over 500000 values and more; their ratio is 1 within a few per cent, and 2.9 where every partial sum
    is rounded at the bias's magnitude.)"""
    w = I.Workload(name="bias", M=M, K=K, N=N, act=I.ACT_NONE, norm=norm, alpha=0.7, post_scale=1.3, eps=1e-5,
                   dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, K ** -0.5), "b": ("uniform", 99.5, 100.5),
                         "gamma": ("normal", 1.0, 0.1), "beta": ("normal", 0.0, 0.1)})
    t = I.generate(w)
    ref, _ = H.oracle_chain(w, t)
    errors = []
    for flags in (FLAG_PANEL, FLAG_64):
        got, _ = H.run_gpu(w, t, "fused", flags=flags)
        errors.append(float(np.sqrt(np.mean((got - ref) ** 2))))
    assert errors[0] <= 1.2 * errors[1], errors
