"""The two mainloops of the 256x256 tiles - by quadrants: two K tiles are in flight when a tile is multiplied,
buffers and register sets change with the tile's parity, copies past the end move nothing and the
chunks past K are zeroed by hand; by k-steps up to four K tiles of 16-bit operands (one of 8-bit ones): one K tile in flight, a
partial one through registers.  Exact integers over one to eleven K tiles, whole and partial."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2512_23424_amd import binding as B
from paper_2512_23424_amd import inputs as I
from tests import _harness as H

pytestmark = pytest.mark.gpu
FLAG_256 = (3 + 1) << 8                     # FGE_FLAG_TILE(FGE_TILE_256x256)


def _rounded(ref, dt):
    """The exact integers as the result type holds them (round to nearest even)."""
    if dt == I.BF16:
        return I.as_f64(I.f64_to_bf16_bits(ref))
    return ref.astype(np.float16).astype(np.float64) if dt == I.F16 else ref


@pytest.mark.parametrize("dt,out", [(I.BF16, I.F32), (I.BF16, I.BF16), (I.F16, I.F16), (I.F8E4M3, I.F32), (I.F8E4M3, I.BF16)])
@pytest.mark.parametrize("gated", [False, True])
def test_k_tiles_of_the_quadrant_mainloop(dt, out, gated):
    unit, tile_k = (16, 128) if dt == I.F8E4M3 else (8, 64)
    _sweep(dt, out, gated, sorted({unit, tile_k - unit, tile_k, tile_k + unit, 2 * tile_k, 2 * tile_k + unit, 3 * tile_k,
                                   4 * tile_k - unit, 4 * tile_k, 5 * tile_k + unit}))


@pytest.mark.parametrize("dt,out", [(I.BF16, I.F32), (I.BF16, I.BF16), (I.F16, I.F16)])
@pytest.mark.parametrize("gated", [False, True])
def test_k_tiles_around_and_past_the_line_between_the_loops(dt, out, gated):
    _sweep(dt, out, gated, (4 * 64 + 8, 5 * 64 - 8, 5 * 64, 6 * 64 - 8, 6 * 64, 6 * 64 + 8, 7 * 64, 8 * 64 + 8, 9 * 64, 11 * 64 + 8))


def _sweep(dt, out, gated, ks):
    for K in ks:
        for M, N in ((260, 264), (530, 520)):
            w = I.Workload(name="quad", M=M, K=K, N=N, in_dtype=dt, out_dtype=out,
                           dist={"X": ("int", -2, 2), "W": ("int", -2, 2), "b": ("int", -3, 3)})
            t = I.generate_gated(w) if gated else I.generate(w)
            d = {k: H.to_device(v) for k, v in t.items()}
            if gated:
                f = {k: I.as_f64(v) for k, v in t.items()}
                ref, _ = O.gated_chain(f["X"], f["W"], f["W2"], f["b"], f["b2"], None, None, act=w.act, norm=w.norm, eps=w.eps)
                got = torch.full((M, N), float("nan"), dtype=H.tdtype(out), device="cuda")
                p = B.make_params(d["X"], d["W"], got)
                assert B.fge_gated_tile_name(w.act, w.norm, p) == "gated256x128_w2x4"
                B.fused_gated_gemm_epilogue(d["X"], d["W"], d["W2"], d["b"], d["b2"], w.act, w.norm, p, got)
                torch.cuda.synchronize()
                got = H.to_host_f64(got)
            else:
                ref, _ = H.oracle_chain(w, t)
                got, _ = H.run_gpu(w, t, "fused", dev=d, flags=FLAG_256)
            ref = _rounded(ref, out)
            assert np.array_equal(got, ref), f"K={K} M={M} N={N}: {int((got != ref).sum())} mismatches"
