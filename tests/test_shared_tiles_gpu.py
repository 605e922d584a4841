"""Tiles shared between workgroups (the last, partial round of 256x256 and gated tiles; all tiles of a problem that has
few of them): each workgroup multiplies a slice of K, the sums meet in the workspace, and a second launch adds and finishes
them.  Slices that end inside a K tile, two and four of them, ragged rows and columns, whole rounds in front,
every row op in each of its forms, and the ways around sharing.  A call's workspace tells whether it shared: filled with a pattern
before the call, it holds a tile's sums (256 KB) per shared tile and slice afterwards."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2512_23424_amd import binding as B
from paper_2512_23424_amd import inputs as I
from tests import _harness as H

pytestmark = pytest.mark.gpu
FLAG_256 = (3 + 1) << 8                     # FGE_FLAG_TILE(FGE_TILE_256x256)
TILE_BYTES = 256 * 256 * 4                  # partial sums of a tile
NORMS = [I.NORM_NONE, I.NORM_SOFTMAX, I.NORM_LAYERNORM, I.NORM_RMSNORM, I.NORM_LOGSUMEXP]


def _workload(dt, M, K, N, act, norm, odt=None):
    f8 = dt == I.F8E4M3
    return I.Workload(name=f"shared{act}{norm}", M=M, K=K, N=N, in_dtype=dt, out_dtype=odt or (I.BF16 if f8 else dt), act=act, norm=norm,
                      alpha=K ** -0.5 if f8 else 0.5, post_scale=1.5, clamp_lo=-1.0, clamp_hi=2.0, eps=1e-5,
                      dist={"X": ("normal", 0.0, 1.0), "W": ("normal", 0.0, 1.0 if f8 else K ** -0.5), "b": ("uniform", -0.5, 0.5),
                            "gamma": ("normal", 1.0, 0.1), "beta": ("normal", 0.0, 0.1)})


def _call(w, t, gated, flags=0, ws_bytes=None):
    """One call on a workspace of the size asked for; (result, aux, bytes of the workspace it has written)."""
    d = {k: H.to_device(v) for k, v in t.items()}
    out = torch.full((w.M, w.N), float("nan"), dtype=H.tdtype(w.out_dtype), device="cuda")
    aux = torch.full((w.M,), float("nan"), device="cuda") if w.norm == I.NORM_LOGSUMEXP else None
    p = B.make_params(d["X"], d["W"], out, alpha=w.alpha, post_scale=w.post_scale, clamp_lo=w.clamp_lo, clamp_hi=w.clamp_hi, eps=w.eps,
                      gamma=d["gamma"], beta=d["beta"], aux_out=aux, flags=flags)
    n = (B.fge_gated_workspace_bytes if gated else B.fge_workspace_bytes)(True, w.act, w.norm, p) if ws_bytes is None else ws_bytes
    raw = torch.full((n + 1024,), 0xA5, dtype=torch.uint8, device="cuda")
    p.workspace, p.workspace_bytes = raw.data_ptr(), n
    if gated:
        B.fused_gated_gemm_epilogue(d["X"], d["W"], d["W2"], d["b"], d["b2"], w.act, w.norm, p, out)
    else:
        B.fused_gemm_epilogue(d["X"], d["W"], d["b"], w.act, w.norm, p, out)
    torch.cuda.synchronize()
    assert bool((raw[n:] == 0xA5).all()), "the call wrote past the end of its workspace"
    words = raw[:n // 4 * 4].view(torch.int32)
    written = 4 * int((words != -0x5a5a5a5b).sum())
    return H.to_host_f64(out), None if aux is None else H.to_host_f64(aux), written


def _reference(w, t, gated):
    if not gated:
        return H.oracle_chain(w, t)
    f = {k: I.as_f64(v) for k, v in t.items()}
    return O.gated_chain(f["X"], f["W"], f["W2"], f["b"], f["b2"], f["gamma"], f["beta"], alpha=w.alpha, post_scale=w.post_scale,
                         act=w.act, clamp_lo=w.clamp_lo, clamp_hi=w.clamp_hi, norm=w.norm, eps=w.eps)


@pytest.mark.parametrize("dt,out", [(I.BF16, I.F32), (I.F16, I.F32), (I.F8E4M3, I.F32)])
@pytest.mark.parametrize("gated", [False, True])
def test_slices_give_exact_sums(dt, out, gated):
    """Small integers: the sums are exact whatever their order.  4 to 9 tiles (gated: 27 in four slices, 68 in two), KT K tiles of which the
    last may be partial."""
    unit, tile_k = (16, 128) if dt == I.F8E4M3 else (8, 64)
    k_tiles, sizes = ((49, 52, 51), ((530, 1032), (1000, 2056))) if gated else ((10, 11, 12, 16, 18), ((260, 264), (530, 520)))
    for i, KT in enumerate(k_tiles):
        K = KT * tile_k + (0, -unit, unit, 0, unit)[i]
        for M, N in sizes:
            w = I.Workload(name="shared", M=M, K=K, N=N, in_dtype=dt, out_dtype=out,
                           dist={"X": ("int", -2, 2), "W": ("int", -2, 2), "b": ("int", -3, 3)})
            t = I.generate_gated(w) if gated else I.generate(w)
            ref, _ = _reference(w, t, gated)
            got, _, written = _call(w, t, gated, 0 if gated else FLAG_256)
            assert written >= (27 * 4 if gated else 4 * 2) * TILE_BYTES, (K, M, N, written / TILE_BYTES)
            assert np.array_equal(got, ref), f"K={K} M={M} N={N}: {int((got != ref).sum())} mismatches"


@pytest.mark.parametrize("M,N,blocks", [(4300, 4096, 16 * 4), (5000, 1000, 80 * 2)])       # 16 tiles left; no whole round, 80 tiles
@pytest.mark.parametrize("norm", NORMS)
def test_left_over_tiles(norm, M, N, blocks):
    """Shared without a row op; with one, tiles that exchange row statistics inside the launch share nothing."""
    w = _workload(I.BF16, M, 2056, N, I.ACT_SILU, norm)
    t = I.generate(w)
    ref, raux = H.oracle_chain(w, t)
    for flags in (FLAG_256, FLAG_256 | B.FLAG_NO_SPLIT_K):
        got, gaux, written = _call(w, t, False, flags)
        H.check(w, got, gaux, ref, raux, f"flags={flags}")
        assert (written >= blocks * TILE_BYTES) == (norm == I.NORM_NONE and flags == FLAG_256), written / TILE_BYTES


@pytest.mark.parametrize("dt", [I.BF16, I.F16, I.F8E4M3])
@pytest.mark.parametrize("norm", NORMS)
def test_all_tiles_shared(dt, norm):
    """Few tiles over a long K: the row op in the tile (one column tile) or in a kernel over fp32 rows."""
    for gated, M, K, N, blocks in ((True, 300, 4104, 1400, 22 * 4), (True, 400, 4104, 3080, 50 * 4), (False, 1500, 8200, 2824, 72 * 2),
                                   (False, 2100, 640, 248, 9 * 2)):
        if dt == I.F8E4M3:
            if N == 2824:                            # (8-bit operands do not gain there and run in 128x128 tiles)
                continue
            K *= 2
        forced = N <= 256
        w = _workload(dt, M, K, N, I.ACT_SILU if gated else I.ACT_GELU_ERF, norm, odt=I.F32 if forced else None)
        t = I.generate_gated(w) if gated else I.generate(w)
        ref, raux = _reference(w, t, gated)
        for flags in (0, B.FLAG_NO_SPLIT_K):
            got, gaux, written = _call(w, t, gated, flags | (FLAG_256 if forced else 0))
            H.check(w, got, gaux, ref, raux, f"gated={gated} flags={flags}")
            assert (written >= blocks * TILE_BYTES) == (flags == 0), (gated, M, N, flags, written / TILE_BYTES)


@pytest.mark.parametrize("norm", [I.NORM_RMSNORM])
def test_an_expired_wait_leaves_nan(norm):
    """Rows that span several tiles behind whole rounds: every first column tile keeps its mark back and waits end after
    one poll: NaN, never partial statistics; all else is right."""
    w = _workload(I.BF16, 4300, 1032, 4096, I.ACT_RELU, norm)
    t = I.generate(w)
    ref, _ = H.oracle_chain(w, t)
    got, _ = H.run_gpu(w, t, "fused", flags=FLAG_256 | B.FLAG_TEST_EXPIRE_WAIT, expect_fault=True)
    ok = np.isfinite(got)
    assert not ok.all()
    den = np.maximum(np.abs(ref), H.C.row_floor(ref))
    assert (np.abs(got - ref)[ok] / den[ok]).max(initial=0.0) <= 2e-2
    got, _ = H.run_gpu(w, t, "fused", flags=FLAG_256)
    H.check(w, got, None, ref, None, "after an expired wait")


# (gated, forced tile, M, K, N, tiles shared x slices): all tiles and a last round, two slices and four, one column tile and several
WAYS = [(False, True, 4300, 2056, 4096, 16 * 4), (False, True, 5000, 4104, 1000, 80 * 2), (False, True, 2100, 1288, 248, 9 * 4),
        (False, False, 1500, 8200, 2824, 72 * 2), (True, False, 300, 4104, 1400, 22 * 4), (True, False, 2304, 1288, 3712, 5 * 4),
        (True, False, 2600, 4104, 128, 11 * 4)]


@pytest.mark.parametrize("way", range(len(WAYS)))
@pytest.mark.parametrize("norm", [I.NORM_NONE, I.NORM_SOFTMAX, I.NORM_LOGSUMEXP])
def test_shared_tiles_are_taken_and_wait_for_nothing(way, norm):
    """The partial sums are there, and a launch whose waits end after one poll - of which there are none - is as right as any."""
    gated, forced, M, K, N, blocks = WAYS[way]
    dt = I.F16 if way % 2 else I.BF16
    w = _workload(dt, M, K, N, I.ACT_SILU, norm, odt=I.F32 if way % 3 == 0 else None)
    t = I.generate_gated(w) if gated else I.generate(w)
    ref, raux = _reference(w, t, gated)
    flags = FLAG_256 if forced else 0
    column_tiles = -(-N // (128 if gated else 256))
    whole_rounds = forced or M == 2304
    # (behind whole rounds, rows over several column tiles - up to 64, logsumexp 16 - are finished by an exchange of statistics instead)
    if not (whole_rounds and norm != I.NORM_NONE and 1 < column_tiles <= (16 if norm == I.NORM_LOGSUMEXP else 64)):
        got, gaux, written = _call(w, t, gated, flags | B.FLAG_TEST_EXPIRE_WAIT)
        H.check(w, got, gaux, ref, raux, "waits of one poll")
        assert written >= blocks * TILE_BYTES, (written / TILE_BYTES, blocks)
    got, gaux, written = _call(w, t, gated, flags | B.FLAG_NO_SPLIT_K)
    H.check(w, got, gaux, ref, raux, "not shared")
    assert written < min(blocks * TILE_BYTES, 2 * TILE_BYTES + 3 * w.M * w.N * 4)


@pytest.mark.parametrize("dt,norm", [(I.BF16, n) for n in NORMS] + [(I.F16, I.NORM_SOFTMAX), (I.F8E4M3, I.NORM_LAYERNORM)])
def test_statistics_of_rows_with_shared_and_unshared_tiles(dt, norm):
    """More column tiles than an exchange inside the launch is made for (66): the last 74 of 330 tiles in two slices, and a second pass
    over rows whose strip pairs come from both launches."""
    K = 2568 if dt != I.F8E4M3 else 5136
    w = _workload(dt, 1030, K, 16648, I.ACT_RELU, norm, odt=I.BF16 if dt != I.F16 else None)
    t = I.generate(w)
    ref, raux = H.oracle_chain(w, t)
    got, gaux, written = _call(w, t, False, FLAG_256 | B.FLAG_TEST_EXPIRE_WAIT)
    H.check(w, got, gaux, ref, raux, "shared")
    assert written >= 74 * 2 * TILE_BYTES


def test_without_the_room_and_under_capture():
    """A workspace that holds the statistics alone, and a captured stream, run without sharing."""
    w = _workload(I.BF16, 300, 4104, 1400, I.ACT_SILU, I.NORM_RMSNORM)
    t = I.generate_gated(w)
    d = {k: H.to_device(v) for k, v in t.items()}
    ref, _ = _reference(w, t, True)
    got, _, _ = _call(w, t, True, ws_bytes=1 << 17)
    H.check(w, got, None, ref, None, "small workspace")
    out = torch.full((w.M, w.N), float("nan"), dtype=torch.bfloat16, device="cuda")
    p = B.make_params(d["X"], d["W"], out, alpha=w.alpha, post_scale=w.post_scale, eps=w.eps, gamma=d["gamma"], beta=d["beta"])
    n = B.fge_gated_workspace_bytes(True, w.act, w.norm, p)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    p.workspace, p.workspace_bytes = ws.data_ptr(), n
    call = lambda: B.fused_gated_gemm_epilogue(d["X"], d["W"], d["W2"], d["b"], d["b2"], w.act, w.norm, p, out)
    call()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    for _ in range(3):
        out.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        H.check(w, H.to_host_f64(out), None, ref, None, "replay")
        call()
        torch.cuda.synchronize()
        H.check(w, H.to_host_f64(out), None, ref, None, "eager")
