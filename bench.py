#!/usr/bin/env python3
"""Benchmark of the fused GEMM + activation + row-normalisation path on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload cfg3] [--no-others] [--no-cpu]

A step is one call of fused_gemm_epilogue (every kernel of the fused path) on one batch of the
workload's seeded synthetic inputs, already resident in HBM.  The headline workload is the
largest MFMA-bound one (cfg3: bf16 8192x4096x4096, SiLU, RMSNorm).

Timing protocol (every figure): W untimed warm-up calls, then the same call repeated for at
least 50 ms so that the chip has settled on the clock it sustains under this load, then
`--blocks` (default 5) blocks of exactly K calls, each block bracketed by a synchronise and a
pair of events on the launch stream.  `ms_per_step` is the MEDIAN block; the fastest and the
slowest block are reported next to it (`ms_per_step_blocks`).

The single JSON line printed on stdout carries, besides the headline throughput:

  roofline     - the dominant kernel (the fused tile kernel) timed with events recorded on the
                 launch stream around each of its launches, against the MFMA (or HBM) peak
  cpu_baseline - the float64 oracle timed on the host cores on a bounded sample of rows
  per_config   - fused / unfused times, TFLOP/s, GB/s, roofline fractions and the fused-over-
                 unfused speedup for all five workloads (geometric mean in `speedup_geomean`)

Everything else goes to stderr."""
import argparse
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_TFLOPS = {"bf16": 2500.0, "f32": 157.3, "f8": 5000.0}      # dense MFMA peaks of MI355X
PEAK_HBM_GBS = 8000.0
# which roof binds each workload's dominant kernel
BOUND = {"cfg1": "mfma", "cfg2": "mfma", "cfg3": "mfma", "cfg4": "mfma", "cfg5": "hbm", "cfg3_f8": "mfma"}
# Plain vector-ALU roof: 256 compute units x 64 lanes per clock x 2.4 GHz = 39.3e12 lane-
# operations per second (the 157.3 TFLOP/s fp32 vector peak counts a packed pair of fused
# multiply-adds, 4 FLOP, per lane and clock; the library is built without packed fp32).
PEAK_VALU_LANE_OPS = 256 * 64 * 2.4e9
# Vector-ALU lane-cycles per output element of a workload's fused kernel, from the shader-
# sequencer counters in profiles/sq_activity_<workload>.txt: SQ_ACTIVE_INST_VALU (busy time of the
# vector ALUs, in units of 4 cycles, a quarter-rate transcendental counting four times as long as
# an addition) x 4 cycles x 16 lanes per SIMD / output elements, minus the issue slots of the
# MFMAs.  None where no profile has been taken.
def valu_lane_cycles_per_element(workload: str):
    path = os.path.join(ROOT, "profiles", f"sq_activity_{workload}.txt")
    if not os.path.exists(path):
        return None
    rec = {}
    for ln in open(path):
        if ":" in ln and not ln.startswith("#"):
            k, v = ln.split(":", 1)
            rec[k.strip()] = v.strip().split()[0] if v.strip() else ""
    try:
        return float(rec["valu_lane_cycles_per_element"])
    except (KeyError, ValueError):
        return None


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def kernel_sources_digest() -> str:
    """SHA-256 over the HIP sources of the library, in name order."""
    import hashlib
    d = os.path.join(ROOT, "paper_2512_23424_amd", "csrc")
    h = hashlib.sha256()
    for name in sorted(os.listdir(d)):
        if name.endswith((".h", ".hip")):
            h.update(name.encode())
            h.update(open(os.path.join(d, name), "rb").read())
    return h.hexdigest()


def measured_traffic(workload: str):
    """HBM bytes per launch of the dominant kernel as the hardware counters saw them
    (profiles/hbm_traffic_<workload>.txt); None when there is no such record or the kernel
    sources have changed since it was taken."""
    path = os.path.join(ROOT, "profiles", f"hbm_traffic_{workload}.txt")
    if not os.path.exists(path):
        return None
    rec = {}
    for ln in open(path):
        if ":" in ln and not ln.startswith("#"):
            k, v = ln.split(":", 1)
            rec[k.strip()] = v.strip()
    if rec.get("kernel_sources_sha256") != kernel_sources_digest():
        return None
    try:
        return float(rec["hbm_bytes_per_launch"])
    except (KeyError, ValueError):
        return None


def gated_ffn(torch, B, I, timed, log):
    """SiLU-and-Mul followed by RMSNorm at cfg3's shape (bf16, two 8192x4096x4096 products):
    the gated tile kernel against the unfused sequence of the same library, with a parity check
    of sampled rows against the oracle."""
    from oracle import compare as C
    from oracle import oracle as O
    w = I.scaled(I.WORKLOADS["cfg3"], dist=dict(I.WORKLOADS["cfg3"].dist, W=("normal", 0.0, 1.0 / 64)))
    log("[bench] generating the gated workload ...")
    t = I.generate_gated(w)

    def up(a):
        return None if a is None else (torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
                                       if a.dtype == np.uint16 else torch.from_numpy(a).cuda())
    d = {k: up(v) for k, v in t.items()}
    sets = [(d["X"], torch.empty(w.M, w.N, dtype=torch.bfloat16, device="cuda")),
            (d["X"].clone(), torch.empty(w.M, w.N, dtype=torch.bfloat16, device="cuda"))]
    ps = []
    for X, out in sets:
        p = B.make_params(X, d["W"], out, eps=w.eps, gamma=d["gamma"])
        n = max(B.fge_gated_workspace_bytes(True, w.act, w.norm, p), B.fge_gated_workspace_bytes(False, w.act, w.norm, p))
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        p.workspace, p.workspace_bytes = ws.data_ptr(), n
        ps.append((p, ws))

    def fused(i):
        B.fused_gated_gemm_epilogue(sets[i][0], d["W"], d["W2"], None, None, w.act, w.norm, ps[i][0], sets[i][1])

    def unfused(i):
        B.unfused_gated_gemm_epilogue(sets[i][0], d["W"], d["W2"], None, None, w.act, w.norm, ps[i][0], sets[i][1])
    rows = np.unique(np.concatenate([[0, w.M - 1], np.random.default_rng(4).integers(0, w.M, 6)]))
    sets[0][1].fill_(float("nan"))
    fused(0)
    torch.cuda.synchronize()
    got = sets[0][1][torch.from_numpy(rows).cuda()].to(torch.float64).cpu().numpy()
    f = {k: I.as_f64(v) for k, v in t.items()}
    ref, _ = O.gated_chain(f["X"][rows], f["W"], f["W2"], None, None, f["gamma"], None, act=w.act, norm=w.norm, eps=w.eps)
    err = C.max_rel_err(got, ref)
    if not (err <= 2e-2):
        raise SystemExit(f"bench.py: gated result off the oracle: {err:.3e}")
    tf_ = timed(fused, 50, 10)
    tu_ = timed(unfused, 25, 5)
    flops = 4.0 * w.M * w.N * w.K
    r = {"workload": "SiLU-and-Mul + RMSNorm, bf16, M=8192 K=4096 N=4096 (two products)",
         "tile": B.fge_gated_tile_name(w.act, w.norm, ps[0][0]), "ms_fused": round(tf_, 5),
         "ms_unfused": round(tu_, 5), "tflops": round(flops / (tf_ * 1e-3) / 1e12, 2),
         "frac_mfma": round(flops / (tf_ * 1e-3) / 1e12 / PEAK_TFLOPS["bf16"], 4),
         "speedup_vs_unfused": round(tu_ / tf_, 3), "parity_err": float(f"{err:.3e}")}
    log(f"[bench] gated: {json.dumps(r)}")
    return r


def row_ops(torch, B, I, timed, log):
    """The standalone row operations (fge_row_op: one kernel, one read and one write of the
    matrix) on large matrices, against the HBM roofline; two rotating buffer sets."""
    res = []
    for M, N, dt, norm, name in ((65536, 4096, torch.bfloat16, I.NORM_RMSNORM, "rmsnorm bf16"),
                                 (65536, 8192, torch.bfloat16, I.NORM_SOFTMAX, "softmax bf16"),
                                 (65536, 4096, torch.float32, I.NORM_LAYERNORM, "layernorm fp32"),
                                 (262144, 512, torch.float32, I.NORM_LOGSUMEXP, "logsumexp fp32"),
                                 (8192, 32000, torch.bfloat16, I.NORM_SOFTMAX, "softmax bf16, 32000 columns")):
        A = [torch.randn(M, N, device="cuda").to(dt) for _ in range(2)]
        out = [torch.empty(M, N, device="cuda", dtype=dt) for _ in range(2)]
        g, be, aux = torch.ones(N, device="cuda"), torch.zeros(N, device="cuda"), torch.empty(M, device="cuda")
        ps = [B.make_params(None, None, out[i], eps=1e-6, gamma=g, beta=be, aux_out=aux) for i in range(2)]
        ms = timed(lambda i: B.fge_row_op(A[i], norm, ps[i], out[i]), 20, 4)
        nbytes = 2 * M * N * A[0].element_size()
        res.append({"op": name, "rows": M, "cols": N, "ms": round(ms, 5), "gbs": round(nbytes / (ms * 1e-3) / 1e9, 1),
                    "frac_hbm": round(nbytes / (ms * 1e-3) / 1e9 / PEAK_HBM_GBS, 4)})
        del A, out
        torch.cuda.empty_cache()
    log(f"[bench] row operations: {json.dumps(res)}")
    return res


def fp8_operands(torch, B, I, timed, log):
    """cfg3's chain and shape with 8-bit E4M3 operands (bf16 out): fused against the unfused
    sequence of the same library, parity of sampled rows against the oracle on the same bytes."""
    from oracle import compare as C
    from oracle import oracle as O
    w = I.EXTRA_WORKLOADS["cfg3_f8"]
    log("[bench] generating the 8-bit workload ...")
    t = I.generate(w)
    W = torch.from_numpy(t["W"]).cuda().view(torch.float8_e4m3fn)
    X = torch.from_numpy(t["X"]).cuda().view(torch.float8_e4m3fn)
    gamma = torch.from_numpy(t["gamma"]).cuda()
    sets = [(X, torch.empty(w.M, w.N, dtype=torch.bfloat16, device="cuda")),
            (X.clone(), torch.empty(w.M, w.N, dtype=torch.bfloat16, device="cuda"))]
    ps = []
    for Xs, out in sets:
        p = B.make_params(Xs, W, out, alpha=w.alpha, eps=w.eps, gamma=gamma)
        n = max(B.fge_workspace_bytes(True, w.act, w.norm, p), B.fge_workspace_bytes(False, w.act, w.norm, p), 16)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        p.workspace, p.workspace_bytes = ws.data_ptr(), n
        ps.append((p, ws))

    def fused(i):
        B.fused_gemm_epilogue(sets[i][0], W, None, w.act, w.norm, ps[i][0], sets[i][1])

    def unfused(i):
        B.unfused_gemm_epilogue(sets[i][0], W, None, w.act, w.norm, ps[i][0], sets[i][1])
    rows = np.unique(np.concatenate([[0, w.M - 1], np.random.default_rng(5).integers(0, w.M, 6)]))
    sets[0][1].fill_(float("nan"))
    fused(0)
    torch.cuda.synchronize()
    got = sets[0][1][torch.from_numpy(rows).cuda()].to(torch.float64).cpu().numpy()
    ref, _ = O.chain(I.as_f64(t["X"][rows]), I.as_f64(t["W"]), None, I.as_f64(t["gamma"]), None, alpha=w.alpha,
                     act=w.act, norm=w.norm, eps=w.eps)
    err = C.max_rel_err(got, ref)
    if not (err <= 2e-2):
        raise SystemExit(f"bench.py: 8-bit result off the oracle: {err:.3e}")
    tf_ = timed(fused, 50, 10)
    tu_ = timed(unfused, 25, 5)
    r = {"workload": "cfg3's chain, E4M3 operands, bf16 out, M=8192 K=4096 N=4096",
         "tile": B.fge_tile_name(True, w.act, w.norm, ps[0][0]), "ms_fused": round(tf_, 5),
         "ms_unfused": round(tu_, 5), "tflops": round(w.flops / (tf_ * 1e-3) / 1e12, 2),
         "frac_mfma": round(w.flops / (tf_ * 1e-3) / 1e12 / PEAK_TFLOPS["f8"], 4),
         "speedup_vs_unfused": round(tu_ / tf_, 3), "parity_err": float(f"{err:.3e}")}
    log(f"[bench] 8-bit operands: {json.dumps(r)}")
    return r


def few_rows(torch, B, I, timed, log):
    """A decode-like problem (16 rows, K = N = 4096, bf16, cfg3's chain): bound by reading W once.
    The fused call cuts K into slices; timed against the same call without the slices and
    against the unfused sequence, checked against the oracle on every row."""
    from oracle import compare as C
    from oracle import oracle as O
    w = I.scaled(I.WORKLOADS["cfg3"], M=16, K=4096, N=4096)
    t = I.generate(w)
    W = [torch.from_numpy(t["W"].view(np.int16)).cuda().view(torch.bfloat16) for _ in range(2)]
    X = torch.from_numpy(t["X"].view(np.int16)).cuda().view(torch.bfloat16)
    gamma = torch.from_numpy(t["gamma"]).cuda()
    out = torch.empty(w.M, w.N, dtype=torch.bfloat16, device="cuda")
    ps = {}
    for name, flags in (("sliced", 0), ("whole", B.FLAG_NO_SPLIT_K)):
        p = B.make_params(X, W[0], out, eps=w.eps, gamma=gamma, flags=flags)
        n = max(B.fge_workspace_bytes(True, w.act, w.norm, p), B.fge_workspace_bytes(False, w.act, w.norm, p), 16)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        p.workspace, p.workspace_bytes = ws.data_ptr(), n
        ps[name] = (p, ws)
    out.fill_(float("nan"))
    B.fused_gemm_epilogue(X, W[0], None, w.act, w.norm, ps["sliced"][0], out)
    torch.cuda.synchronize()
    ref, _ = O.chain(I.as_f64(t["X"]), I.as_f64(t["W"]), None, I.as_f64(t["gamma"]), None, act=w.act, norm=w.norm, eps=w.eps)
    err = C.max_rel_err(out.to(torch.float64).cpu().numpy(), ref)
    if not (err <= 2e-2):
        raise SystemExit(f"bench.py: few-rows result off the oracle: {err:.3e}")
    ts = timed(lambda i: B.fused_gemm_epilogue(X, W[i], None, w.act, w.norm, ps["sliced"][0], out), 200, 20)
    tw = timed(lambda i: B.fused_gemm_epilogue(X, W[i], None, w.act, w.norm, ps["whole"][0], out), 200, 20)
    tu = timed(lambda i: B.unfused_gemm_epilogue(X, W[i], None, w.act, w.norm, ps["whole"][0], out), 200, 20)
    r = {"workload": "cfg3's chain, bf16, M=16 K=4096 N=4096", "kernel": "few_rows" if B.fge_few_rows(False, w.act, w.norm, ps["sliced"][0]) else "k_slices",
         "ms_fused": round(ts, 5), "ms_fused_whole_k": round(tw, 5), "ms_unfused": round(tu, 5),
         "gbs": round(w.algorithmic_bytes / (ts * 1e-3) / 1e9, 1),
         "frac_hbm": round(w.algorithmic_bytes / (ts * 1e-3) / 1e9 / PEAK_HBM_GBS, 4),
         "speedup_vs_unfused": round(tu / ts, 3), "parity_err": float(f"{err:.3e}")}
    log(f"[bench] few rows: {json.dumps(r)}")
    return r


def odd_extents(torch, B, I, timed, log):
    """The headline chain on extents off the 16-byte grid: 4097 x 4095 x 4099 (bf16, dense rows, so
    every row of X, W and out starts at an odd element).  The fused call repacks the operands
    into zero-padded buffers, runs the tile kernels and lets the element-granular row kernel write
    the result; against the same chain at the next shape on the grid, 4104 x 4096 x 4104 (the same
    17 x 17 tiles of 256 x 256: the cost of the odd extents alone), at 4096^3 (16 x 16 tiles, one
    round of the chip instead of two: what the one row and three columns past the tile boundary
    cost) and against the element-granular product (what such a shape ran on before; two steps
    only, it is slow)."""
    from oracle import compare as C
    from oracle import oracle as O
    res = {}
    for name, (M, K, N) in (("odd", (4097, 4095, 4099)), ("aligned", (4104, 4096, 4104)), ("cube", (4096, 4096, 4096))):
        w = I.scaled(I.WORKLOADS["cfg3"], M=M, K=K, N=N, dist=dict(I.WORKLOADS["cfg3"].dist, W=("normal", 0.0, 1.0 / 64)))
        t = I.generate(w)
        X = torch.from_numpy(t["X"].view(np.int16)).cuda().view(torch.bfloat16)
        W = torch.from_numpy(t["W"].view(np.int16)).cuda().view(torch.bfloat16)
        gamma = torch.from_numpy(t["gamma"]).cuda()
        out = torch.empty(M, N, dtype=torch.bfloat16, device="cuda")
        p = B.make_params(X, W, out, eps=w.eps, gamma=gamma)
        n = max(B.fge_workspace_bytes(True, w.act, w.norm, p), 16)
        ws = torch.empty(n, dtype=torch.uint8, device="cuda")
        p.workspace, p.workspace_bytes = ws.data_ptr(), n
        out.fill_(float("nan"))
        B.fused_gemm_epilogue(X, W, None, w.act, w.norm, p, out)
        torch.cuda.synchronize()
        rows = np.unique(np.concatenate([[0, M - 1], np.random.default_rng(8).integers(0, M, 6)]))
        ref, _ = O.chain(I.as_f64(t["X"][rows]), I.as_f64(t["W"]), None, I.as_f64(t["gamma"]), None, act=w.act, norm=w.norm, eps=w.eps)
        err = C.max_rel_err(out[torch.from_numpy(rows).cuda()].to(torch.float64).cpu().numpy(), ref)
        if not (err <= 2e-2):
            raise SystemExit(f"bench.py: odd-extents result ({name}) off the oracle: {err:.3e}")
        res[name] = {"tile": B.fge_tile_name(True, w.act, w.norm, p), "parity_err": float(f"{err:.3e}"),
                     "ms": round(timed(lambda i: B.fused_gemm_epilogue(X, W, None, w.act, w.norm, p, out), 20, 5), 5)}
        if name == "odd":           # the element-granular path: a workspace that only holds its fp32 rows
            q = B.make_params(X, W, out, eps=w.eps, gamma=gamma)
            q.workspace, q.workspace_bytes = ws.data_ptr(), (M * N * 4 + 255) // 256 * 256
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            B.fused_gemm_epilogue(X, W, None, w.act, w.norm, q, out)
            torch.cuda.synchronize()
            e0.record()
            for _ in range(2):
                B.fused_gemm_epilogue(X, W, None, w.act, w.norm, q, out)
            e1.record()
            torch.cuda.synchronize()
            res[name]["ms_element_granular"] = round(e0.elapsed_time(e1) / 2, 4)
        del X, W, out, ws
        torch.cuda.empty_cache()
    r = {"workload": "cfg3's chain, bf16, M=4097 K=4095 N=4099 (dense rows)", "path": res["odd"]["tile"],
         "ms_fused": res["odd"]["ms"], "ms_fused_4104x4096x4104": res["aligned"]["ms"],
         "ratio_to_aligned": round(res["odd"]["ms"] / res["aligned"]["ms"], 3), "ms_fused_4096_cubed": res["cube"]["ms"],
         "ms_element_granular": res["odd"]["ms_element_granular"],
         "tflops": round(2.0 * 4097 * 4095 * 4099 / (res["odd"]["ms"] * 1e-3) / 1e12, 2), "parity_err": res["odd"]["parity_err"]}
    log(f"[bench] odd extents: {json.dumps(r)}")
    return r


def wide_rows(torch, B, I, timed, log):
    """Rows wider than a wave's registers hold: 2048 x 4096 x 32000 (bf16), logits with a row
    softmax and with a row logsumexp (out = the logits, aux = lse) - the rows are split over 125
    column tiles and finished by the second pass.  Against the unfused sequence; sampled rows
    against the oracle."""
    from oracle import compare as C
    from oracle import oracle as O
    res = []
    for norm, label in ((I.NORM_SOFTMAX, "softmax"), (I.NORM_LOGSUMEXP, "logsumexp")):
        w = I.scaled(I.WORKLOADS["cfg4"], M=2048, K=4096, N=32000, batch=1, act=I.ACT_NONE, norm=norm,
                     alpha=1.0, dist=dict(I.WORKLOADS["cfg4"].dist, W=("normal", 0.0, 1.0 / 64)))
        t = I.generate(w)
        X = torch.from_numpy(t["X"].view(np.int16)).cuda().view(torch.bfloat16)
        W = torch.from_numpy(t["W"].view(np.int16)).cuda().view(torch.bfloat16)
        b = torch.from_numpy(t["b"]).cuda()
        out = [torch.empty(w.M, w.N, dtype=torch.bfloat16, device="cuda") for _ in range(2)]
        aux = torch.empty(w.M, device="cuda")
        ps = []
        for o in out:
            p = B.make_params(X, W, o, aux_out=aux)
            n = max(B.fge_workspace_bytes(True, w.act, w.norm, p), B.fge_workspace_bytes(False, w.act, w.norm, p), 16)
            ws = torch.empty(n, dtype=torch.uint8, device="cuda")
            p.workspace, p.workspace_bytes = ws.data_ptr(), n
            ps.append((p, ws))
        rows = np.unique(np.concatenate([[0, w.M - 1], np.random.default_rng(6).integers(0, w.M, 6)]))
        out[0].fill_(float("nan")); aux.fill_(float("nan"))
        B.fused_gemm_epilogue(X, W, b, w.act, w.norm, ps[0][0], out[0])
        torch.cuda.synchronize()
        idx = torch.from_numpy(rows).cuda()
        ref, raux = O.chain(I.as_f64(t["X"][rows]), I.as_f64(t["W"]), I.as_f64(t["b"]), None, None, act=w.act, norm=w.norm)
        err = C.max_rel_err(out[0][idx].to(torch.float64).cpu().numpy(), ref)
        if norm == I.NORM_LOGSUMEXP:
            err = max(err, C.max_rel_err_vec(aux[idx].to(torch.float64).cpu().numpy(), raux))
        if not (err <= 2e-2):
            raise SystemExit(f"bench.py: wide-rows result off the oracle: {err:.3e}")
        # (the device has idled through the oracle's rows: a longer warm-up brings the clocks back)
        tf_ = timed(lambda i: B.fused_gemm_epilogue(X, W, b, w.act, w.norm, ps[i][0], out[i]), 20, 20)
        tu_ = timed(lambda i: B.unfused_gemm_epilogue(X, W, b, w.act, w.norm, ps[i][0], out[i]), 20, 20)
        res.append({"workload": f"logits + row {label}, bf16, M=2048 K=4096 N=32000",
                    "tile": B.fge_tile_name(True, w.act, w.norm, ps[0][0]), "ms_fused": round(tf_, 5),
                    "ms_unfused": round(tu_, 5), "tflops": round(w.flops / (tf_ * 1e-3) / 1e12, 2),
                    "frac_mfma": round(w.flops / (tf_ * 1e-3) / 1e12 / PEAK_TFLOPS["bf16"], 4),
                    "speedup_vs_unfused": round(tu_ / tf_, 3), "parity_err": float(f"{err:.3e}")})
        del out, ps
        torch.cuda.empty_cache()
    log(f"[bench] wide rows: {json.dumps(res)}")
    return res


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=10)
    ap.add_argument("--workload", default="cfg3")
    ap.add_argument("--no-others", action="store_true", help="skip the per-config table")
    ap.add_argument("--no-cpu", action="store_true", help="skip the oracle timing")
    ap.add_argument("--blocks", type=int, default=5, help="timed blocks of --steps calls; the median is reported")
    ap.add_argument("--precondition-ms", type=float, default=50.0,
                    help="run the timed call for at least this long before the first timed block")
    ap.add_argument("--only-fused", action="store_true",
                    help="run a known-size copy, then just the fused steps (for profiler runs)")
    ap.add_argument("--sources-digest", action="store_true",
                    help="print the digest of the kernel sources that traffic records are tied to")
    args = ap.parse_args()
    if args.sources_digest:
        print(kernel_sources_digest())
        return 0
    if args.gpus != 1:
        log("bench.py: the library runs on ONE GPU; the path shards over rows without any exchange, "
            "but no multi-GPU launch is provided.  Use --gpus 1.")
        return 2

    import torch
    from paper_2512_23424_amd import binding as B
    from paper_2512_23424_amd import inputs as I
    if not torch.cuda.is_available():
        log("bench.py: no GPU visible")
        return 3
    B.lib()                                        # fail loudly if the HIP library is missing
    torch.cuda.set_device(0)

    def tdtype(code):
        return torch.bfloat16 if code == I.BF16 else torch.float32

    def upload(a):
        if a is None:
            return None
        if a.dtype == np.uint16:
            return torch.from_numpy(a.view(np.int16)).cuda().view(torch.bfloat16)
        if a.dtype == np.uint8:
            return torch.from_numpy(a).cuda().view(torch.float8_e4m3fn)
        return torch.from_numpy(a).cuda()

    def dtname(w):
        return {I.BF16: "bf16", I.F8E4M3: "f8"}.get(w.in_dtype, "f32")

    class Case:
        """Device-resident inputs (two rotating X / out sets so consecutive steps do not find
        their operands in the 256 MB last-level cache) and prepared parameter blocks."""

        def __init__(self, w):
            self.w = w
            t = I.generate(w)
            self.host = t
            self.W, self.b = upload(t["W"]), upload(t["b"])
            self.gamma, self.beta = upload(t["gamma"]), upload(t["beta"])
            X = upload(t["X"])
            self.sets = []
            for s in range(2):
                Xs = X if s == 0 else X.clone()
                if w.batch > 1:
                    Xs = Xs.view(w.batch, w.M, w.K)
                    out = torch.empty(w.batch, w.M, w.N, dtype=tdtype(w.out_dtype), device="cuda")
                else:
                    out = torch.empty(w.rows, w.N, dtype=tdtype(w.out_dtype), device="cuda")
                aux = (torch.empty(w.rows, dtype=torch.float32, device="cuda")
                       if w.norm == I.NORM_LOGSUMEXP else None)
                self.sets.append((Xs, out, aux))
            p0 = self.params(0, None)
            nf = B.fge_workspace_bytes(True, w.act, w.norm, p0)
            nu = B.fge_workspace_bytes(False, w.act, w.norm, p0)
            self.ws = torch.zeros(max(nf, nu, 16), dtype=torch.uint8, device="cuda")    # (zeros: the fault word starts cleared)
            self.p = [self.params(s, self.ws) for s in range(2)]
            self.tile = B.fge_tile_name(True, w.act, w.norm, p0)
            # what fused_gemm_epilogue runs: one kernel (whole rows, or split rows finished by
            # the tiles themselves), or the tile kernel plus the light second pass
            self.one_kernel = (B.fge_fault_word_offset(w.act, w.norm, p0) is not None
                               or not B.fge_fused_needs_finish(w.act, w.norm, p0))
            self.two_pass = not self.one_kernel

        def params(self, s, ws):
            w = self.w
            Xs, out, aux = self.sets[s]
            return B.make_params(Xs, self.W, out, alpha=w.alpha, post_scale=w.post_scale,
                                 clamp_lo=w.clamp_lo, clamp_hi=w.clamp_hi, eps=w.eps,
                                 gamma=self.gamma, beta=self.beta, aux_out=aux, workspace=ws)

        def fused(self, s):
            Xs, out, _ = self.sets[s]
            B.fused_gemm_epilogue(Xs, self.W, self.b, self.w.act, self.w.norm, self.p[s], out)

        def fault_word(self):
            """The int32 in the workspace that a one-kernel launch raises when a wait between its
            workgroups runs out (None for the other forms).  The unfused sequence keeps its
            intermediates in the same workspace, so the word is cleared before fused calls are
            timed and read after them."""
            off = B.fge_fault_word_offset(self.w.act, self.w.norm, self.p[0])
            return None if off is None else self.ws[off:off + 4].view(torch.int32)

        def unfused(self, s):
            Xs, out, _ = self.sets[s]
            B.unfused_gemm_epilogue(Xs, self.W, self.b, self.w.act, self.w.norm, self.p[s], out)

        def fused_stages(self, s, e0, e1):
            Xs, out, _ = self.sets[s]
            e0.record()
            if self.one_kernel:
                B.fused_gemm_epilogue(Xs, self.W, self.b, self.w.act, self.w.norm, self.p[s], out)
                e1.record()
            else:
                B.fge_fused_tiles(Xs, self.W, self.b, self.w.act, self.w.norm, self.p[s], out)
                e1.record()
                B.fge_fused_finish(self.w.act, self.w.norm, self.p[s], out)

    def timed_blocks(fn, steps, warmup, blocks=None, pre_ms=None):
        """ms per step of each of `blocks` blocks of exactly `steps` calls (see the module text)."""
        blocks = args.blocks if blocks is None else blocks
        pre_ms = args.precondition_ms if pre_ms is None else pre_ms
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for i in range(warmup):
            fn(i & 1)
        torch.cuda.synchronize()
        if pre_ms > 0:
            e0.record()
            fn(0)
            e1.record()
            torch.cuda.synchronize()
            one = max(e0.elapsed_time(e1), 1e-3)
            for i in range(min(20000, int(pre_ms / one) + 1)):
                fn(i & 1)
        out = []
        for _ in range(max(1, blocks)):
            torch.cuda.synchronize()
            e0.record()
            for i in range(steps):
                fn(i & 1)
            e1.record()
            torch.cuda.synchronize()
            out.append(e0.elapsed_time(e1) / steps)
        return out

    def timed(fn, steps, warmup):
        return float(np.median(timed_blocks(fn, steps, warmup)))          # ms per step, median block

    def fused_blocks_checked(case, steps, warmup):
        """timed_blocks of the case's fused call; stops if a one-kernel launch reported a wait
        that ran out."""
        word = case.fault_word()
        if word is not None:
            word.zero_()
        blocks = timed_blocks(case.fused, steps, warmup)
        if word is not None and int(word[0]) != 0:
            raise SystemExit(f"bench.py: {case.w.name}: a wait between workgroups ran out (fault word set)")
        return blocks

    def graphed(fn, calls=100, replays=10):
        """ms per step with the launches recorded once into a HIP graph and replayed: what a
        launch-bound step costs once the host is out of the loop (kernels only, no memsets)."""
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            for i in range(calls):
                fn(i & 1)
        g.replay()
        torch.cuda.synchronize()
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(replays):
            g.replay()
        e1.record()
        torch.cuda.synchronize()
        return e0.elapsed_time(e1) / (calls * replays)

    def kernel_time(case, steps):
        """Average duration of the fused tile kernel: events recorded on the launch stream
        (torch's current stream, the one the library is given) around each launch."""
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
              for _ in range(steps)]
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(ev):
            case.fused_stages(i & 1, a, b)
        torch.cuda.synchronize()
        return sum(a.elapsed_time(b) for a, b in ev) / steps

    def parity(case, nrows=8):
        """Poisoned-output run checked on sampled complete rows against the oracle."""
        from oracle import compare as C
        from oracle import oracle as O
        w = case.w
        rows = np.unique(np.concatenate([[0, w.rows - 1],
                                         np.random.default_rng(3).integers(0, w.rows, nrows)]))
        Xs, out, aux = case.sets[0]
        out.fill_(float("nan"))
        case.fused(0)
        torch.cuda.synchronize()
        got = out.reshape(w.rows, w.N)[torch.from_numpy(rows).cuda()].to(torch.float64).cpu().numpy()
        f = {k: I.as_f64(v) for k, v in case.host.items()}
        ref, raux = O.chain(f["X"][rows], f["W"], f["b"], f["gamma"], f["beta"], alpha=w.alpha,
                            post_scale=w.post_scale, act=w.act, clamp_lo=w.clamp_lo,
                            clamp_hi=w.clamp_hi, norm=w.norm, eps=w.eps)
        err = C.max_rel_err(got, ref)
        tol = 2e-2 if w.in_dtype in (I.BF16, I.F8E4M3) else 1e-4
        if not (err <= tol):
            raise SystemExit(f"bench.py: {w.name} fused result off the oracle: {err:.3e} > {tol}")
        return err

    def report(case, t_fused, t_unfused, t_kernel):
        w = case.w
        dt = dtname(w)
        tf = w.flops / (t_fused * 1e-3) / 1e12
        gbs = w.algorithmic_bytes / (t_fused * 1e-3) / 1e9
        r = {"tile": case.tile, "kernels_fused": 2 if case.two_pass else 1,
             "ms_fused": round(t_fused, 5), "tflops": round(tf, 2), "gbs": round(gbs, 1),
             "frac_hbm": round(gbs / PEAK_HBM_GBS, 4)}
        if dt == "f32" and "splitbf16" in case.tile:
            # fp32 operands multiplied as three bf16 products on the bf16 matrix pipe: the roof
            # for useful FLOPs is a third of that pipe's peak
            r["frac_mfma"] = round(tf / (PEAK_TFLOPS["bf16"] / 3.0), 4)
            r["mfma_roof"] = "bf16 pipe / 3 (split product)"
        else:
            r["frac_mfma"] = round(tf / PEAK_TFLOPS[dt], 4)
        # plain vector-ALU roof (the activation and row-op arithmetic), where the kernel's lane-
        # cycles per element have been counted
        lc = valu_lane_cycles_per_element(w.name)
        if lc is not None:
            lane_ops = lc * w.rows * w.N
            r["frac_valu"] = round(lane_ops / (t_fused * 1e-3) / PEAK_VALU_LANE_OPS, 4)
            r["valu_lane_cycles_per_element"] = lc
        fr = {k: r[k] for k in ("frac_mfma", "frac_hbm", "frac_valu") if k in r}
        r["binding_roof"] = max(fr, key=fr.get)[5:]
        if t_unfused is not None:
            r["ms_unfused"] = round(t_unfused, 5)
            r["speedup_vs_unfused"] = round(t_unfused / t_fused, 3)
        if t_kernel is not None:
            r["ms_tile_kernel"] = round(t_kernel, 5)
        return r

    # ------------------------------------------------------------------ headline workload
    w = I.WORKLOADS[args.workload] if args.workload in I.WORKLOADS else I.EXTRA_WORKLOADS[args.workload]
    log(f"[bench] generating {w.name} ...")
    case = Case(w)
    err = parity(case)
    log(f"[bench] {w.name}: tile {case.tile}, parity on sampled rows {err:.2e}")
    if args.only_fused:
        # a plain copy of known size first (the library's elementwise kernel with the identity
        # activation: reads and writes 128 MiB each): hardware counters of the run are scaled by
        # what they read for it
        src = torch.zeros(8192, 4096, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        pc = B.make_params(None, None, dst)
        for _ in range(5):
            B.fge_activation(src, 0, pc, dst)
        torch.cuda.synchronize()
        t_fused = float(np.median(fused_blocks_checked(case, args.steps, args.warmup)))
        log(f"[bench] fused {t_fused:.4f} ms/step")
        return 0
    fused_blocks = fused_blocks_checked(case, args.steps, args.warmup)
    t_fused = float(np.median(fused_blocks))
    # The dominant kernel's average launch duration.  When the fused path is that one kernel, the
    # events around the timed region measure exactly it, under the same sustained load (the chip
    # lowers its clock a few milliseconds into a run of back-to-back launches; launches timed one
    # by one with idle gaps between them come out about 10 % shorter).
    t_kernel_gaps = kernel_time(case, args.steps)
    t_kernel = t_kernel_gaps if case.two_pass else t_fused
    t_unfused = timed(case.unfused, max(5, args.steps // 2), 3)
    head = report(case, t_fused, t_unfused, t_kernel_gaps)
    log(f"[bench] {w.name}: {json.dumps(head)}")

    dt = dtname(w)
    if BOUND[w.name] == "hbm":
        achieved = w.algorithmic_bytes / (t_kernel * 1e-3) / 1e9
        roof = {"bound": "hbm", "achieved": round(achieved, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                "frac": round(achieved / PEAK_HBM_GBS, 4), "traffic": None}
    else:
        achieved = w.flops / (t_kernel * 1e-3) / 1e12
        roof = {"bound": "mfma", "achieved": round(achieved, 2), "peak": PEAK_TFLOPS[dt],
                "unit": "TFLOP/s", "frac": round(achieved / PEAK_TFLOPS[dt], 4), "traffic": None}
    roof["traffic"] = measured_traffic(w.name)
    roof["kernel"] = f"tile_kernel<{dt}> {case.tile}"
    roof["kernel_ms"] = round(t_kernel, 5)
    roof["kernel_ms_single_launches"] = round(t_kernel_gaps, 5)

    # ------------------------------------------------------------------ CPU baseline (oracle)
    cpu = None
    if not args.no_cpu:
        from oracle import oracle as O
        f = {k: I.as_f64(v) for k, v in case.host.items()}

        def run_rows(n):
            t0 = time.perf_counter()
            O.chain(f["X"][:n], f["W"], f["b"], f["gamma"], f["beta"], alpha=w.alpha,
                    post_scale=w.post_scale, act=w.act, clamp_lo=w.clamp_lo, clamp_hi=w.clamp_hi,
                    norm=w.norm, eps=w.eps)
            return time.perf_counter() - t0
        threads = O.threads()
        probe = max(threads, 8)
        t_probe = run_rows(probe)
        n = int(min(w.rows, max(probe, probe * 12.0 / max(t_probe, 1e-6))))   # about 12 s of work
        n -= n % threads or 0
        n = max(n, threads)
        t_cpu = run_rows(n)
        cpu = {"value": round(2.0 * n * w.N * w.K / t_cpu / 1e12, 6), "unit": "TFLOP/s",
               "cores": threads, "kind": "oracle",
               "sample": f"first {n} of {w.rows} rows of {w.name}, all {w.N} columns, {t_cpu:.2f} s"}
        log(f"[bench] oracle: {json.dumps(cpu)}")
    del case
    torch.cuda.empty_cache()

    # ------------------------------------------------------------------ the other workloads
    per = {w.name: head}
    if not args.no_others:
        for name in ("cfg1", "cfg2", "cfg3", "cfg4", "cfg5"):
            if name == w.name:
                continue
            wl = I.WORKLOADS[name]
            log(f"[bench] generating {name} ...")
            c = Case(wl)
            e = parity(c)
            steps = 1000 if name == "cfg1" else 50
            tf_ = float(np.median(fused_blocks_checked(c, steps, 10)))
            tk_ = kernel_time(c, min(steps, 50))
            tu_ = timed(c.unfused, steps if name == "cfg1" else 25, 5)
            per[name] = report(c, tf_, tu_, tk_)
            per[name]["parity_err"] = float(f"{e:.3e}")
            if name == "cfg1":                      # launch bound: the same steps replayed from a graph
                gf, gu = graphed(c.fused), graphed(c.unfused)
                per[name].update(ms_fused_graph=round(gf, 5), ms_unfused_graph=round(gu, 5),
                                 speedup_vs_unfused_graph=round(gu / gf, 3))
            log(f"[bench] {name}: {json.dumps(per[name])}")
            del c
            torch.cuda.empty_cache()
    sp = [v["speedup_vs_unfused"] for v in per.values() if "speedup_vs_unfused" in v]
    # ------------------------------------------------------------------ the gated form
    gated = None
    if not args.no_others:
        gated = gated_ffn(torch, B, I, timed, log)
    f8 = None if args.no_others else fp8_operands(torch, B, I, timed, log)
    rows = None if args.no_others else row_ops(torch, B, I, timed, log)
    few = None if args.no_others else few_rows(torch, B, I, timed, log)
    wide = None if args.no_others else wide_rows(torch, B, I, timed, log)
    odd = None if args.no_others else odd_extents(torch, B, I, timed, log)
    geo = math.exp(sum(math.log(s) for s in sp) / len(sp)) if sp else None

    line = {
        "metric": "fused GEMM+epilogue TFLOP/s (% MFMA or HBM roofline) and speedup vs unfused",
        "value": head["tflops"], "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": head["ms_fused"],
        "ms_per_step_blocks": {"n": len(fused_blocks), "min": round(min(fused_blocks), 5), "max": round(max(fused_blocks), 5),
                               "precondition_ms": args.precondition_ms},
        "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": dt, "data": "synthetic",
        "config": {"workload": f"{w.name}: M={w.rows} K={w.K} N={w.N}, "
                               f"{'bf16 in/out' if dt == 'bf16' else 'E4M3 in, bf16 out' if dt == 'f8' else 'fp32'}, fp32 accumulate, "
                               f"act={w.act} rowop={w.norm} (codes of include/fge.h)",
                   "tile": head["tile"], "speedup_vs_unfused": head.get("speedup_vs_unfused")},
        "roofline": roof, "cpu_baseline": cpu, "per_config": per, "gated_ffn": gated, "fp8_operands": f8, "row_ops": rows, "few_rows": few, "wide_rows": wide, "odd_extents": odd,
        "speedup_geomean": None if geo is None else round(geo, 3),
        "paper_context": "paper reports 1.46x geomean over PyTorch eager (Triton, Ascend 910B, "
                         "KernelBench L1); no number for this chain",
    }
    print(json.dumps(line), flush=True)
    return 0


if __name__ == "__main__":
    sys.exit(main())
