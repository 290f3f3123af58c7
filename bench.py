"""Benchmark of the W4A4 DiT-linear hot path on one MI355X.

One step = the whole hot path over the four linears of a DiT block (qkv,
proj, fc1, fc2): for each linear, clq_rotate_quant_act on its fp16 input,
then clq_w4a4_linear against its offline-quantized weights.  Inputs and
weights are resident in HBM before timing starts; weights are quantized
once, outside the timed region (as the method does offline).

Default workload: the video DiT block, hidden 1152, MLP 4608, 16 latent
frames x 30 x 45 patches x batch 2 -> M = 43200 tokens, Hadamard block 64
(the largest per-layer shapes; rotate+quant's bandwidth-bound regime).
`--workload pixart_block` (M = 8192) and `flux_block` (width 3072, M = 4608,
block 128) time the other block configurations the same way.  `--codes fp6`
runs the same W4A4 step with the 4-bit codes stored as fp6 (e2m3) and the
GEMM on the fp6 matrix instruction (clq_rotate_quant_act_f6 /
clq_w4a4_linear_f6); its roofline is priced against the fp6 peak.

Prints ONE JSON line:
  value      effective TOPS of the step = sum(2 M N K) / step time, the step
             time from K back-to-back steps (no events between launches);
             step_ms_percentiles: median / p10 / p90 of single steps (HIP
             events at step boundaries, a separate pass)
  roofline   the GEMM kernel (dominant): algorithmic int8-MFMA ops per launch
             / average launch time (HIP events on the launch stream, in a
             pass of K steps after the timed one), against the dense int8
             peak (5.0 POP/s); traffic = HBM bytes per launch from the
             committed rocprofv3 FETCH_SIZE/WRITE_SIZE summary when it was
             taken on the current kernel source, else null
  rotate_quant  algorithmic bytes / launch time against HBM (8 TB/s), with
             the 256 MB Infinity Cache flushed by a 512 MB read before every
             launch (cold: the kernel's own rate), over the four launches;
             in_step_*: the same from the events pass, where each launch
             follows the previous linear's GEMM and its write-back
  clocks     graphics (SCLK) and memory (MCLK) clock and socket power
             sampled through amd-smi over 2.5 s of the same back-to-back
             steps right after the timed loop (its first second dropped:
             the readings trail the load)
  ceilings   measured ceilings beside the nominal peaks: a 1 GiB device copy
             (HBM) and the library's matrix-core probe loops (int8 MFMA on
             int4-shaped operands, and fp6 MFMA on the same codes as fp6; two
             workgroups per compute unit), with the clock and power during
             each probe; roofline.frac_of_measured_ceiling (against the probe
             of the instruction the GEMM issues) and
             rotate_quant.*_frac_of_copy_ceiling divide by them
  cpu_baseline  the CPU oracle timed on the host cores on a bounded sample
             of the same workload (token rows of every layer), plus one
             thread on a smaller sample
  extra      the other code storage on the same block, the PixArt block
             (M = 8192) with both, and the 28-block stack at 16384 tokens,
             timed the same way (context, not the headline)
"""
import argparse
import json
import math
import os
import sys
import threading
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import numpy as np  # noqa: E402

import workloads  # noqa: E402

INT8_PEAK_TOPS = 5000.0      # dense int8 MFMA, MI355X (5.0 POP/s)
FP6_PEAK_TOPS = 10100.0      # dense fp6 / fp4 MFMA, MI355X (10.1 PFLOP/s)
HBM_PEAK_GBPS = 8000.0       # HBM3E, MI355X
TRAFFIC_FILES = {
    ("video_block_m43200_h1152_b64", "int4"): os.path.join(ROOT, "profiles", "gemm_traffic_video_block_m43200.txt"),
    ("flux_block_m4608_h3072_b128", "int4"): os.path.join(ROOT, "profiles", "gemm_traffic_flux_block_m4608.txt"),
    ("video_block_m43200_h1152_b64", "fp6"): os.path.join(ROOT, "profiles", "gemm_f6_traffic_video_block_m43200.txt"),
}
BLOCKS = {"video_block": workloads.C4, "pixart_block": workloads.C2, "flux_block": workloads.C3}


def rq_bytes(l, abits=4, codes="int4"):
    """Algorithmic HBM bytes of one rotate+quant launch: read M*K fp16, write
    M*K/2 packed int4 codes (3*M*K/4 as fp6 codes, M*K int8 codes for 8-bit
    activations) and M fp32 scales."""
    out = (l.K // 2 if codes == "int4" else 3 * l.K // 4) if abits == 4 else l.K
    return l.M * (2 * l.K + out + 4)


def gemm_ops(l):
    return 2 * l.M * l.N * l.K


def rq_kernel_name(l, abits=4, codes="int4"):
    """The activation kernel the library runs for this layer: one or two
    8-column chunks per lane by the row length, one workgroup per row beyond
    16384 columns (code-width template argument 6: the 4-bit codes written as
    fp6)."""
    qb = 6 if (abits == 4 and codes == "fp6") else abits
    if l.K > 16384:
        return f"rotate_quant_wide_kernel<{l.block}, false, {qb}>"
    return f"rotate_quant_kernel<{l.block}, {qb}, false, {1 if l.K <= 8192 else 2}>"


def load_traffic(path, kernel_src_sha):
    """Per-launch HBM traffic from a committed rocprofv3 PMC summary, only if
    it was taken on the current kernel source."""
    if path is None or not os.path.exists(path):
        return None
    vals = {}
    for line in open(path):
        if line.startswith("traffic:"):
            for kv in line.split()[1:]:
                k, v = kv.split("=")
                vals[k] = v
    if vals.get("kernel_sha") != kernel_src_sha:
        return None
    return float(vals["bytes_per_launch"])


def kernel_sha(codes="int4"):
    """Hash of the GEMM kernels' sources (the kernels the traffic figures
    describe)."""
    import hashlib
    h = hashlib.sha256()
    for src in ("tile_gemm.h", "w4a4_gemm.hip" if codes == "int4" else "w4a4_f6.hip"):
        h.update(open(os.path.join(ROOT, "paper_2509_24416_amd", "csrc", src), "rb").read())
    return h.hexdigest()[:16]


def cpu_model():
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def blas_threads():
    """Threads of numpy's BLAS (the numpy oracles' matrix products), as the
    thread-pool library reports them; 1 if it cannot tell."""
    try:
        from threadpoolctl import threadpool_info
        n = [i.get("num_threads", 1) for i in threadpool_info() if i.get("user_api") == "blas"]
        return int(max(n)) if n else 1
    except Exception:
        return 1


class ClockSampler:
    """Samples the GPU's graphics and memory clocks and socket power through
    amd-smi in a background thread (every ~20 ms) while a timed region runs.
    Reports None where amd-smi is unavailable."""

    def __init__(self, torch, dev):
        self.samples = []
        self.handle = None
        self.err = None
        try:
            import amdsmi
            self.amdsmi = amdsmi
            amdsmi.amdsmi_init()
            handles = amdsmi.amdsmi_get_processor_handles()
            want = None
            try:
                p = torch.cuda.get_device_properties(dev)
                want = (int(getattr(p, "pci_domain_id", 0)), int(p.pci_bus_id), int(p.pci_device_id))
            except Exception:
                pass
            for h in handles:
                if want is None:
                    break
                bdf = amdsmi.amdsmi_get_gpu_device_bdf(h)   # "dddd:bb:dd.f"
                dom, bus, rest = bdf.split(":")
                if (int(dom, 16), int(bus, 16), int(rest.split(".")[0], 16)) == want:
                    self.handle = h
                    break
            if self.handle is None and len(handles) == 1:
                self.handle = handles[0]
        except Exception as e:   # no amd-smi: clocks are reported as null
            self.err = repr(e)
        self._stop = threading.Event()
        self._t = None
        self.t0 = time.perf_counter()

    def _read(self):
        a = self.amdsmi
        g = a.amdsmi_get_clock_info(self.handle, a.AmdSmiClkType.GFX)["clk"]
        m = a.amdsmi_get_clock_info(self.handle, a.AmdSmiClkType.MEM)["clk"]
        pw = None
        try:
            pi = a.amdsmi_get_power_info(self.handle)
            pw = pi.get("socket_power") or pi.get("current_socket_power") or pi.get("average_socket_power")
        except Exception:
            pass
        return g, m, pw

    def _loop(self):
        while not self._stop.is_set():
            try:
                self.samples.append((time.perf_counter(),) + tuple(self._read()))
            except Exception as e:
                self.err = repr(e)
                return
            time.sleep(0.02)

    def __enter__(self):
        self.t0 = time.perf_counter()
        if self.handle is not None:
            self._t = threading.Thread(target=self._loop, daemon=True)
            self._t.start()
        return self

    def __exit__(self, *exc):
        self._stop.set()
        if self._t is not None:
            self._t.join()

    def summary(self, settle_s=0.3):
        """Median / min / max over the samples taken after the first settle_s
        seconds of the sampled region (the readings trail the load)."""
        if not self.samples:
            return {"sclk_mhz": None, "mclk_mhz": None, "power_w": None, "samples": 0,
                    "note": self.err or "amd-smi handle not found"}
        a = np.array([[x if isinstance(x, (int, float)) else np.nan for x in s] for s in self.samples],
                     dtype=np.float64)
        keep = a[:, 0] >= self.t0 + settle_s
        if keep.sum() >= 3:
            a = a[keep]
        a = a[:, 1:]

        def stats(col):
            v = a[:, col]
            v = v[np.isfinite(v)]
            if v.size == 0:
                return None
            return {"median": float(np.median(v)), "min": float(v.min()), "max": float(v.max())}
        return {"sclk_mhz": stats(0), "mclk_mhz": stats(1), "power_w": stats(2), "samples": int(a.shape[0])}


def pct(v):
    v = np.asarray(v, np.float64)
    return {"median": round(float(np.median(v)), 5), "p10": round(float(np.percentile(v, 10)), 5),
            "p90": round(float(np.percentile(v, 90)), 5)}


def cpu_baseline(layers, inputs, budget_s=15.0, wbits=4, abits=4):
    """Times the CPU oracle's online path (rotate + quantize the activations,
    integer GEMM, fp64 epilogue) on a sample of token rows of every layer,
    sized to roughly budget_s seconds, on all the threads the oracle uses,
    then on one thread for a fifth of the budget; returns TOPS on those
    samples."""
    import oracle
    threads = oracle.get_threads()
    wq = {}
    for l in layers:  # offline step, not timed (as on the GPU)
        _, W, b = inputs[l.name]
        wq[l.name] = oracle.quantize_weights(W, l.block, bits=wbits)

    def run(rows):
        ops = 0
        t0 = time.perf_counter()
        for l in layers:
            X, _, b = inputs[l.name]
            _, xc, xs = oracle.quantize_act(X[:rows], l.block, bits=abits)
            _, wc, ws = wq[l.name]
            acc = oracle.gemm_i32(xc, wc)
            oracle.epilogue(acc, xs, ws, b)
            ops += 2 * rows * l.N * l.K
        return time.perf_counter() - t0, ops

    def sized(budget):
        t_cal, _ = run(32)
        rows = int(min(layers[0].M, max(32, 32 * budget / max(t_cal, 1e-3))))
        return max(16, rows // 16 * 16)

    rows = sized(budget_s)
    t, ops = run(rows)
    out = {"value": ops / t / 1e12, "unit": "TOPS", "cores": threads, "kind": "oracle",
           "cpu_model": cpu_model(),
           "sample": f"first {rows} token rows of each of the {len(layers)} linears "
                     f"({ops / 2e9:.1f} G MAC, {t:.1f} s; weights quantized beforehand, untimed)"}
    try:
        oracle.set_threads(1)
        rows1 = sized(budget_s / 5)
        t1, ops1 = run(rows1)
        out["single_thread"] = {"value": ops1 / t1 / 1e12, "unit": "TOPS", "cores": 1,
                                "sample": f"first {rows1} token rows of each linear ({t1:.1f} s)"}
    finally:
        oracle.set_threads(threads)
    return out


def bench_block(wl, args, clq, torch, dev, wbits=4, abits=4, steps=None, warmup=None, cold_reps=None,
                sample_clocks=True, clock_s=2.5, codes="int4"):
    """Times the hot path over the four linears of a DiT block workload
    (codes: "int4", or "fp6" for the W4A4 path with its codes stored as fp6).
    Returns a dict of measurements (see the module docstring)."""
    steps = args.steps if steps is None else steps
    warmup = args.warmup if warmup is None else warmup
    cold_reps = args.cold_reps if cold_reps is None else cold_reps
    layers = list(wl.layers)
    inputs = {l.name: workloads.layer_inputs(l) for l in layers}
    quant_w = clq.clq_quantize_weights if wbits == 4 else clq.clq_quantize_weights8
    if abits == 4 and codes == "fp6":
        quant_w = clq.clq_quantize_weights_f6
        act_bytes, rq_fn, lin_fn = clq.clq_act_bytes_f6, clq.clq_rotate_quant_act_f6, clq.clq_w4a4_linear_f6
    elif abits == 4:
        act_bytes, rq_fn, lin_fn = clq.clq_act_bytes, clq.clq_rotate_quant_act, clq.clq_w4a4_linear
    else:
        act_bytes, rq_fn, lin_fn = clq.clq_act8_bytes, clq.clq_rotate_quant_act8, clq.clq_a8_linear

    # resident device data; weights quantized once (offline step)
    state = []
    for l in layers:
        X, W, b = inputs[l.name]
        Xd = torch.from_numpy(X).to(dev)
        qw = quant_w(torch.from_numpy(W).to(dev), l.block)
        bd = torch.from_numpy(b).to(dev)
        Xq = torch.empty(act_bytes(l.M, l.K), dtype=torch.uint8, device=dev)
        xs = torch.empty(l.M, dtype=torch.float32, device=dev)
        Y = torch.empty((l.M, l.N), dtype=torch.float16, device=dev)
        state.append((l, Xd, qw, bd, Xq, xs, Y))
    stream = torch.cuda.current_stream()
    torch.cuda.synchronize()

    def step(events=None):
        for i, (l, Xd, qw, bd, Xq, xs, Y) in enumerate(state):
            if events is not None:
                events[i][0].record(stream)
            rq_fn(Xd, l.block, out=Xq, scale_out=xs)
            if events is not None:
                events[i][1].record(stream)
            lin_fn(Xq, xs, qw, bd, out=Y)
            if events is not None:
                events[i][2].record(stream)

    for _ in range(warmup):
        step()
    torch.cuda.synchronize()

    # timed region: exactly `steps` steps, launched back to back
    t0 = time.perf_counter()
    for _ in range(steps):
        step()
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    ms_per_step = wall * 1e3 / steps

    # clocks and power: amd-smi's readings trail the load by up to a second,
    # so they are sampled over a separate run of back-to-back steps (same
    # work) lasting clock_s seconds, the first second dropped
    sampler = None
    if sample_clocks:
        sampler = ClockSampler(torch, dev)
        n_clk = max(1, int(clock_s * 1e3 / ms_per_step))
        with sampler:
            for _ in range(n_clk):
                step()
            torch.cuda.synchronize()

    # single-step times: one event pair per step, nothing between launches
    se = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
    for s in range(steps):
        se[s][0].record(stream)
        step()
        se[s][1].record(stream)
    torch.cuda.synchronize()
    step_ms = [a.elapsed_time(b) for a, b in se]

    # per-launch pass: the same `steps` steps again with HIP events recorded
    # around every launch on the launch stream (the records themselves add
    # gaps between launches, so the step time above is taken without them)
    ev = [[[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in layers] for _ in range(steps)]
    torch.cuda.synchronize()
    for s in range(steps):
        step(ev[s])
    torch.cuda.synchronize()
    rq_t = np.array([[ev[s][i][0].elapsed_time(ev[s][i][1]) for i in range(len(layers))] for s in range(steps)])
    gm_t = np.array([[ev[s][i][1].elapsed_time(ev[s][i][2]) for i in range(len(layers))] for s in range(steps)])
    rq_ms = rq_t.mean(axis=0)
    gemm_ms = gm_t.mean(axis=0)

    # rotate+quant and GEMM with the Infinity Cache flushed before each launch
    # (by reading 512 MB: a flush that writes would leave dirty lines to be
    # written back during the timed launch)
    cold_rq = np.full(len(layers), np.nan)
    cold_gemm = np.full(len(layers), np.nan)
    if cold_reps > 0:
        flush = torch.ones(512 * 1024 * 1024 // 4, dtype=torch.float32, device=dev)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        for i, (l, Xd, qw, bd, Xq, xs, Y) in enumerate(state):
            t_rq, t_g = [], []
            for _ in range(cold_reps):
                flush.sum()
                e0.record(stream)
                rq_fn(Xd, l.block, out=Xq, scale_out=xs)
                e1.record(stream)
                e1.synchronize()
                t_rq.append(e0.elapsed_time(e1))
                flush.sum()
                e0.record(stream)
                lin_fn(Xq, xs, qw, bd, out=Y)
                e1.record(stream)
                e1.synchronize()
                t_g.append(e0.elapsed_time(e1))
            cold_rq[i] = np.median(t_rq)
            cold_gemm[i] = np.median(t_g)
        del flush
    res = dict(layers=layers, inputs=inputs, ms_per_step=ms_per_step, step_ms=step_ms, rq_t=rq_t, gm_t=gm_t,
               rq_ms=rq_ms, gemm_ms=gemm_ms, cold_rq=cold_rq, cold_gemm=cold_gemm,
               clocks=sampler.summary(settle_s=1.0) if sampler is not None else None,
               total_ops=sum(gemm_ops(l) for l in layers))
    del state
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return res


def measure_ceilings(clq, torch, dev, seconds=1.0):
    """Measured ceilings beside the nominal peaks: a 1 GiB device-to-device
    copy (torch copy_, 2 GiB moved per launch) for HBM, and the library's
    matrix-core probe loop (int4-shaped random operands, no memory traffic,
    two workgroups per compute unit) for int8 MFMA, with the clocks and power
    sampled while the probe runs."""
    out = {}
    src = torch.ones(1 << 29, dtype=torch.float16, device=dev)
    dst = torch.empty_like(src)
    for _ in range(3):
        dst.copy_(src)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(10):
        dst.copy_(src)
    e1.record()
    e1.synchronize()
    ms = e0.elapsed_time(e1) / 10
    out["hbm_copy_GBps"] = round(2 * src.numel() * 2 / (ms * 1e-3) / 1e9, 1)
    out["hbm_copy_note"] = "torch copy_ of 1 GiB (read 1 GiB + write 1 GiB per launch), 10 launches"
    del src, dst
    ops = torch.randint(0, 256, (clq.clq_diag_mfma_probe_bytes(),), dtype=torch.uint8, device=dev)
    grid = 2 * torch.cuda.get_device_properties(dev).multi_processor_count
    sink = torch.empty(grid * 256, dtype=torch.int32, device=dev)
    probes = [("mfma_probe", clq.clq_diag_mfma_probe, INT8_PEAK_TOPS,
               "v_mfma_i32_32x32x32_i8 loop on random int4 codes widened to 16 q"),
              ("mfma_f6_probe", clq.clq_diag_mfma_probe_f6, FP6_PEAK_TOPS,
               "v_mfma_f32_32x32x64_f8f6f4 (fp6 e2m3 operands) loop on random int4 codes as fp6")]
    for key, probe, peak, what in probes:
        n = probe(ops, 200, grid, sink)   # warm up, and size the timed launches
        torch.cuda.synchronize()
        t = time.perf_counter()
        probe(ops, 200, grid, sink)
        torch.cuda.synchronize()
        t = time.perf_counter() - t
        iters = max(200, int(200 * (seconds / 4) / max(t, 1e-6)))
        sampler = ClockSampler(torch, dev)
        with sampler:
            for _ in range(4):   # brings the clock to its loaded state (and the readings up to date)
                probe(ops, iters, grid, sink)
            e0.record()
            for _ in range(4):
                n = probe(ops, iters, grid, sink)
            e1.record()
            e1.synchronize()
        ms = e0.elapsed_time(e1) / 4
        out[f"{key}_TOPS"] = round(n / (ms * 1e-3) / 1e12, 1)
        out[f"{key}_frac_of_nominal"] = round(n / (ms * 1e-3) / 1e12 / peak, 4)
        out[f"{key}_ms"] = round(ms, 3)
        out[f"{key}_clocks"] = sampler.summary(settle_s=1.0)
        out[f"{key}_note"] = (f"{what}, {grid} workgroups x 4 waves, 8 accumulators per wave, "
                              "no memory traffic")
    return out


def block_summary(wl, r, abits=4, codes="int4"):
    """Compact per-layer and per-kernel figures of a bench_block result."""
    layers = r["layers"]
    value = r["total_ops"] / (r["ms_per_step"] * 1e-3) / 1e12
    gemm_avg_ms = float(r["gemm_ms"].mean())
    ops_launch = r["total_ops"] / len(layers)
    per = {}
    for i, l in enumerate(layers):
        per[l.name] = {
            "M": l.M, "K": l.K, "N": l.N,
            "gemm_us": pct(r["gm_t"][:, i] * 1e3), "gemm_TOPS": round(gemm_ops(l) / (r["gemm_ms"][i] * 1e-3) / 1e12, 1),
            "gemm_cold_us": round(float(r["cold_gemm"][i]) * 1e3, 2) if np.isfinite(r["cold_gemm"][i]) else None,
            "rq_kernel": rq_kernel_name(l, abits, codes),
            "rq_us": pct(r["rq_t"][:, i] * 1e3),
            "rq_GBps": round(rq_bytes(l, abits, codes) / (r["rq_ms"][i] * 1e-3) / 1e9, 1),
            "rq_cold_us": round(float(r["cold_rq"][i]) * 1e3, 2) if np.isfinite(r["cold_rq"][i]) else None,
            "rq_cold_GBps": (round(rq_bytes(l, abits, codes) / (r["cold_rq"][i] * 1e-3) / 1e9, 1)
                             if np.isfinite(r["cold_rq"][i]) else None)}
    return dict(value=value, gemm_avg_ms=gemm_avg_ms, ops_launch=ops_launch, per=per)


def obs_bytes(B, N, D, metric):
    """Algorithmic HBM bytes of one OBS channel-score pass: read the fp16
    calibration batch, write D scores; the sort / sum metrics also write and
    read back the fp32 mean matrix."""
    b = B * N * D * 2 + D * 4
    if metric not in ("absmax", "range"):
        b += 2 * N * D * 4
    return b


def bench_obs(args, clq, torch, dev):
    """OBS calibration (Sec. 3.3): channel scores of a PixArt-style
    calibration batch (32 samples x 4096 tokens x 1152 channels, the input
    width of qkv/proj/fc1) with the abs-max metric the paper keeps, then the
    column swap.  value = GB/s of the score pass (HBM-bound)."""
    B, N, D = 32, 4096, 1152
    X = workloads.calibration(B, N, D, "L1", seed=2024)
    Xd = torch.from_numpy(X).to(dev)
    metrics = ("absmax", "range", "par", "topk_mean", "percentile")
    ws = {m: torch.zeros(clq.clq_obs_workspace_bytes(N, D, m), dtype=torch.uint8, device=dev)
          for m in metrics}
    scores = torch.empty(D, dtype=torch.float32, device=dev)
    perm = torch.empty(D, dtype=torch.int32, device=dev)
    stream = torch.cuda.current_stream()

    def step():
        clq.clq_obs_channel_scores(Xd, "absmax", workspace=ws["absmax"], out=scores)
        clq.clq_obs_permutation(scores, out=perm)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
    torch.cuda.synchronize()
    ms_per_step = (time.perf_counter() - t0) * 1e3 / args.steps

    # per-launch times (HIP events on the launch stream around `steps`
    # back-to-back launches of one entry point, so that host-side launch
    # overhead overlaps the GPU work), per metric, and of the swap
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)

    def timed(fn):
        fn()
        torch.cuda.synchronize()
        e0.record(stream)
        for _ in range(args.steps):
            fn()
        e1.record(stream)
        e1.synchronize()
        return e0.elapsed_time(e1) / args.steps

    per = {}
    for m in metrics:
        t_sc = timed(lambda: clq.clq_obs_channel_scores(Xd, m, workspace=ws[m], out=scores))
        t_pm = timed(lambda: clq.clq_obs_permutation(scores, out=perm))
        per[m] = (t_sc, t_pm)
    sc_ms = per["absmax"][0]
    achieved = obs_bytes(B, N, D, "absmax") / (sc_ms * 1e-3) / 1e9
    value = obs_bytes(B, N, D, "absmax") / (ms_per_step * 1e-3) / 1e9
    out = {
        "metric": "OBS calibration channel-score pass, HBM GB/s",
        "value": round(value, 1), "unit": "GB/s", "n_gpus": 1, "steps": args.steps,
        "warmup": args.warmup, "ms_per_step": round(ms_per_step, 5), "higher_is_better": True,
        "scaling": "weak", "vs_baseline": None, "dtype": "f32", "data": "synthetic",
        "config": {"workload": "obs_calibration_b32_n4096_d1152", "B": B, "N": N, "D": D,
                   "metric": "absmax", "parallelism": "none (one GPU)"},
        "roofline": {"kernel": "obs_mean_kernel<0> (+ obs_finish_kernel)", "bound": "hbm",
                     "achieved": round(achieved, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                     "frac": round(achieved / HBM_PEAK_GBPS, 4), "traffic": None,
                     "avg_launch_us": round(sc_ms * 1e3, 2),
                     "bytes_per_launch": obs_bytes(B, N, D, "absmax")},
        "per_metric": {m: {"scores_us": round(per[m][0] * 1e3, 2),
                           "scores_GBps": round(obs_bytes(B, N, D, m) / (per[m][0] * 1e-3) / 1e9, 1),
                           "swap_us": round(per[m][1] * 1e3, 2)} for m in metrics},
        "gpu": torch.cuda.get_device_name(dev),
    }
    if not args.no_cpu_baseline:
        # the oracle on the first 4 samples of the same batch
        from oracle import obs as oobs
        t0 = time.perf_counter()
        oobs.obs(X[:4], "absmax")
        t = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(obs_bytes(4, N, D, "absmax") / t / 1e9, 3), "unit": "GB/s",
                               "cores": 1, "kind": "oracle",
                               "sample": f"first 4 of the 32 samples ({t:.2f} s, numpy, one thread)"}
    print(json.dumps(out), flush=True)


def bench_clps(args, clq, torch, dev):
    """CLPS single-layer clip search (Sec. 3.4): the PixArt qkv layer (1152 ->
    3456) on 4096 calibration tokens, 20 candidate clip ratios.  value =
    effective TOPS of the search (20 quantized GEMMs of 2 M N K each, plus the
    window, weight quantization and error passes, over the search time)."""
    M, K, N, b, G = 4096, 1152, 3456, 64, 20
    X = workloads.activations(M, K, "L1", 2101)
    W = workloads.weights(N, K, 2102)
    Xd, Wd = torch.from_numpy(X).to(dev), torch.from_numpy(W).to(dev)
    # the target output X W^T in fp32 (input to the search, computed once)
    Y0 = (Xd.float() @ Wd.float().T).contiguous()
    ws = torch.empty(clq.clq_clps_workspace_bytes(M, N, K), dtype=torch.uint8, device=dev)
    stream = torch.cuda.current_stream()

    def step():
        return clq.clq_clps_search(Xd, Wd, Y0, b, grid=G, workspace=ws)

    for _ in range(max(1, args.warmup // 10)):
        step()
    torch.cuda.synchronize()
    steps = max(3, args.steps // 10)
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    t0 = time.perf_counter()
    e0.record(stream)
    for _ in range(steps):
        al, er, best = step()
    e1.record(stream)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t0) * 1e3 / steps
    ev_ms = e0.elapsed_time(e1) / steps
    ops = G * 2.0 * M * N * K
    value = ops / (ms * 1e-3) / 1e12
    out = {
        "metric": "CLPS single-layer clip search, effective TOPS (20 candidates)",
        "value": round(value, 2), "unit": "TOPS", "n_gpus": 1, "steps": steps, "warmup": max(1, args.warmup // 10),
        "ms_per_step": round(ms, 4), "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "int4", "data": "synthetic",
        "config": {"workload": "clps_pixart_qkv_m4096_k1152_n3456_g20", "M": M, "K": K, "N": N, "block": b,
                   "grid": G, "gamma": 0.01, "parallelism": "none (one GPU)"},
        "search_ms_events": round(ev_ms, 4),
        "best_alpha": float(al[int(best.item())].item()),
        "errors_first_last": [float(er[0].item()), float(er[-1].item())],
        "gpu": torch.cuda.get_device_name(dev),
    }
    if not args.no_cpu_baseline:
        # the oracle's search on the first 256 tokens, 4 candidates
        from oracle import clps as oclps
        t0 = time.perf_counter()
        Y0h = Y0[:256].cpu().numpy()
        oclps.search(X[:256], W, Y0h, b, G=4)
        t = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(4 * 2.0 * 256 * N * K / t / 1e12, 4), "unit": "TOPS",
                               "cores": blas_threads(), "kind": "oracle", "cpu_model": cpu_model(),
                               "sample": f"256 of the 4096 tokens, 4 of the 20 candidates ({t:.1f} s)"}
    print(json.dumps(out), flush=True)


_STACK_W = {}


def stack_weights(torch, dev, nb=28):
    """Device weights and biases of the 28-block stack (drawn once; they do
    not depend on M or the block size)."""
    if nb not in _STACK_W:
        wl = workloads.dit_stack(nb, 4096, 64)
        weights = []
        for j in range(nb):
            blk = {}
            for l in wl.layers[4 * j:4 * j + 4]:
                blk[l.name.split(".")[1]] = (torch.from_numpy(workloads.weights(l.N, l.K, l.seed + 1)).to(dev),
                                             torch.from_numpy(workloads.bias(l.N, l.seed + 2)).to(dev))
            weights.append(blk)
        _STACK_W[nb] = weights
    return _STACK_W[nb]


def stack_point(clq, torch, dev, M, b, steps, perms=None, fold=False, eager=False, fuse=False, codes="int4"):
    """One stack configuration: graph replays timed back to back, plus
    single-replay percentiles (events at replay boundaries)."""
    from paper_2509_24416_amd.stack import DiTStack
    st = DiTStack(stack_weights(torch, dev), M, b, perms=perms, fold=fold, fuse=fuse, codes=codes)
    x = torch.from_numpy(workloads.activations(M, 1152, "L1", 500)).to(dev)
    st.forward(x)
    st.capture()
    for _ in range(3):
        st.replay()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        st.replay()
    torch.cuda.synchronize()
    g_ms = (time.perf_counter() - t0) * 1e3 / steps
    stream = torch.cuda.current_stream()
    ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)) for _ in range(steps)]
    for a, e in ev:
        a.record(stream)
        st.replay()
        e.record(stream)
    torch.cuda.synchronize()
    plans = [clq.clq_w4a4_rq_schedule(M, N, K, b)["fused"] if fuse else 0
             for (K, N) in ((1152, 3456), (1152, 1152), (1152, 4608), (4608, 1152))]
    out = {"graph_ms": round(g_ms, 4), "graph_TOPS": round(st.ops / (g_ms * 1e-3) / 1e12, 1),
           "replay_ms_percentiles": pct([a.elapsed_time(e) for a, e in ev]),
           "launches_per_step": len(st.blocks) * (8 - sum(plans)), "fused_layers": plans}
    if eager:
        t0 = time.perf_counter()
        for _ in range(steps):
            st.forward()
        torch.cuda.synchronize()
        e_ms = (time.perf_counter() - t0) * 1e3 / steps
        out["eager_ms"] = round(e_ms, 4)
        out["eager_TOPS"] = round(st.ops / (e_ms * 1e-3) / 1e12, 1)
    out["ops"] = st.ops
    del st
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return out


def bench_stack(args, clq, torch, dev):
    """The multi-layer path: 28 PixArt-width DiT blocks (112 linears, 223 MB
    of resident int4 weights), rotate+quant + W4A4 GEMM per linear, replayed
    as one HIP graph.  value = effective TOPS at M = 4096 tokens, block 64;
    M = 1024 / 16384, the eager step, the Hadamard block sweep 32 / 64 / 128
    at every M, the stack with each input's rotate+quantize folded into its
    GEMM launch where the schedule allows (clq_w4a4_rq_linear), and the stack
    on the fp6 storage of the codes are reported beside it."""
    nb = 28
    res, fused = {}, {}
    for M in (4096, 1024, 16384):
        for b in (64, 32, 128):
            steps = args.steps if M == 4096 else max(5, args.steps // 4)
            print(f"bench: dit_stack M={M} block={b}", file=sys.stderr, flush=True)
            res[(M, b)] = stack_point(clq, torch, dev, M, b, steps, eager=(b == 64))
        # the same stack with each rotate+quantize folded into its GEMM launch
        # where the schedule allows (clq_w4a4_rq_linear)
        fused[M] = stack_point(clq, torch, dev, M, 64, max(5, args.steps // 4), fuse=True)
    # the same stack on the fp6 storage of the codes, block 64
    fp6 = {}
    for M in (4096, 1024, 16384):
        print(f"bench: dit_stack M={M} block=64 fp6 codes", file=sys.stderr, flush=True)
        fp6[M] = stack_point(clq, torch, dev, M, 64, args.steps if M == 4096 else max(5, args.steps // 4),
                             codes="fp6")
    # one swap vector per layer input (random stand-ins for OBS outputs):
    # gathered by every rotate+quant, or folded into the producing layers
    from paper_2509_24416_amd.stack import LAYERS
    weights = stack_weights(torch, dev)
    perms = [{name: torch.from_numpy(workloads.random_perm(weights[j][name][0].shape[1], 1000 + 4 * j + i)).to(dev)
              for i, name in enumerate(LAYERS)} for j in range(nb)]
    swap = {}
    for fold in (False, True):
        swap["folded_ms" if fold else "gather_ms"] = stack_point(clq, torch, dev, 4096, 64, args.steps,
                                                                 perms=perms, fold=fold)["graph_ms"]
    head = res[(4096, 64)]
    out = {
        "metric": "DiT stack (28 blocks x 4 W4A4 linears) effective TOPS, one HIP graph per step",
        "value": head["graph_TOPS"], "unit": "TOPS", "n_gpus": 1, "steps": args.steps,
        "warmup": 3, "ms_per_step": head["graph_ms"], "higher_is_better": True, "scaling": "weak",
        "vs_baseline": None, "dtype": "int4", "data": "synthetic",
        "config": {"workload": "dit_stack_28x4_m4096_h1152_b64", "blocks": nb, "M": 4096, "block": 64,
                   "launches_per_step": 2 * 4 * nb, "parallelism": "none (one GPU)"},
        "per_M_block": {f"M{M}_b{b}": v for (M, b), v in res.items()},
        "fused_block64": {f"M{M}": v for M, v in fused.items()},
        "fp6codes_block64": {f"M{M}": v for M, v in fp6.items()},
        "swap_vectors_m4096": swap,
        "gpu": torch.cuda.get_device_name(dev),
    }
    print(json.dumps(out), flush=True)


# Shapes for the schedule sweep: token counts from 512 to 32768 against
# layer widths other than the block workloads' (square 2048 and 5120, a
# 2560 -> 10240 expansion and its 10240 -> 2560 projection), plus the 1152 /
# 4608 PixArt widths at token counts the block workloads do not use.
SWEEP_KN = [(2048, 2048), (5120, 5120), (2560, 10240), (10240, 2560), (1152, 4608), (4608, 1152)]
SWEEP_M = [512, 1536, 3072, 6144, 12288, 24576]
GEMM_KERNELS = ["tiles256", "tiles128", "split4", "split2"]
SCHEDULES = {1: "split_k", 2: "whole_tiles", 3: "halves128", 4: "halves64"}


def bench_gemm_schedule(args, clq, torch, dev):
    """The GEMM's automatic kernel choice against every forced schedule (the
    CLQ_DEBUG_GEMM_SCHEDULE knob: k split over workgroups where that balances
    the launch, whole tiles, the
    two-halves kernel on 128- and 64-token tiles) on shapes outside the block
    workloads.  HIP events around `reps` back-to-back launches per schedule,
    after warmup; every schedule computes the same result.  value = geometric
    mean over the shapes of (fastest forced time / automatic time): 1.0 when
    the automatic choice is always the fastest."""
    reps = max(5, args.steps // 25)
    ws = torch.zeros(clq.clq_w4a4_workspace_bytes(), dtype=torch.uint8, device=dev)
    shapes = [(M, K, N) for K, N in SWEEP_KN for M in SWEEP_M]
    if args.sweep_block_shapes:
        shapes = [(l.M, l.K, l.N) for wl in (workloads.C2, workloads.C3, workloads.C4) for l in wl.layers]
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    records, ratios = [], []
    try:
        for M, K, N in shapes:
            W = torch.from_numpy(workloads.weights(N, K, seed=N + K)).to(dev)
            qw = clq.clq_quantize_weights(W, 64)
            X = torch.from_numpy(workloads.activations(M, K, "L1", seed=M + K)).to(dev)
            Xq, xs = clq.clq_rotate_quant_act(X, 64)
            Y = torch.empty((M, N), dtype=torch.float16, device=dev)
            # every schedule warmed up, then three rounds over all of
            # them; the median round per schedule (launches timed later
            # in a sequence read faster while the clock settles)
            forces = []
            for force in (0, 1, 2, 3, 4):
                clq.clq_debug_set(3, force)
                plan = clq.clq_w4a4_schedule(M, N, K)
                if force >= 3 and K < 256:
                    continue   # k loop too short for the two-halves kernel
                if force == 0:
                    auto_plan = plan
                forces.append(force)
                for _ in range(5):
                    clq.clq_w4a4_linear(Xq, xs, qw, out=Y, workspace=ws)
            rounds = {f: [] for f in forces}
            for _ in range(3):
                for force in forces:
                    clq.clq_debug_set(3, force)
                    e0.record()
                    for _ in range(reps):
                        clq.clq_w4a4_linear(Xq, xs, qw, out=Y, workspace=ws)
                    e1.record()
                    e1.synchronize()
                    rounds[force].append(e0.elapsed_time(e1) * 1e3 / reps)
            clq.clq_debug_set(3, 0)
            times = {("auto" if f == 0 else SCHEDULES[f]): round(sorted(v)[1], 2) for f, v in rounds.items()}
            forced = {k: v for k, v in times.items() if k != "auto"}
            best = min(forced, key=forced.get)
            ratio = forced[best] / times["auto"]
            ratios.append(ratio)
            records.append({"M": M, "N": N, "K": K, "auto_kernel": "split_k" if auto_plan["split_stages"] > 0 else GEMM_KERNELS[auto_plan["kernel"]],
                            "auto_split": auto_plan["split_stages"] > 0, "us": times, "fastest_forced": best,
                            "fastest_over_auto": round(ratio, 4),
                            "auto_TOPS": round(2.0 * M * N * K / (times["auto"] * 1e-6) / 1e12, 1)})
            print(f"bench: gemm_schedule {M}x{N}x{K} {times}", file=sys.stderr, flush=True)
            del X, Xq, xs, Y, W, qw
    finally:
        clq.clq_debug_set(3, 0)
    gm = math.exp(sum(math.log(r) for r in ratios) / len(ratios))
    worst = min(records, key=lambda r: r["fastest_over_auto"])
    out = {
        "metric": "GEMM schedule heuristics: fastest forced schedule time / automatic schedule time (geometric mean)",
        "value": round(gm, 4), "unit": "ratio", "n_gpus": 1, "steps": reps, "warmup": 3,
        "higher_is_better": True, "scaling": "none", "vs_baseline": None, "dtype": "int4", "data": "synthetic",
        "config": {"workload": "gemm_schedule_sweep_block_shapes" if args.sweep_block_shapes else "gemm_schedule_sweep",
                   "block": 64, "shapes": [list(x) for x in shapes], "parallelism": "none (one GPU)"},
        "shapes": len(records), "auto_fastest_or_within_2pct": sum(r["fastest_over_auto"] >= 0.98 for r in records),
        "worst": {k: worst[k] for k in ("M", "N", "K", "auto_kernel", "fastest_forced", "fastest_over_auto")},
        "records": records, "gpu": torch.cuda.get_device_name(dev),
    }
    print(json.dumps(out), flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=500)
    ap.add_argument("--warmup", type=int, default=1000)
    ap.add_argument("--cold-reps", type=int, default=10)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-clocks", action="store_true",
                    help="skip the 2.5 s clock and power sampling pass")
    ap.add_argument("--no-ceilings", action="store_true",
                    help="skip the measured HBM-copy and matrix-core ceilings")
    ap.add_argument("--no-extra", action="store_true",
                    help="skip the PixArt block and 28-block stack figures beside the headline")
    ap.add_argument("--workload", default="video_block",
                    choices=["video_block", "pixart_block", "flux_block", "video_block_w4a8", "video_block_w8a8",
                             "pixart_block_w4a8", "pixart_block_w8a8", "obs_calibration", "clps_search",
                             "dit_stack", "gemm_schedule"],
                    help="video_block: the W4A4 hot path on the video DiT block, M = 43200 (default); "
                         "pixart_block (M = 8192) and flux_block (width 3072, M = 4608, block 128): the same "
                         "on the other block configurations; *_w4a8 / *_w8a8: 8-bit activations (and "
                         "weights); obs_calibration: the OBS channel-score pass; clps_search: the CLPS "
                         "clip search; dit_stack: the 28-block stack, one HIP graph per step; "
                         "gemm_schedule: the GEMM's automatic kernel choice against every forced schedule "
                         "on shapes outside the block workloads")
    ap.add_argument("--codes", default="int4", choices=["int4", "fp6"],
                    help="W4A4 operand storage: int4 (nibble-packed, int8 matrix instructions; default) or fp6 "
                         "(the same codes as e2m3, fp6 matrix instructions)")
    ap.add_argument("--sweep-block-shapes", action="store_true",
                    help="gemm_schedule: sweep the block workloads' own layer shapes instead")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain 1 GiB device copy 5 times (reference for the HBM "
                         "byte counters) and exit")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: the benchmark runs on exactly one GPU; --gpus {args.gpus} is not supported "
              "(the hot path would shard by token rows with no collective: each GPU runs the same "
              "kernels on its share of the rows)", file=sys.stderr)
        sys.exit(2)

    import torch

    dev = torch.device("cuda:0")
    if args.copy_calibration:
        src = torch.ones(1 << 29, dtype=torch.float16, device=dev)
        dst = torch.empty_like(src)
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        print(json.dumps({"copy_calibration_bytes_each_way": src.numel() * 2, "launches": 5}))
        return

    import paper_2509_24416_amd as clq

    if args.workload == "obs_calibration":
        bench_obs(args, clq, torch, dev)
        return
    if args.workload == "clps_search":
        bench_clps(args, clq, torch, dev)
        return
    if args.workload == "dit_stack":
        bench_stack(args, clq, torch, dev)
        return
    if args.workload == "gemm_schedule":
        bench_gemm_schedule(args, clq, torch, dev)
        return

    base = args.workload.split("_w")[0]
    wbits, abits = 4, 4
    if args.workload.endswith("_w4a8"):
        wbits, abits = 4, 8
    elif args.workload.endswith("_w8a8"):
        wbits, abits = 8, 8
    codes = args.codes
    if codes == "fp6" and (wbits, abits) != (4, 4):
        print("bench.py: --codes fp6 applies to the W4A4 workloads only", file=sys.stderr)
        sys.exit(2)
    wl = BLOCKS[base]
    print(f"bench: {wl.name} W{wbits}A{abits} ({codes} codes): {args.warmup} warmup + {args.steps} timed steps",
          file=sys.stderr, flush=True)
    r = bench_block(wl, args, clq, torch, dev, wbits, abits, sample_clocks=not args.no_clocks, codes=codes)
    sm = block_summary(wl, r, abits, codes)
    layers = r["layers"]
    achieved = sm["ops_launch"] / (sm["gemm_avg_ms"] * 1e-3) / 1e12
    rq_avg_bytes = sum(rq_bytes(l, abits, codes) for l in layers) / len(layers)
    rq_achieved = rq_avg_bytes / (float(r["rq_ms"].mean()) * 1e-3) / 1e9
    cold_bytes = sum(rq_bytes(l, abits, codes) for l in layers)
    cold_rq_total = float(np.nansum(r["cold_rq"]))
    cold_gbps = cold_bytes / (cold_rq_total * 1e-3) / 1e9 if cold_rq_total > 0 else 0.0
    traffic = (load_traffic(TRAFFIC_FILES.get((wl.name, codes)), kernel_sha(codes))
               if (wbits, abits) == (4, 4) else None)
    plans = [clq.clq_w4a4_schedule(l.M, l.N, l.K) for l in layers] if (abits == 4 and codes == "int4") else None
    if codes == "fp6":
        plans = [{"kernel": clq.clq_w4a4_schedule_f6(l.M, l.N, l.K)} for l in layers]
        kinds = {clq.F6_SCHEDULES[p["kernel"]].split(" (")[0] for p in plans}
    else:   # (the 8-bit settings choose as the int4 storage does without a workspace)
        kinds = {"w4a4_gemm_kernel" if p["split_stages"] > 0 else
                 "split_gemm_kernel" if p["kernel"] >= 2 else "tile_gemm_kernel"
                 for p in plans or [clq.clq_w4a4_schedule(l.M, l.N, l.K, with_workspace=False) for l in layers]}
    gemm_name = " / ".join(sorted(kinds)) + " (mean over the 4 linears)"
    # the roofline prices a launch against the peak of the matrix
    # instruction it issues: int8 for the int4 path (codes widened to int8),
    # fp6 for the fp6-stored codes
    peak = FP6_PEAK_TOPS if codes == "fp6" else INT8_PEAK_TOPS
    setting = f"W{wbits}A{abits}"
    out = {
        "metric": f"{setting} linear effective TOPS + % int8-MFMA peak; rotate+quant HBM GB/s",
        "value": round(sm["value"], 2),
        "unit": "TOPS",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": round(r["ms_per_step"], 5),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": ("fp6" if codes == "fp6" else "int4") if (wbits, abits) == (4, 4) else
                 ("int4 x int8" if wbits == 4 else "int8"),
        "data": "synthetic",
        "config": {"workload": wl.name + ("" if (wbits, abits) == (4, 4) else f"_{setting.lower()}")
                   + ("_fp6codes" if codes == "fp6" else ""),
                   "codes": codes,
                   "M": layers[0].M, "hidden": layers[0].K, "mlp": layers[2].N,
                   "block": layers[0].block, "layers": {l.name.split(".")[1]: [l.K, l.N] for l in layers},
                   "parallelism": "none (one GPU)"},
        "pct_int8_peak": round(100 * sm["value"] / INT8_PEAK_TOPS, 2),
        "step_ms_percentiles": pct(r["step_ms"]),
        "roofline": {"kernel": gemm_name, "bound": "mfma", "achieved": round(achieved, 1),
                     "peak": peak, "unit": "TFLOP/s",
                     "peak_instruction": ("fp6 MFMA (dense 10.1 PFLOP/s)" if codes == "fp6"
                                          else "int8 MFMA (dense 5.0 POP/s)"),
                     "frac": round(achieved / peak, 4),
                     "frac_of_int8_peak": round(achieved / INT8_PEAK_TOPS, 4),
                     "traffic": traffic, "avg_launch_us": round(sm["gemm_avg_ms"] * 1e3, 2),
                     "ops_per_launch": sm["ops_launch"],
                     "launch_us_percentiles": pct(r["gm_t"].mean(axis=1) * 1e3)},
        # the graded figure is the cold-cache one (each launch after a
        # 512 MB read flush); the in-step figure has each launch follow the
        # previous linear's GEMM, whose output lines are still being written
        # back, so it measures the pipeline rather than the kernel
        "rotate_quant": {"kernels": {l.name: rq_kernel_name(l, abits, codes) for l in layers}, "bound": "hbm",
                         "basis": "cold cache, all four launches" if cold_rq_total > 0 else "in step",
                         "achieved": round(cold_gbps if cold_rq_total > 0 else rq_achieved, 1),
                         "peak": HBM_PEAK_GBPS, "unit": "GB/s",
                         "frac": round((cold_gbps if cold_rq_total > 0 else rq_achieved) / HBM_PEAK_GBPS, 4),
                         "bytes_per_launch": rq_avg_bytes,
                         "cold_avg_launch_us": (round(cold_rq_total * 1e3 / len(layers), 2) if cold_rq_total > 0 else None),
                         "in_step_GBps": round(rq_achieved, 1),
                         "in_step_frac": round(rq_achieved / HBM_PEAK_GBPS, 4),
                         "in_step_avg_launch_us": round(float(r["rq_ms"].mean()) * 1e3, 2)},
        "per_layer": sm["per"],
        "gemm_schedule": ({l.name: plans[i] for i, l in enumerate(layers)} if plans else None),
        "clocks": r["clocks"],
        "gpu": torch.cuda.get_device_name(dev),
    }
    if not args.no_ceilings:
        print("bench: measured ceilings", file=sys.stderr, flush=True)
        ceil = measure_ceilings(clq, torch, dev)
        out["ceilings"] = ceil
        out["roofline"]["frac_of_measured_ceiling"] = round(
            achieved / ceil["mfma_f6_probe_TOPS" if codes == "fp6" else "mfma_probe_TOPS"], 4)
        out["rotate_quant"]["frac_of_copy_ceiling"] = round(out["rotate_quant"]["achieved"] / ceil["hbm_copy_GBps"], 4)
        out["rotate_quant"]["in_step_frac_of_copy_ceiling"] = round(rq_achieved / ceil["hbm_copy_GBps"], 4)
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(layers, r["inputs"], wbits=wbits, abits=abits)
    r = None
    if not args.no_extra and (wbits, abits) == (4, 4):
        extra = {}
        for name, c2 in (("video_block", "int4"), ("video_block", "fp6"), ("pixart_block", "int4"),
                         ("pixart_block", "fp6")):
            if (name, c2) == (base, codes):
                continue
            wl2 = BLOCKS[name]
            key = wl2.name + ("_fp6codes" if c2 == "fp6" else "")
            print(f"bench: extra {key}", file=sys.stderr, flush=True)
            r2 = bench_block(wl2, args, clq, torch, dev, steps=max(20, args.steps // 2),
                             warmup=max(20, args.warmup // 2), cold_reps=0, sample_clocks=False, codes=c2)
            s2 = block_summary(wl2, r2, codes=c2)
            g_tops = s2["ops_launch"] / (s2["gemm_avg_ms"] * 1e-3) / 1e12
            extra[key] = {"codes": c2, "value_TOPS": round(s2["value"], 2),
                          "ms_per_step": round(r2["ms_per_step"], 5),
                          "step_ms_percentiles": pct(r2["step_ms"]),
                          "gemm_avg_us": round(s2["gemm_avg_ms"] * 1e3, 2),
                          "gemm_frac": round(g_tops / (FP6_PEAK_TOPS if c2 == "fp6" else INT8_PEAK_TOPS), 4),
                          "gemm_frac_of_int8_peak": round(g_tops / INT8_PEAK_TOPS, 4),
                          "per_layer": {k: {"gemm_us": v["gemm_us"]["median"], "gemm_TOPS": v["gemm_TOPS"],
                                            "rq_us": v["rq_us"]["median"], "rq_GBps": v["rq_GBps"]}
                                        for k, v in s2["per"].items()}}
            del r2
        print("bench: extra dit_stack m16384", file=sys.stderr, flush=True)
        extra["dit_stack_28x4_m16384_h1152_b64"] = stack_point(clq, torch, dev, 16384, 64, steps=20)
        extra["dit_stack_28x4_m16384_h1152_b64_fp6codes"] = stack_point(clq, torch, dev, 16384, 64, steps=20,
                                                                         codes="fp6")
        out["extra"] = extra
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
