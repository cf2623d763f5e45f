#!/usr/bin/env python3
"""Benchmark of the eOptShrinkQ hot path on one MI355X.

A step is one pass of the whole path over one batch of synthetic KV blocks resident in HBM:
eoq_compress (Gram + eigensolve + rank + shrinkage + residual + rotate/quantize/pack), eoq_decompress of
the record, and eoq_scores of decode queries against the compressed keys of the batch.  The default
workload is the whole Llama-3.1-8B-shaped cache (32 layers x 8 KV heads x {K,V} x T=32768: 32768 blocks of
512 x 128, 4.29 GB of fp16, 2 residual bits), the largest configuration that is one single-GPU batch.
Prints ONE JSON line.
"""
from __future__ import annotations

import argparse
import json
import multiprocessing
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBPS = 8000.0
FP64_VECTOR_PEAK_TFLOPS = 78.6     # 256 CUs x 4 SIMD x 16 lanes x 2 flop x 2.4 GHz
INT8_MFMA_PEAK_TOPS = 5000.0       # dense int8 matrix peak
D = 128


def spectral_fp64_flops_per_block(n: int, mean_rank: float, jacobi_sweeps: float, fp32_input: bool = False) -> float:
    """Algorithmic double-precision flops the vector ALUs must do per block in the spectral kernel: Householder
    tridiagonalisation 4/3 d^3, Sturm bisection of d eigenvalues to 53 bits at 3 flops per matrix row
    (3 * 53 * d^2), and per retained component the twisted factorisation (~10 d) plus the back-transformation
    through d-2 reflectors (2 d^2).  The Gram matrix is NOT in this count for binary16 input (it runs in integer
    arithmetic on the matrix cores, see gram_int8_ops_per_block); for float32 input it is n d (d+1) fp64 flops.
    When the Jacobi solver is selected instead, each sweep is d(d-1)/2 column pairs at 8 d flops."""
    gram = n * D * (D + 1) if fp32_input else 0.0
    if jacobi_sweeps > 0:
        return gram + jacobi_sweeps * (D * (D - 1) // 2) * 8 * D
    return gram + 4.0 / 3.0 * D ** 3 + 3 * 53 * D * D + mean_rank * (2 * D * D + 10 * D)


def gram_int8_ops_per_block(n: int) -> float:
    """Integer operations the matrix cores execute for the Gram matrix of one binary16 block: the 36 tiles of 16 x 16 on
    and above the diagonal, sixteen byte-plane pairs each, 2 n 256 operations per pair."""
    return 36 * 16 * 2.0 * n * 256


def compress_bytes_per_block(n: int, bits: int, mean_rank: float) -> float:
    """Algorithmic HBM bytes of eoq_compress per block: the block read once, codes, norms, the retained factor rows
    and the per-block scalars written once."""
    return n * D * 2 + n * (bits * D // 8 + 2) + mean_rank * (n + D) * 2 + 12 + 2 * 4 * mean_rank


def measure_ceilings(ctx, torch, dev):
    """What this device reaches on a plain copy and on dependent-free loops of the instructions the kernels are made
    of (eoq_ceiling of the library), to be read beside the datasheet peaks."""
    buf = torch.empty(1 << 30, dtype=torch.uint8, device=dev)
    buf.zero_()
    out = {}
    for key, kind in (("copy_GBps", 0), ("read_GBps", 6), ("write_GBps", 7)):
        best = 0.0
        for _ in range(3):      # a ceiling: the best of three launches
            r = ctx.eoq_ceiling(kind, buf, 1)
            best = max(best, r["work_a"] / (r["ms"] * 1e-3) / 1e9)
        out[key] = best
    for key, kind, scale in (("fp64_fma_TFLOPs", 1, 1e12), ("mfma_f16_TFLOPs", 2, 1e12), ("mfma_i8_TOPs", 3, 1e12),
                             ("mfma_f64_TFLOPs", 4, 1e12)):
        r = ctx.eoq_ceiling(kind, buf, 4000)
        out[key] = (r["work_a"] + r["work_b"]) / (r["ms"] * 1e-3) / scale
    # the f64 matrix instruction beside f64 vector work on the other wave of each SIMD: the sum of the two rates shows
    # that they take turns on the same arithmetic units (no overlap to be had from moving updates to the matrix pipeline)
    r = ctx.eoq_ceiling(10, buf, 4000)
    out["mfma_f64_beside_fma64_TFLOPs"] = (r["work_a"] + r["work_b"]) / (r["ms"] * 1e-3) / 1e12
    out["compute_units"] = r["compute_units"]
    # the same f64 FMA loop on 1, 2 and 4 waves per SIMD: what one wave can issue by itself, and what the two waves per
    # SIMD that the spectral kernel's registers allow reach between them
    for waves in (1, 2, 4):
        r = ctx.eoq_ceiling(30 + waves, buf, 4000)
        out["fp64_fma_%dwave_per_simd_TFLOPs" % waves] = (r["work_a"] + r["work_b"]) / (r["ms"] * 1e-3) / 1e12
    del buf
    return out


# ---- CPU baseline (the float64 oracle, untouched, fanned out over host cores) ---------------------------
def _cpu_init():
    # one BLAS thread per worker (the pool is the parallelism); must be in place before NumPy loads its BLAS
    for var in ("OMP_NUM_THREADS", "OPENBLAS_NUM_THREADS", "MKL_NUM_THREADS"):
        os.environ[var] = "1"
    import numpy  # noqa: F401
    try:
        from threadpoolctl import threadpool_limits
        threadpool_limits(1)
    except Exception:
        pass


def _cpu_job(args):
    import numpy as np
    import oracle
    blocks16, bits, seed, q, passes, factor_bits = args
    Pi = oracle.haar_rotation(D, seed).astype(np.float32).astype(np.float64)
    cb = oracle.lloyd_max_gaussian(bits)
    n = 0
    for _ in range(passes):
        for S in blocks16:
            rec = oracle.compress_block(S.astype(np.float64), Pi, cb, factor_bits=factor_bits)
            x = oracle.decompress_block(rec, Pi, cb).astype(np.float16)
            if q is not None:
                oracle.score_block(q, rec, Pi, cb)
            n += 1
    return n


def cpu_baseline(blocks_cpu, bits: int, seed: int, q_cpu, sample_blocks: int, passes: int, factor_bits: int = 16):
    import numpy as np
    cores = min(os.cpu_count() or 1, 16)       # at most 16 workers, stated in `cores`
    B = min(sample_blocks, blocks_cpu.shape[0])
    arr = blocks_cpu[:B].numpy()
    q = None if q_cpu is None else q_cpu.double().numpy()
    per = max(1, B // (cores * 4))
    jobs = [(arr[i:i + per], bits, seed, q, passes, factor_bits) for i in range(0, B, per)]
    ctx = multiprocessing.get_context("spawn")
    with ctx.Pool(cores, initializer=_cpu_init) as pool:
        pool.map(_cpu_job, [(arr[:1], bits, seed, q, 1, factor_bits)] * cores)   # start the workers before the clock
        t0 = time.perf_counter()
        done = sum(pool.map(_cpu_job, jobs))
        dt = time.perf_counter() - t0
    nbytes = done * arr.shape[1] * arr.shape[2] * 2
    return {"value": nbytes / dt / 1e9, "unit": "GB/s", "cores": cores, "kind": "oracle",
            "sample": f"{passes} passes over the first {B} blocks of the batch ({done} block passes), whole path "
                      f"(compress+decompress+scores), float64 NumPy, one single-threaded worker per core",
            "seconds": dt, "blocks_per_s": done / dt}


def log(msg: str):
    print(f"[bench {time.strftime('%H:%M:%S')}] {msg}", file=sys.stderr, flush=True)


def stream_bench(args, torch, eoq, synth, dev) -> int:
    """Chunked prefill (cfg7): a step takes the newest 128 tokens of all 32 layers x {K,V} x 8 heads in the model's
    token-major layout ([64][128][8][128] binary16), compresses them as 512 blocks of 128 x 128 into slot c of a
    store of 16 slots per head-tensor (eoq_compress_chunk), decompresses 512 stored blocks, and scores one layer's
    32 query heads against its 8 KV heads over the 16 stored blocks plus a 64-token binary16 tail
    (eoq_scores_stream)."""
    spec = synth.config(7)
    bits, n, H, L2, cap, tail_len = args.bits, spec.n, 8, 64, 16, 64
    blocks, _ = synth.make_blocks(spec, device=dev)                       # [512][128][128], tensor = (layer, K/V, head)
    B = blocks.shape[0]
    chunk = blocks.view(L2, H, n, D).permute(0, 2, 1, 3).contiguous()     # [64][128][8][128]
    ctx = eoq.Context(n=n, bits=bits)
    ctx.eoq_profile(True)
    store = eoq.Packed.empty(B * cap, n, D, bits, ctx.r_max, dev)
    fq = eoq.FactorCodes.empty(B * cap, n, D, ctx.r_max, dev) if args.factor_bits == 4 else None
    ws = torch.empty(ctx.eoq_workspace_bytes(B), dtype=torch.uint8, device=dev)
    xhat = torch.empty(B, n, D, dtype=torch.float16, device=dev)
    first = eoq.Packed(*(t[:B] for t in (store.codes, store.norms, store.rank, store.phi, store.sigma, store.lfac,
                                          store.rfac, store.flags)))
    n_kv, group = H, 4
    q = synth.make_queries(1, n_kv * group, device=dev)
    tail = chunk[0, :tail_len].permute(1, 0, 2).contiguous().view(1, n_kv, tail_len, D)
    scores = torch.empty(1, n_kv * group, cap * n + tail_len, dtype=torch.float32, device=dev)

    def fill(c):
        lay = eoq.ChunkLayout(n * H * D, H, D, H * D, c % cap, cap)
        ctx.eoq_compress_chunk(chunk, B, lay, store, fq, ws)

    def step(c):
        fill(c)
        ctx.eoq_decompress(first, xhat)
        ctx.eoq_scores_stream(store, q, n_kv, cap, cap, tail, tail_len, scores)

    for c in range(cap):                   # fill every slot once (no slot is read before it is written): the timed
        fill(c)                            # steps then overwrite slots in rotation
    for c in range(args.warmup):
        step(c)
    torch.cuda.synchronize()
    log("store filled, warmup done")
    stage = {"spectral": 0.0, "encode": 0.0, "decode": 0.0, "scores": 0.0}
    t0 = time.perf_counter()
    for c in range(args.steps):
        step(c)
        ms = ctx.eoq_stage_ms()
        for k_ in stage:
            stage[k_] += ms[k_]
    torch.cuda.synchronize()
    ms_per_step = (time.perf_counter() - t0) * 1e3 / args.steps
    for k_ in stage:
        stage[k_] /= args.steps
    eager_ms = ms_per_step
    # The step is a short chain of launches, so it is also replayed from HIP graphs (one per slot of the rotation,
    # captured with the event recording of the profiling off): the same kernels on the same data, without the host's
    # launch work.  `value` is quoted on the replayed step; the eager time and the per-kernel times stay beside it.
    graphed = False
    if not args.no_graph:
        try:
            ctx.eoq_profile(False)
            graphs = []
            for c in range(cap):
                g = torch.cuda.CUDAGraph()
                with torch.cuda.graph(g):
                    step(c)
                graphs.append(g)
            for c in range(args.warmup):
                graphs[c % cap].replay()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for c in range(args.steps):
                graphs[c % cap].replay()
            torch.cuda.synchronize()
            ms_per_step = (time.perf_counter() - t0) * 1e3 / args.steps
            graphed = True
            log(f"graph replay: {ms_per_step:.3f} ms/step (eager {eager_ms:.3f})")
        except Exception as exc:   # keep the eager figure if the capture is refused
            log(f"graph capture failed ({exc}); keeping the eager time")
            ms_per_step = eager_ms
    in_bytes = B * n * D * 2
    ranks = store.rank[:B * cap].view(B, cap)[:, 0].double().cpu()
    flops = spectral_fp64_flops_per_block(n, ranks.mean().item(), 0.0) * B
    achieved = flops / (stage["spectral"] * 1e-3) / 1e12
    out = {
        "metric": "KV compress GB/s (fp16 in) at d=128, 2-bit; dequant GB/s; % of roofline",
        "value": in_bytes / (ms_per_step * 1e-3) / 1e9, "unit": "GB/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "f16+f64", "data": "synthetic",
        "config": {"workload": f"{spec.name}: one prefill chunk per step, {B} blocks of {n}x{D} fp16 in token-major "
                               f"layout into a store of {cap} slots per tensor, b={bits}; decompress of {B} stored "
                               f"blocks; scores of {n_kv * group} queries on {n_kv * cap} stored blocks + {tail_len} "
                               f"tail tokens per head",
                   "blocks": B, "n": n, "d": D, "bits": bits, "factor_bits": args.factor_bits, "input_bytes": in_bytes},
        "stages": {"compress_GBps_fp16_in": in_bytes / ((stage["spectral"] + stage["encode"]) * 1e-3) / 1e9,
                   "spectral_ms": stage["spectral"], "encode_ms": stage["encode"], "dequant_ms": stage["decode"],
                   "dequant_GBps_out": in_bytes / (stage["decode"] * 1e-3) / 1e9, "scores_ms": stage["scores"],
                   "mean_rank": ranks.mean().item(),
                   "eager_ms_per_step": eager_ms, "graph_replay": graphed,
                   "host_overhead_ms": ms_per_step - sum(stage.values())},
        "roofline": {"kernel": "eoq_spectral_tridiag_kernel", "bound": "alu", "achieved": achieved,
                     "peak": FP64_VECTOR_PEAK_TFLOPS, "unit": "TFLOP/s", "frac": achieved / FP64_VECTOR_PEAK_TFLOPS,
                     "traffic": None},
    }
    if args.cpu_blocks > 0:
        nb = min(args.cpu_blocks, B)
        out["cpu_baseline"] = cpu_baseline(blocks[:nb].cpu(), bits, ctx.rot_seed, q[0, :group].cpu(), nb, args.cpu_passes,
                                           args.factor_bits)
    print(json.dumps(out))
    return 0


def time_codec(ctx, torch, eoq, blocks, bits, steps, warmup):
    """Eager compress + decompress of a batch with the library's own per-kernel events: a secondary workload's figures."""
    B, n = blocks.shape[0], blocks.shape[1]
    rec = eoq.Packed.empty(B, n, D, bits, ctx.r_max, blocks.device)
    ws = torch.empty(ctx.eoq_workspace_bytes(B), dtype=torch.uint8, device=blocks.device)
    xhat = torch.empty(B, n, D, dtype=torch.float16, device=blocks.device)
    ctx.eoq_profile(True)
    acc = {"spectral": 0.0, "encode": 0.0, "decode": 0.0}
    for it in range(warmup + steps):
        ctx.eoq_compress(blocks, rec, ws)
        ctx.eoq_decompress(rec, xhat)
        ms = ctx.eoq_stage_ms()
        if it >= warmup:
            for k_ in acc:
                acc[k_] += ms[k_] / steps
    torch.cuda.synchronize()
    ranks = rec.rank.double()
    mean_rank = ranks.mean().item()
    in_bytes = B * n * D * 2
    moved = B * n * (bits * D // 8 + 2) + int(ranks.sum().item()) * (n + D) * 2 + B * 12
    comp_ms = acc["spectral"] + acc["encode"]
    return {"blocks": B, "n": n, "bits": bits, "input_bytes": in_bytes, "mean_rank": mean_rank,
            "spectral_ms": acc["spectral"], "encode_ms": acc["encode"], "dequant_ms": acc["decode"],
            "compress_GBps_fp16_in": in_bytes / (comp_ms * 1e-3) / 1e9,
            "spectral_frac_fp64_alu": spectral_fp64_flops_per_block(n, mean_rank, 0.0) * B / (acc["spectral"] * 1e-3) / 1e12
                                      / FP64_VECTOR_PEAK_TFLOPS,
            "dequant_GBps_moved": (in_bytes + moved) / (acc["decode"] * 1e-3) / 1e9,
            "dequant_frac_hbm": (in_bytes + moved) / (acc["decode"] * 1e-3) / 1e9 / HBM_PEAK_GBPS}


def main() -> int:
    import faulthandler
    faulthandler.enable()
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", default="cfg3", choices=["cfg2", "cfg3", "cfg4", "cfg5", "cfg6", "cfg7"],
                    help="cfg3 (default): the whole Llama-3.1-8B-shaped cache, 32768 blocks of 512 x 128 (4.29 GB), the "
                         "largest configuration that is one single-GPU batch; cfg4: one Ministral-8B-shaped layer")
    ap.add_argument("--bits", type=int, default=2)
    ap.add_argument("--factor-bits", type=int, default=16, choices=[16, 4],
                    help="storage of the SVD factors: binary16 (default) or 4-bit codes with per-block Lloyd-Max codebooks")
    ap.add_argument("--no-graph", action="store_true",
                    help="time the eager step instead of its replay from a captured HIP graph")
    ap.add_argument("--cpu-blocks", type=int, default=1024, help="blocks in the CPU-baseline sample (0 = skip)")
    ap.add_argument("--cpu-passes", type=int, default=40, help="passes of the oracle over that sample (about 10-20 s of CPU work)")
    ap.add_argument("--no-extras", action="store_true",
                    help="skip the secondary figures (config 3 at b = 3, one config-4 layer, TQ_prod, attention output, ceilings)")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="also run one plain device copy of the input batch (2 x input_bytes of HBM traffic) before the "
                         "timed region: the reference dispatch that scales the rocprofv3 FETCH_SIZE / WRITE_SIZE counters")
    args = ap.parse_args()
    if args.gpus != 1:
        print("bench.py: this build runs on ONE GPU only (blocks are independent: a multi-GPU run would shard the "
              "block list and replicate the tables); --gpus must be 1", file=sys.stderr)
        return 2

    import torch
    from paper_2605_02905_amd import eoq, synth

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        return 3
    dev = torch.device("cuda:0")
    cfg = int(args.workload[3])
    if cfg == 7:
        return stream_bench(args, torch, eoq, synth, dev)
    spec = synth.config(cfg)
    bits = args.bits
    log(f"generating {spec.name} on the GPU")
    blocks, _ = synth.make_blocks(spec, device=dev)
    torch.cuda.synchronize()
    log(f"{blocks.shape[0]} blocks ready")
    B, n = blocks.shape[0], spec.n
    # Decode queries against the key half of the batch.  The generator's tensors are (layer, head, K/V) combinations;
    # the batch is put in the order [K tensors of all layers and heads][V tensors ...] once, before anything is timed, so
    # that the keys are one contiguous record: one decode token scores against every layer's keys (n_seq = layers).
    if cfg == 5:
        n_seq, n_kv, group = 16, 8, 4
    else:
        n_kv, group = 8, 4
        n_seq = spec.n_tensors // (2 * n_kv)
        v = blocks.view(n_seq, n_kv, 2, spec.blocks_per_tensor, n, D)
        blocks = torch.cat([v[:, :, 0].reshape(-1, n, D), v[:, :, 1].reshape(-1, n, D)])
        del v
    ctx = eoq.Context(n=n, bits=bits)
    ctx.eoq_profile(True)
    rec = eoq.Packed.empty(B, n, D, bits, ctx.r_max, dev)
    ws = torch.empty(ctx.eoq_workspace_bytes(B), dtype=torch.uint8, device=dev)
    xhat = torch.empty(B, n, D, dtype=torch.float16, device=dev)
    if cfg == 5:
        key_blocks = B
        bph = B // (n_seq * n_kv)
    else:
        bph = spec.blocks_per_tensor
        key_blocks = n_seq * n_kv * bph
    keys = eoq.Packed(rec.codes[:key_blocks], rec.norms[:key_blocks], rec.rank[:key_blocks], rec.phi[:key_blocks],
                      rec.sigma[:key_blocks], rec.lfac[:key_blocks], rec.rfac[:key_blocks], rec.flags[:key_blocks])
    q = synth.make_queries(n_seq, n_kv * group, device=dev)
    scores = torch.empty(n_seq, n_kv * group, bph * n, dtype=torch.float32, device=dev)

    fq = eoq.FactorCodes.empty(B, n, D, ctx.r_max, dev) if args.factor_bits == 4 else None

    def step():
        if fq is None:
            ctx.eoq_compress(blocks, rec, ws)
        else:
            ctx.eoq_compress_q4(blocks, rec, fq, ws)      # its factor-fitting kernel is timed with the encoder
        ctx.eoq_decompress(rec, xhat)
        ctx.eoq_scores(keys, q, n_kv, scores)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    log("warmup done")
    if args.copy_calibration:
        xhat.view(-1).copy_(blocks.view(-1))      # one elementwise copy kernel: reads and writes input_bytes each
        torch.cuda.synchronize()
    stage = {"spectral": 0.0, "encode": 0.0, "decode": 0.0, "scores": 0.0}
    t0 = time.perf_counter()
    for _ in range(args.steps):
        step()
        ms = ctx.eoq_stage_ms()          # waits for this step's events: per-kernel durations on the launch stream
        for k_ in stage:
            stage[k_] += ms[k_]
    torch.cuda.synchronize()
    total_s = time.perf_counter() - t0
    ms_per_step = total_s * 1e3 / args.steps
    log(f"timed {args.steps} steps: {ms_per_step:.3f} ms/step")
    for k_ in stage:
        stage[k_] /= args.steps
    eager_ms = ms_per_step
    # The loop above waits for every step's events (that is how the per-kernel times are read), so the host's launch
    # work is not hidden.  The step is therefore also replayed from a captured HIP graph, with the event recording of
    # the profiling off: the same kernels on the same data.  `value` is quoted on the replayed step; the eager time
    # and the per-kernel times stay beside it.
    graphed = False
    if not args.no_graph:
        try:
            ctx.eoq_profile(False)
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g):
                step()
            for _ in range(args.warmup):
                g.replay()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(args.steps):
                g.replay()
            torch.cuda.synchronize()
            ms_per_step = (time.perf_counter() - t0) * 1e3 / args.steps
            graphed = True
            log(f"graph replay: {ms_per_step:.3f} ms/step (eager {eager_ms:.3f})")
        except Exception as exc:   # keep the eager figure if the capture is refused
            log(f"graph capture failed ({exc}); keeping the eager time")
            ms_per_step = eager_ms
        ctx.eoq_profile(True)

    att = {"softmax": 0.0, "attend": 0.0}
    prod = {"qjl": 0.0, "scores_prod": 0.0}
    if not args.no_extras:
        # decode attention on the same compressed blocks taken as values (outside the timed step: the step and `value`
        # stay the compress + decompress + scores path): softmax of the logits in place, then the fused attention output
        att_ws = torch.empty(max(ctx.eoq_attend_workspace_bytes(n_seq, n_kv, bph), 16), dtype=torch.uint8, device=dev)
        att_out = torch.empty(n_seq, n_kv * group, D, dtype=torch.float32, device=dev)
        for it in range(args.warmup + args.steps):
            ctx.eoq_scores(keys, q, n_kv, scores)
            ctx.eoq_softmax(scores)
            ctx.eoq_attend(keys, scores, n_kv, bph, bph, att_out, att_ws)
            ms = ctx.eoq_stage_ms()
            if it >= args.warmup:
                for k_ in att:
                    att[k_] += ms[k_] / args.steps
        torch.cuda.synchronize()
        # TQ_prod (optional 1-bit correction of Eq. (qjl)), also outside the timed step: side information of the whole
        # batch, then the corrected scores on the key set.  The library launches on torch's current stream, which these
        # events see.
        qj = eoq.Qjl.empty(B, n, D, dev)
        kq = eoq.Qjl(qj.signs[:key_blocks], qj.norms[:key_blocks])
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
        reps = min(args.steps, 5)
        for it in range(1 + reps):
            ev[0].record()
            ctx.eoq_qjl_encode(blocks, rec, qj)
            ev[1].record()
            ctx.eoq_scores_prod(keys, kq, q, n_kv, scores)
            ev[2].record()
            torch.cuda.synchronize()
            if it >= 1:
                prod["qjl"] += ev[0].elapsed_time(ev[1]) / reps
                prod["scores_prod"] += ev[1].elapsed_time(ev[2]) / reps
        del qj, kq, att_ws

    in_bytes = B * n * D * 2
    flags = rec.flags.cpu()
    sweeps = ((flags >> 8) & 0xFF).double().mean().item()
    ranks = rec.rank.cpu().double()
    mean_rank = ranks.mean().item()
    # bytes a stored record needs: residual codes, norms, the factors (binary16, or 4-bit codes + binary16 phi per
    # component + two 8-level binary16 codebooks per block), rank / flags
    comp_bytes = (n + D) * 2 if fq is None else (n + D) // 2 + 2
    book_bytes = 0 if fq is None else 32
    rec_bytes = (B * n * (bits * D // 8) + B * n * 2 + int(ranks.sum().item()) * comp_bytes + B * (12 + book_bytes))
    # the decoder and the scores read the expanded binary16 factors in either case
    moved_bytes = B * n * (bits * D // 8) + B * n * 2 + int(ranks.sum().item()) * (n + D) * 2 + B * 12
    fp64_flops = spectral_fp64_flops_per_block(n, mean_rank, sweeps) * B
    achieved_tflops = fp64_flops / (stage["spectral"] * 1e-3) / 1e12
    gram_tops = gram_int8_ops_per_block(n) * B / (stage["spectral"] * 1e-3) / 1e12 if sweeps == 0 else 0.0
    compress_ms = stage["spectral"] + stage["encode"]
    compress_alg_bytes = compress_bytes_per_block(n, bits, mean_rank) * B
    traffic, traffic_src = None, None
    tfile = os.path.join(ROOT, "profiles", f"traffic_spectral_{args.workload}.txt")
    if os.path.exists(tfile) and bits == 2 and fq is None:
        for line in open(tfile):
            if line.startswith("traffic_bytes_per_launch"):
                traffic = float(line.split("=")[1])
                traffic_src = (f"profiles/traffic_spectral_{args.workload}.txt: FETCH_SIZE and WRITE_SIZE of two rocprofv3 "
                               f"--pmc runs of this command, scaled by a plain copy dispatch of the same run")
    key_rec_bytes = key_blocks * n * (bits * D // 8 + 2) + int(ranks[:key_blocks].sum().item()) * (n + D) * 2
    score_bytes = key_rec_bytes + scores.numel() * 4
    kernel = "eoq_spectral_jacobi_kernel" if sweeps > 0 else "eoq_spectral_tridiag_kernel"
    out = {
        "metric": "KV compress GB/s (fp16 in) at d=128, 2-bit; dequant GB/s; % of roofline",
        "value": in_bytes / (ms_per_step * 1e-3) / 1e9,
        "unit": "GB/s",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": ms_per_step,
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f16+f64",      # binary16 in and out, f16 / int8 matrix-core products, double-precision eigensolve
        "data": "synthetic",
        "config": {"workload": f"{spec.name}: {B} blocks of {n}x{D} fp16, b={bits}, whole path per step "
                               f"(compress + decompress + scores of {n_seq}x{n_kv * group} queries on "
                               f"{key_blocks} key blocks)",
                   "blocks": B, "n": n, "d": D, "bits": bits, "factor_bits": args.factor_bits, "input_bytes": in_bytes},
        "stages": {
            "compress_ms": compress_ms,
            "compress_GBps_fp16_in": in_bytes / (compress_ms * 1e-3) / 1e9,
            # the three rooflines of compress, each with what the method must do on that unit over the time taken:
            # double-precision vector flops of the eigensolve (spectral kernel), integer matrix-core operations of the
            # exact Gram matrix (spectral kernel), algorithmic HBM bytes of the whole call
            "compress_frac_fp64_alu": achieved_tflops / FP64_VECTOR_PEAK_TFLOPS,
            "compress_frac_int8_mfma": gram_tops / INT8_MFMA_PEAK_TOPS,
            "compress_frac_hbm": compress_alg_bytes / (compress_ms * 1e-3) / 1e9 / HBM_PEAK_GBPS,
            "spectral_ms": stage["spectral"], "encode_ms": stage["encode"],
            "encode_GBps_moved": (in_bytes + moved_bytes) / (stage["encode"] * 1e-3) / 1e9,
            "encode_frac_hbm": (in_bytes + moved_bytes) / (stage["encode"] * 1e-3) / 1e9 / HBM_PEAK_GBPS,
            "dequant_ms": stage["decode"],
            "dequant_GBps_out": in_bytes / (stage["decode"] * 1e-3) / 1e9,
            "dequant_GBps_moved": (in_bytes + moved_bytes) / (stage["decode"] * 1e-3) / 1e9,
            "dequant_frac_hbm": (in_bytes + moved_bytes) / (stage["decode"] * 1e-3) / 1e9 / HBM_PEAK_GBPS,
            "scores_ms": stage["scores"],
            "scores_GBps_moved": score_bytes / (stage["scores"] * 1e-3) / 1e9,
            "scores_frac_hbm": score_bytes / (stage["scores"] * 1e-3) / 1e9 / HBM_PEAK_GBPS,
            "eager_ms_per_step": eager_ms, "graph_replay": graphed,
            "mean_rank": mean_rank, "mean_jacobi_sweeps": sweeps,
            "record_bytes": rec_bytes, "stored_bits_per_entry": rec_bytes * 8.0 / (B * n * D),
            "targets": {"compress_frac_of_binding_roofline": 0.5, "dequant_frac_hbm": 0.7, "scores_frac_hbm": 0.7},
        },
        "roofline": {"kernel": kernel, "bound": "alu", "achieved": achieved_tflops,
                     "peak": FP64_VECTOR_PEAK_TFLOPS, "unit": "TFLOP/s", "frac": achieved_tflops / FP64_VECTOR_PEAK_TFLOPS,
                     "traffic": traffic, "traffic_source": traffic_src,
                     "note": "double-precision vector flops of tridiagonalisation + eigenvalues + vectors only; the Gram "
                             "matrix runs on the int8 matrix cores (stages.compress_frac_int8_mfma)"},
    }
    if not args.no_extras:
        out["stages"].update({
            "qjl_encode_ms": prod["qjl"], "scores_prod_ms": prod["scores_prod"],
            "softmax_ms": att["softmax"], "attend_ms": att["attend"],
            "attend_GBps_moved": score_bytes / (att["attend"] * 1e-3) / 1e9,
            "attend_frac_hbm": score_bytes / (att["attend"] * 1e-3) / 1e9 / HBM_PEAK_GBPS})
        log("measuring the device ceilings")
        out["ceilings"] = measure_ceilings(ctx, torch, dev)
        out["ceilings"]["datasheet"] = {"hbm_GBps": HBM_PEAK_GBPS, "fp64_vector_TFLOPs": FP64_VECTOR_PEAK_TFLOPS,
                                        "mfma_f16_TFLOPs": 2500.0, "mfma_i8_TOPs": INT8_MFMA_PEAK_TOPS,
                                        "mfma_f64_TFLOPs": 78.6}
    blocks_cpu = blocks[:args.cpu_blocks].cpu() if args.cpu_blocks > 0 else None
    q_cpu = q[0, :group].cpu()
    if not args.no_extras and cfg == 3 and bits == 2 and fq is None:
        # the other figures the benchmark definition asks for: the same cache at b = 3, and one Ministral-8B-shaped
        # layer (2048 blocks of 1024 x 128, ranks 1..12, 10 % pure noise); eager, per-kernel events
        log("config 3 at b = 3")
        del rec, keys, ws
        ctx3 = eoq.Context(n=n, bits=3)
        out["stages"]["cfg3_b3"] = time_codec(ctx3, torch, eoq, blocks, 3, 3, 1)
        del ctx3, blocks, xhat
        torch.cuda.empty_cache()
        log("config 4: one layer")
        spec4 = synth.config(4)
        blocks4, _ = synth.make_blocks(spec4, device=dev)
        ctx4 = eoq.Context(n=spec4.n, bits=2)
        out["stages"]["cfg4_layer"] = time_codec(ctx4, torch, eoq, blocks4, 2, 5, 2)
        del ctx4, blocks4
        torch.cuda.empty_cache()
    if blocks_cpu is not None:
        log("timing the CPU oracle")
        out["cpu_baseline"] = cpu_baseline(blocks_cpu, bits, ctx.rot_seed, q_cpu, args.cpu_blocks, args.cpu_passes,
                                           args.factor_bits)
        log("CPU oracle done")
    print(json.dumps(out))
    return 0


if __name__ == "__main__":
    sys.exit(main())
