#!/usr/bin/env python3
"""Benchmark of the intercept hot path on one MI355X.

One step = one pass of the whole hot path over one synthetic batch:
    paged_attn_mixed over the 13B-shaped mixed batch (128 decode sequences + 8 recomputation
    chunks of 512 rows), then kv_pack_blocks and kv_unpack_blocks of 2000 scattered 320 KiB
    blocks (the 13B-shaped swap).
Inputs are resident in HBM before the timed region; the per-call descriptor upload is inside it.
Prints ONE JSON line.  `python bench.py --gpus N` with N > 1 exits: this path runs on one GPU.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

import numpy as np

HBM_PEAK_GBPS = 8000.0        # MI355X HBM3E, vendor figure
# HBM bytes per launch of the dominant kernel, from rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE runs of this same
# command, scaled by the pack kernel's known 640 000 KiB (FETCH_SIZE x 2.0, WRITE_SIZE x 1.0 on this GPU);
# figures and commands in the profiles/ file named next to each.  Only valid for the default launch plan of
# these workloads; the JSON line says where the figure comes from (`traffic_source`).
MEASURED_TRAFFIC = {"mixed_13b/row": ((2816595 * 2.0 + 1448) * 1024, "profiles/row_and_tile_persist_kernels_mixed_13b.md"),
                    "gptj_decode/row": ((660150 * 2.0 + 560) * 1024, "profiles/row_persist_kernel_gptj_decode.md"),
                    "gptj_mixed/tile": ((156760 * 2.0 + 32824) * 1024, "profiles/tile_and_row_kernels_gptj_mixed.md"),
                    "gptj_mixed/row": ((635491 * 2.0 + 552) * 1024, "profiles/tile_and_row_kernels_gptj_mixed.md"),
                    "gqa_70b/group": ((544853 * 2.0 + 5416) * 1024, "profiles/group_and_tile_kernels_gqa_70b.md"),
                    "gqa_70b/tile": ((123847 * 2.0 + 65579) * 1024, "profiles/group_and_tile_kernels_gqa_70b.md"),
                    "long_ctx/tile": ((5353236 * 2.0 + 262731) * 1024, "profiles/tile_persist_kernel_long_ctx.md")}
SWAP_LOOP, SWAP_REPS = 50, 7   # pack / unpack timing: launches per event pair, loops
MFMA_BF16_PEAK_TFLOPS = 2500.0  # dense bf16, vendor figure


def parse_args():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=100)
    ap.add_argument("--warmup", type=int, default=50)
    ap.add_argument("--workload", default="mixed_13b",
                    choices=["mixed_13b", "gptj_decode", "long_ctx", "tiny", "gqa_70b", "gptj_mixed"])
    ap.add_argument("--clock-ramp", type=float, default=0.4,
                    help="seconds of untimed back-to-back steps before the warm-up steps (GPU clocks ramp after an idle gap)")
    ap.add_argument("--no-other-configs", action="store_true",
                    help="skip the short timing of the other attention configurations after the main workload")
    ap.add_argument("--decode-part", type=int, default=0)
    ap.add_argument("--span-part", type=int, default=0)
    ap.add_argument("--span-kernel", type=int, default=0)
    ap.add_argument("--row-variant", type=int, default=0)
    ap.add_argument("--serial-spans", type=int, default=0)
    ap.add_argument("--row-launch", type=int, default=0)
    ap.add_argument("--row-slots", type=int, default=0)
    ap.add_argument("--mode", default="hot_path", choices=["hot_path", "swap_pipeline", "saturation", "ceilings"],
                    help="hot_path: the step described above (default); swap_pipeline: the layer-pipelined "
                         "swap to pinned host memory, alone and behind the attention call; saturation: "
                         "T_fwd profile of the attention call against query tokens, saturation point, waste model")
    ap.add_argument("--layers", type=int, default=8, help="swap_pipeline: layers (pools) moved per call")
    ap.add_argument("--swap-blocks", type=int, default=512, help="swap_pipeline: blocks per layer per call")
    ap.add_argument("--stages", type=int, default=2, help="swap_pipeline: staging buffers")
    ap.add_argument("--no-swap", action="store_true", help="time the attention call only")
    ap.add_argument("--decode-only", action="store_true", help="drop the recomputation spans from the batch")
    ap.add_argument("--no-append", action="store_true", help="skip the kv_write_span timing after the steps")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--cpu-seconds", type=float, default=20.0, help="target oracle time for the CPU sample")
    return ap.parse_args()


def cpu_baseline(batch, pool_t, q_bits, target_s):
    """Time the fp64 oracle (as it stands) on a bounded sample of the same batch, on the host cores.

    The sample is sized from a short calibration run so that it costs about target_s seconds."""
    import torch
    import oracle
    from paper_2402_01869_amd import workloads as W

    def fetch(ids):
        idx = torch.from_numpy(np.asarray(ids)).to(pool_t.device)
        return pool_t.view(torch.int16)[idx].cpu().numpy().view(np.uint16)

    def run(items):
        seqs = sorted({s for s, _ in items})
        remap = {s: j for j, s in enumerate(seqs)}
        small, sub = W.compact_referenced(batch, seqs, fetch)
        iseq = np.array([remap[s] for s, _ in items], dtype=np.int32)
        irow = np.array([i for _, i in items], dtype=np.int32)
        t0 = time.perf_counter()
        oracle.paged_attn_items(small, sub.ctx_len, sub.q_len, sub.q_start, sub.block_tables, q_bits, sub.scale,
                                iseq, irow)
        return time.perf_counter() - t0

    def keys_of(items):
        return int(sum(int(batch.ctx_len[s]) - int(batch.q_len[s]) + i + 1 for s, i in items))

    rng = np.random.default_rng(1)
    # candidate rows in a fixed random order: all decode rows, then random span rows
    dec = [(s, 0) for s in range(batch.num_seqs) if batch.q_len[s] == 1]
    span = [(s, int(i)) for s in range(batch.num_seqs) if batch.q_len[s] > 1
            for i in rng.permutation(int(batch.q_len[s]))]
    cand = dec + [span[i] for i in rng.permutation(len(span))]
    probe = cand[:max(32, oracle.num_threads() * 2)]
    run(probe[:4])                       # page in the library and the thread pool
    dt = run(probe)
    rate = keys_of(probe) / max(dt, 1e-6)
    items, used = [], 0
    for it in cand:
        k = keys_of([it])
        if items and used + k > rate * target_s:
            break
        items.append(it); used += k
    dt = run(items)
    n_dec = sum(1 for s, _ in items if batch.q_len[s] == 1)
    return {"value": round(used * batch.token_bytes / dt / 1e9, 3), "unit": "GB/s", "cores": oracle.num_threads(),
            "kind": "oracle", "seconds": round(dt, 3),
            "sample": f"{n_dec} decode rows + {len(items) - n_dec} span rows of the same batch "
                      f"({used} visible keys x {batch.token_bytes} B of KV per key, counted once per row)"}


def swap_pipeline_bench(args):
    """Section 4.1 on this machine: L layers' blocks gathered, moved over the host link and scattered
    back, layer by layer; first alone, then while the 13B-shaped attention call runs in a loop."""
    import torch
    from paper_2402_01869_amd import binding as B
    from paper_2402_01869_amd import workloads as W

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    acfg, scfg = W.MIXED_13B, W.KV_SWAP
    H, D, L, n = acfg.num_heads, acfg.head_dim, args.layers, args.swap_blocks
    bb = scfg.block_bytes
    lay_blocks = max(4 * n, 2048)
    rng = np.random.default_rng(scfg.seed)
    lay_t = []
    for l in range(L):
        t = torch.empty((lay_blocks, bb), dtype=torch.uint8, device=dev)
        W.fill_bytes_device(t, scfg.seed + l)
        lay_t.append(t)
    lay = [B.KvPool(B.make_cfg(lay_blocks, H, D), t.data_ptr(), t.numel()) for t in lay_t]
    need = B.LayerSwapper.staging_bytes(lay[0], L, n, args.stages)
    staging = torch.empty(need, dtype=torch.uint8, device=dev)
    sw = B.LayerSwapper(lay, n, staging.data_ptr(), need, args.stages)
    perm = rng.permutation(lay_blocks).astype(np.int32)
    src, dst = perm[:n], perm[n:2 * n]
    pin = B.PinnedBuffer(L * n * bb)
    moved = float(L) * n * bb
    reps = max(3, min(args.steps, 10))

    def timed(fn):
        fn(); sw.sync()
        ts = []
        for _ in range(reps):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            fn(); sw.sync()
            ts.append(time.perf_counter() - t0)
        return float(np.median(ts)), float(np.min(ts))

    out_med, out_min = timed(lambda: sw.swap_out(src, pin.ptr, n * bb))
    in_med, in_min = timed(lambda: sw.swap_in(dst, pin.ptr, n * bb))

    # link ceiling: one contiguous copy of the same size, device <-> the same pinned memory
    flat = torch.empty(int(moved), dtype=torch.uint8, device=dev)
    pin_t = torch.from_numpy(pin.array)

    def copy_time(d2h):
        ts = []
        for _ in range(reps + 1):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            if d2h:
                pin_t.copy_(flat, non_blocking=True)
            else:
                flat.copy_(pin_t, non_blocking=True)
            torch.cuda.synchronize()
            ts.append(time.perf_counter() - t0)
        return float(np.median(ts[1:]))
    d2h_s, h2d_s = copy_time(True), copy_time(False)

    # attention loop alone, then with swaps queued behind it
    pool_t = torch.empty(W.pool_shape(acfg.pool_blocks, H, 16, D), dtype=torch.bfloat16, device=dev)
    W.fill_pool_device_normal(pool_t, acfg.seed)
    pool = B.KvPool.from_tensor(pool_t, H, D)
    batch = W.make_batch(acfg, acfg.seed)
    desc = B.HostDesc.from_batch(batch, flags=0)
    q = torch.from_numpy(W.randn_bf16((batch.total_q_rows, H, D), np.random.default_rng(1)).view(np.int16)).to(dev)
    out = torch.zeros_like(q)
    ws = torch.empty(pool.workspace_bytes(desc), dtype=torch.uint8, device=dev)
    stream = torch.cuda.current_stream().cuda_stream
    pool.paged_attn_mixed(desc, q.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), stream)
    desc.struct.flags = B.IC_FLAG_TRUSTED

    cur = torch.cuda.current_stream()

    def attn_loop(k, period, swap_fn=None):
        """k attention calls on the caller's stream; with period > 0 a swap-out of all layers is handed to
        the swapper before every period-th call (one chunk per iteration, as the scheduler would), so the
        link is busy for the whole loop -> (ms per attention call, swaps queued, seconds until they are
        through, average kernel times from a second pass with an event pair around every kernel)."""
        def one_pass():
            n_sw = 0
            for i in range(k):
                if period and i % period == 0:
                    swap_fn()
                    n_sw += 1
                pool.paged_attn_mixed(desc, q.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), stream)
            cur.synchronize()                  # the caller's stream only: the swapper has its own
            return n_sw
        for i in range(args.warmup):
            pool.paged_attn_mixed(desc, q.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), stream)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        n_sw = one_pass()
        t1 = time.perf_counter()
        sw.sync()
        t2 = time.perf_counter()
        pool.prof_begin(5 * k + 8)
        one_pass()
        pr = pool.prof_end()
        sw.sync()
        kern = {a: round(pr[a]["total_ms"] / pr[a]["launches"], 4) for a in ("upload", "row", "tile", "merge") if pr[a]["launches"]}
        return (t1 - t0) * 1e3 / k, n_sw, t2 - t0, kern

    k = max(args.steps, 100)
    alone_ms, _, _, alone_kern = attn_loop(k, 0)
    period = max(1, int(out_med * 1e3 / alone_ms))       # attention calls that fit in one swap
    behind_ms, n_swaps, swap_s, behind_kern = attn_loop(k, period, lambda: sw.swap_out(src, pin.ptr, n * bb))
    in_ms, n_in, in_s, in_kern = attn_loop(k, period, lambda: sw.swap_in(dst, pin.ptr, n * bb))
    link = moved / out_med
    token_bytes = acfg.token_bytes          # one layer's M; t_fwd below is one layer's attention call
    result = {
        "metric": "layer-pipelined KV swap over the host link, GB/s", "value": round(moved / out_med / 1e9, 2),
        "unit": "GB/s", "n_gpus": 1, "steps": reps, "warmup": 1, "ms_per_step": round(out_med * 1e3, 3),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "u8", "data": "synthetic",
        "config": {"workload": f"swap pipeline: {L} layers x {n} blocks x {bb // 1024} KiB (13B-shaped layer), "
                               f"{args.stages} staging buffers, pools of {lay_blocks} blocks"},
        "swap_out": {"bytes": moved, "median_ms": round(out_med * 1e3, 3), "min_ms": round(out_min * 1e3, 3),
                     "GBps": round(moved / out_med / 1e9, 2),
                     "frac_of_contiguous_copy": round(d2h_s / out_med, 4)},
        "swap_in": {"bytes": moved, "median_ms": round(in_med * 1e3, 3), "min_ms": round(in_min * 1e3, 3),
                    "GBps": round(moved / in_med / 1e9, 2),
                    "frac_of_contiguous_copy": round(h2d_s / in_med, 4)},
        "contiguous_copy": {"d2h_GBps": round(moved / d2h_s / 1e9, 2), "h2d_GBps": round(moved / h2d_s / 1e9, 2)},
        "behind_attention": {"attn_calls": k, "attn_ms_alone": round(alone_ms, 4),
                             "attn_ms_with_swap_out_running": round(behind_ms, 4),
                             "attn_slowdown": round(behind_ms / alone_ms - 1.0, 4),
                             "kernel_ms_alone": alone_kern, "kernel_ms_with_swap_out_running": behind_kern,
                             "swap_outs_queued": n_swaps, "attn_calls_per_swap_out": period,
                             "swap_out_GBps_meanwhile": round(n_swaps * moved / swap_s / 1e9, 2),
                             "attn_ms_with_swap_in_running": round(in_ms, 4),
                             "attn_slowdown_swap_in": round(in_ms / alone_ms - 1.0, 4),
                             "kernel_ms_with_swap_in_running": in_kern,
                             "swap_in_GBps_meanwhile": round(n_in * moved / in_s / 1e9, 2)},
        "swap_limit": {"t_fwd_s": round(alone_ms * 1e-3, 6), "link_bytes_per_s": round(link, 0),
                       "token_bytes": token_bytes,
                       "tokens_per_iteration": B.swap_limit_tokens(alone_ms * 1e-3, link, token_bytes),
                       "note": "t_fwd is one layer's attention call and token_bytes one layer's M: the ratio "
                               "equals the whole model's if every layer behaves alike"},
    }
    print(json.dumps(result))


def ceilings_bench(args):
    """What an MFMA-only loop reaches on this GPU (ic_mfma_ceiling) with zero, one and random N(0,1) bf16 operands:
    context for the tile kernel's fraction of the vendor peak."""
    import torch
    from paper_2402_01869_amd import binding as B
    from paper_2402_01869_amd import workloads as W
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    sink = torch.empty(B.IC_CEILING_SINK_BYTES, dtype=torch.uint8, device=dev)
    n16 = B.IC_CEILING_OPERAND_BYTES // 2
    rng = np.random.default_rng(7)
    sets = {"zeros": np.zeros(n16, dtype=np.uint16), "ones": np.full(n16, 0x3F80, dtype=np.uint16),
            "random_normal": W.randn_bf16((n16,), rng)}
    out = {}
    for name, bits in sets.items():
        ops = torch.from_numpy(bits.view(np.int16)).to(dev)
        best = None
        for _ in range(3):
            rc, tf, ghz = B.mfma_ceiling(ops.data_ptr(), ops.numel() * 2, sink.data_ptr(), sink.numel(), 200000)
            if rc != B.IC_OK:
                raise RuntimeError(B.strerror(rc))
            if best is None or tf > best[0]:
                best = (tf, ghz)
        out[name] = {"TFLOPs": round(best[0], 1), "shader_GHz": round(best[1], 3),
                     "frac_vendor_peak": round(best[0] / MFMA_BF16_PEAK_TFLOPS, 4)}
    # streaming read and plain copy of 1.25 GiB (the bytes one pack call moves), two buffer pairs alternating
    n = 1280 << 20
    bufs = [torch.empty(n, dtype=torch.uint8, device=dev).random_(0, 256) for _ in range(4)]
    hbm = {}
    for name, mode in (("read", 0), ("copy", 1)):
        best = 0.0
        for rep in range(6):
            src, dst = bufs[2 * (rep & 1)], bufs[2 * (rep & 1) + 1]
            rc, g = B.hbm_ceiling(src.data_ptr(), dst.data_ptr(), n, mode, 5)
            if rc != B.IC_OK:
                raise RuntimeError(B.strerror(rc))
            best = max(best, g)
        hbm[name] = {"GBps": round(best, 1), "frac_vendor_peak": round(best / HBM_PEAK_GBPS, 4)}
    del bufs
    # the decode kernels' access pattern without their arithmetic: the blocks of the 13B-shaped batch's decode
    # sequences (randomly placed) and as many consecutive blocks, tile by tile
    acfg = W.MIXED_13B
    batch = W.make_batch(acfg)
    pool_t = torch.empty(W.pool_shape(acfg.pool_blocks, acfg.num_heads, 16, acfg.head_dim), dtype=torch.bfloat16, device=dev)
    W.fill_pool_device_normal(pool_t, acfg.seed)
    pool = B.KvPool.from_tensor(pool_t, acfg.num_heads, acfg.head_dim)
    ids = np.concatenate([batch.blocks_of(s) for s in range(batch.num_seqs) if batch.q_len[s] == 1]).astype(np.int32)
    sink16 = torch.zeros(16, dtype=torch.uint8, device=dev)
    paged = {}
    for name, lists in (("random_blocks", [ids, ids[::-1].copy()]),
                        ("consecutive_blocks", [np.arange(len(ids), dtype=np.int32),
                                                np.arange(len(ids), 2 * len(ids), dtype=np.int32)])):
        best = 0.0
        for rep in range(6):   # two lists alternate so that no pass finds its blocks in the last-level cache
            best = max(best, pool.paged_read_ceiling(lists[rep & 1], sink16.data_ptr(), 1))
        paged[name] = {"GBps": round(best, 1), "frac_vendor_peak": round(best / HBM_PEAK_GBPS, 4),
                       "bytes": float(len(ids)) * pool.block_bytes}
    pool.close()
    print(json.dumps({"metric": "MFMA-only loop rate, v_mfma_f32_32x32x16_bf16 on register operands", "unit": "TFLOP/s",
                      "n_gpus": 1, "vendor_peak_TFLOPs": MFMA_BF16_PEAK_TFLOPS, "operands": out,
                      "hbm_vendor_peak_GBps": HBM_PEAK_GBPS, "hbm_streaming": hbm,
                      "paged_tile_read_13b_decode_blocks": paged}))


def saturation_bench(args):
    """Section 4.2 on this machine, attention only: time of one layer's attention call for the 13B-shaped
    decode batch plus a growing number of recomputation query tokens -> T_fwd profile, saturation
    point S, chunk size, and the waste of Eq. 1 / Eq. 4 for one interception with this profile."""
    import dataclasses
    import torch
    from paper_2402_01869_amd import binding as B
    from paper_2402_01869_amd import workloads as W

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    base = W.MIXED_13B
    H, D = base.num_heads, base.head_dim
    pool_t = torch.empty(W.pool_shape(base.pool_blocks, H, 16, D), dtype=torch.bfloat16, device=dev)
    W.fill_pool_device_normal(pool_t, base.seed)
    pool = B.KvPool.from_tensor(pool_t, H, D)
    stream = torch.cuda.current_stream().cuda_stream
    sweep = [(0, 0), (1, 64), (1, 128), (1, 256), (1, 512), (2, 512), (3, 512), (4, 512), (6, 512), (8, 512),
             (12, 512), (16, 512), (32, 512), (64, 512), (128, 512)]
    q_tokens, seconds, rows = [], [], []
    for n_span, span_len in sweep:
        cfg = dataclasses.replace(base, n_span=n_span, span_len=span_len)
        batch = W.make_batch(cfg, base.seed)
        desc = B.HostDesc.from_batch(batch, flags=0)
        q = torch.randn((batch.total_q_rows, H, D), device=dev).to(torch.bfloat16)
        out = torch.empty_like(q)
        ws = torch.empty(pool.workspace_bytes(desc), dtype=torch.uint8, device=dev)
        pool.paged_attn_mixed(desc, q.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), stream)
        desc.struct.flags = B.IC_FLAG_TRUSTED
        for timed in (False, True):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(args.steps if timed else args.warmup):
                pool.paged_attn_mixed(desc, q.data_ptr(), out.data_ptr(), ws.data_ptr(), ws.numel(), stream)
            torch.cuda.synchronize()
        dt = (time.perf_counter() - t0) / args.steps
        q_tokens.append(float(batch.total_q_rows)); seconds.append(dt)
        rows.append({"spans": n_span, "span_len": span_len, "query_tokens": batch.total_q_rows,
                     "kv_bytes": batch.kv_bytes(), "ms": round(dt * 1e3, 4),
                     "tokens_per_s": round(batch.total_q_rows / dt, 1)})
    S = B.saturation_point(q_tokens, seconds, 0.95)
    running = base.n_decode
    chunk = B.chunk_tokens(S, running)
    # T_fwd for the waste model: ADDED iteration time against recomputed tokens (profile minus the decode-only point)
    added_tok = [qt - q_tokens[0] for qt in q_tokens[1:]]
    added_s = [max(sc - seconds[0], 0.0) for sc in seconds[1:]]
    table = B.TfwdTable(added_tok, added_s)
    M = float(base.token_bytes)
    dec = W.make_batch(dataclasses.replace(base, n_span=0), base.seed)
    C_other = float(dec.ctx_len.astype(np.int64).sum())
    C = 2560.0                                   # an intercepted request's context (the paper's workloads: 750-2200 tokens mean)
    n_chunks = B.chunk_count(int(C), chunk) if chunk > 0 else -1
    w_discard = B.waste_discard(table, C, C_other, M)
    w_chunk = B.waste_chunked_discard(table, C, C_other, M, max(n_chunks, 1))
    result = {
        "metric": "saturation point S of the attention call (query tokens)", "value": S, "unit": "tokens",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(seconds[-1] * 1e3, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None, "dtype": "bf16", "data": "synthetic",
        "config": {"workload": f"{base.name} decode batch ({base.n_decode} sequences) + k spans of up to 512 rows, "
                               f"H{H} D{D}; attention call of one layer only"},
        "profile": rows, "saturation_frac": 0.95, "saturated_within_profile": bool(S < q_tokens[-1]), "running_tokens": running, "chunk_tokens": chunk,
        "waste_example": {"ctx_tokens": C, "other_tokens": C_other, "token_bytes_one_layer": M,
                          "n_chunks": n_chunks,
                          "waste_discard_byte_s": w_discard, "waste_chunked_discard_byte_s": w_chunk,
                          "chunked_over_discard": round(w_chunk / w_discard, 4) if w_discard > 0 else None,
                          "preserve_breakeven_s": w_chunk / (C * M),
                          "note": "T_fwd = added time of ONE layer's attention call against recomputed tokens; a whole "
                                  "model adds its GEMMs, so S here is an upper bound on the model's"},
    }
    print(json.dumps(result))


class AttnSetup:
    """Device inputs of one attention workload: the pool, two batches (different tables and q) that alternate between
    calls so that no call finds the previous one's keys in the last-level cache, outputs and one workspace."""

    def __init__(self, acfg, args, dev):
        import torch
        from paper_2402_01869_amd import binding as B
        from paper_2402_01869_amd import workloads as W
        self.acfg, self.dev = acfg, dev
        H, D = acfg.num_heads, acfg.head_dim
        self.pool_t = torch.empty(W.pool_shape(acfg.pool_blocks, acfg.kv_heads, 16, D), dtype=torch.bfloat16, device=dev)
        W.fill_pool_device_normal(self.pool_t, acfg.seed, chunk_blocks=4096 if acfg.pool_blocks > (1 << 17) else 2048)
        self.pool = B.KvPool.from_tensor(self.pool_t, H, D, num_kv_heads=acfg.kv_heads)
        self.pool.set_tuning(args.decode_part, args.span_part, args.span_kernel, args.row_variant, args.serial_spans,
                             args.row_launch, args.row_slots)
        self.batches = [W.make_batch(acfg, acfg.seed), W.make_batch(acfg, acfg.seed + 1000)]
        self.descs, self.qs, self.q_bits, self.outs = [], [], [], []
        ws_bytes = 0
        for i, b in enumerate(self.batches):
            d = B.HostDesc.from_batch(b, flags=0)
            q_bits = W.randn_bf16((b.total_q_rows, H, D), np.random.default_rng(acfg.seed + 7 + i))
            self.descs.append(d)
            self.q_bits.append(q_bits)
            self.qs.append(torch.from_numpy(q_bits.view(np.int16)).to(dev))
            self.outs.append(torch.zeros((b.total_q_rows, H, D), dtype=torch.int16, device=dev))
            ws_bytes = max(ws_bytes, self.pool.workspace_bytes(d))
        self.ws = torch.empty(ws_bytes, dtype=torch.uint8, device=dev)
        self.stream = torch.cuda.current_stream().cuda_stream
        # one validated pass (full host checks), then trusted descriptors for the timed loops
        for k in range(2):
            self.call(k)
        torch.cuda.synchronize()
        for d in self.descs:
            d.struct.flags = B.IC_FLAG_TRUSTED
        self.kv_bytes = float(np.mean([b.kv_bytes() for b in self.batches]))
        self.dec_bytes = float(np.mean([int(b.ctx_len[b.q_len == 1].astype(np.int64).sum()) * b.token_bytes
                                        for b in self.batches]))
        self.span_flops = float(np.mean([b.span_flops() for b in self.batches]))

    def call(self, k, desc=None):
        k &= 1
        self.pool.paged_attn_mixed(desc or self.descs[k], self.qs[k].data_ptr(), self.outs[k].data_ptr(),
                                   self.ws.data_ptr(), self.ws.numel(), self.stream)

    def close(self):
        self.pool.close()
        del self.pool_t, self.ws, self.qs, self.outs


def wall_ms(fn, n, warm):
    """Wall time per call of fn(i), i = 0..n-1, after `warm` untimed calls; the GPU is drained on both sides."""
    import torch
    for i in range(warm):
        fn(i)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(n):
        fn(i)
    torch.cuda.synchronize()
    return (time.perf_counter() - t0) * 1e3 / n


def clock_ramp(fn, seconds):
    """Run fn(i) back to back for `seconds` of wall time: after an idle gap the GPU's clocks take tens of milliseconds
    to come up, and calls made meanwhile run up to 20 % slower.  Untimed, separate from the warm-up steps."""
    import torch
    t0, i = time.perf_counter(), 0
    while time.perf_counter() - t0 < seconds:
        for _ in range(8):
            fn(i)
            i += 1
        torch.cuda.synchronize()
    return i


def kernel_table(prof, steps=None):
    out = {}
    for k, v in prof.items():
        if v["launches"]:
            out[k] = {"launches": v["launches"], "avg_ms": round(v["total_ms"] / v["launches"], 5),
                      "min_ms": round(v["min_ms"], 5), "max_ms": round(v["max_ms"], 5)}
    return out


def attention_kernel_names(pool, desc, acfg):
    """Names of the kernels the pool launches for this batch under its tuning, from the planner's own report."""
    from paper_2402_01869_amd import binding as B
    D, how = acfg.head_dim, pool.plan_launches(desc)
    beside = bool(how["side_by_side"])
    row = {B.IC_LAUNCH_SLIM: "row_persist_slim_kernel", B.IC_LAUNCH_PER_ITEM: "row_attn_kernel"}.get(how["row_launch"], "row_persist_kernel")
    tile = f"tile_attn_kernel<{D}>" if how["tile_launch"] == B.IC_LAUNCH_PER_ITEM else f"tile_persist_kernel<{D}, {'true' if beside else 'false'}>"
    group = "group_slim_kernel" if how["group_launch"] == B.IC_LAUNCH_SLIM else f"group_attn_kernel<{D}, {'true' if how['n_split_units'] else 'false'}>"
    return {"row": f"{row}<{D}>", "group": group, "tile": tile, "merge": f"merge_kernel<{D}>",
            "side_by_side": beside, "beside_tile": group if how["group_launch"] else f"{row}<{D}>"}


def attention_report(S, args, steps, warm, default_plan):
    """Times one attention workload: wall time per call, per-kernel HIP-event times, the call's roofline figures and the
    dominant kernel's."""
    acfg, pool = S.acfg, S.pool
    names = attention_kernel_names(pool, S.descs[0], acfg)
    ms = wall_ms(S.call, steps, warm)
    pool.prof_begin(8 * steps + 8)
    ms_ev = wall_ms(S.call, steps, 0)
    prof = pool.prof_end()
    kern = kernel_table({k: prof[k] for k in ("upload", "row", "group", "tile", "merge")})
    roofline_ms = max(S.kv_bytes / (HBM_PEAK_GBPS * 1e9), S.span_flops / (MFMA_BF16_PEAK_TFLOPS * 1e12)) * 1e3
    rep = {"workload": f"{acfg.name}: {acfg.n_decode} decode + {acfg.n_span}x{acfg.span_len}-row spans, H{acfg.num_heads}"
                       f"{'/' + str(acfg.kv_heads) if acfg.kv_heads != acfg.num_heads else ''} D{acfg.head_dim}, "
                       f"pool {acfg.pool_blocks} blocks",
           "calls": steps, "ms": round(ms, 4), "ms_with_kernel_events": round(ms_ev, 4),
           "kv_bytes": S.kv_bytes, "kv_read_GBps": round(S.kv_bytes / (ms * 1e-3) / 1e9, 1),
           "frac_hbm_peak": round(S.kv_bytes / (ms * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4),
           "span_flops": S.span_flops, "roofline_time_ms": round(roofline_ms, 4),
           "roofline_frac": round(roofline_ms / ms, 4),
           "bound": "mfma" if S.span_flops / (MFMA_BF16_PEAK_TFLOPS * 1e12) > S.kv_bytes / (HBM_PEAK_GBPS * 1e9) else "hbm",
           "side_by_side": names["side_by_side"],
           "kernels": {names.get(k, k): v for k, v in kern.items()}}
    tile_ms = kern.get("tile", {}).get("avg_ms")
    if tile_ms:
        rep["span_mfma_frac"] = round(S.span_flops / (tile_ms * 1e-3) / 1e12 / MFMA_BF16_PEAK_TFLOPS, 4)
    # dominant kernel: the longest of the call's kernels, priced against the roofline that bounds IT
    cand = {k: kern[k]["avg_ms"] for k in ("row", "group", "tile") if k in kern}
    dom = max(cand, key=cand.get)
    rep["dominant_kernel"] = names[dom]
    tkey = f"{acfg.name}/{dom}"
    traffic = MEASURED_TRAFFIC.get(tkey) if default_plan else None
    if dom == "tile":
        ach = S.span_flops / (cand[dom] * 1e-3) / 1e12
        roof = {"kernel": names[dom], "runs_beside": names["beside_tile"] if names["side_by_side"] else None, "bound": "mfma",
                "achieved": round(ach, 1), "peak": MFMA_BF16_PEAK_TFLOPS, "unit": "TFLOP/s",
                "frac": round(ach / MFMA_BF16_PEAK_TFLOPS, 4), "flops_per_launch": S.span_flops}
    else:
        # its algorithmic bytes: the KV of the sequences it serves, each context once (everything if no tile kernel runs)
        dom_bytes = S.kv_bytes if "tile" not in kern else S.dec_bytes
        ach = dom_bytes / (cand[dom] * 1e-3) / 1e9
        roof = {"kernel": names[dom], "runs_beside": names["tile"] if names["side_by_side"] else None, "bound": "hbm",
                "achieved": round(ach, 1), "peak": HBM_PEAK_GBPS, "unit": "GB/s", "frac": round(ach / HBM_PEAK_GBPS, 4),
                "bytes_per_launch": dom_bytes}
    roof["avg_launch_ms"] = cand[dom]
    roof["traffic"] = traffic[0] if traffic else None
    roof["traffic_source"] = (f"{traffic[1]} (rocprofv3 --pmc FETCH_SIZE / WRITE_SIZE of an earlier run of this command, "
                              "calibrated on the pack kernel; not measured by this run)") if traffic else None
    rep["roofline"] = roof
    return rep, prof


def main():
    args = parse_args()
    if args.gpus != 1:
        print("bench.py: this hot path runs on ONE GPU (no sharding or collectives are built); "
              "run with --gpus 1", file=sys.stderr)
        sys.exit(2)
    sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
    from paper_2402_01869_amd import binding as B
    B.lib()  # fail loudly if the HIP library is missing
    if args.mode != "hot_path":
        return {"swap_pipeline": swap_pipeline_bench, "saturation": saturation_bench,
                "ceilings": ceilings_bench}[args.mode](args)
    import torch
    from paper_2402_01869_amd import workloads as W

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    acfg = W.ATTN_CONFIGS[args.workload]
    scfg = W.TINY_SWAP if args.workload == "tiny" else W.KV_SWAP
    if args.decode_only:
        import dataclasses
        acfg = dataclasses.replace(acfg, n_span=0)
    H, D = acfg.num_heads, acfg.head_dim
    default_plan = not (args.decode_only or args.decode_part or args.span_part or args.serial_spans or args.span_kernel
                        or args.row_launch or args.row_slots or args.row_variant)

    S = AttnSetup(acfg, args, dev)
    pool, stream = S.pool, S.stream

    # ---- swap inputs: its own pool (config shape), two staging buffers alternated
    do_swap = not args.no_swap
    if do_swap:
        spool_t = torch.empty((scfg.pool_blocks, scfg.block_bytes), dtype=torch.uint8, device=dev)
        W.fill_bytes_device(spool_t, scfg.seed)
        spool = B.KvPool(B.make_cfg(scfg.pool_blocks, scfg.num_heads, scfg.head_dim), spool_t.data_ptr(), spool_t.numel())
        src, dst = W.make_swap_lists(scfg)
        stagings = [torch.empty((scfg.n_move, scfg.block_bytes), dtype=torch.uint8, device=dev) for _ in range(2)]
        sbytes = stagings[0].numel()
        for st_ in stagings:
            spool.kv_pack_blocks(src, st_.data_ptr(), sbytes, stream)

    def step(i):
        k = i & 1
        S.call(k)
        if do_swap:
            spool.kv_pack_blocks(src, stagings[k].data_ptr(), sbytes, stream)
            spool.kv_unpack_blocks(dst, stagings[k ^ 1].data_ptr(), sbytes, stream)

    # Per-kernel HIP events are created now (and switched off again) so that nothing but a
    # synchronize sits between the loops below.
    pool.prof_begin(8 * args.steps + 8)
    pool.prof_end()
    if do_swap:
        spool.prof_begin(4 * args.steps + 8)
        spool.prof_end()

    ramp_steps = clock_ramp(step, args.clock_ramp)
    for i in range(args.warmup):
        step(i)
    torch.cuda.synchronize()

    # ---- loop 1: EXACTLY K steps, nothing but the three calls per step -> ms_per_step, value
    t0 = time.perf_counter()
    for i in range(args.steps):
        step(i)
    torch.cuda.synchronize()
    ms_per_step = (time.perf_counter() - t0) * 1e3 / args.steps

    # ---- loop 2: K more steps with a HIP event pair around every kernel, recorded by the library on
    # the stream each kernel is launched on -> average launch durations
    pool.prof_begin(8 * args.steps + 8)
    if do_swap:
        spool.prof_begin(4 * args.steps + 8)
    ms_per_step_events = wall_ms(step, args.steps, 0)
    step_prof = pool.prof_end()
    if do_swap:
        sp = spool.prof_end()
        step_prof["pack"], step_prof["unpack"] = sp["pack"], sp["unpack"]

    # ---- loop 3: the attention call alone (kernels overlap inside it): wall time, per-kernel events, roofline
    attn, _ = attention_report(S, args, args.steps, min(10, args.steps), default_plan)

    # ---- loop 3b: the same calls from descriptor images planned and uploaded once (what the layers after the
    # first do in an iteration: kernel launches only)
    plans, plan_ws = [], []
    for k in range(2):
        w = torch.empty(pool.workspace_bytes(S.descs[k]), dtype=torch.uint8, device=dev)
        plan_ws.append(w)
        plans.append(pool.plan_create(S.descs[k], w.data_ptr(), w.numel(), stream))
    attn_planned_ms = wall_ms(lambda i: pool.paged_attn_planned(plans[i & 1], S.qs[i & 1].data_ptr(),
                                                                S.outs[i & 1].data_ptr(), stream),
                              args.steps, min(10, args.steps))
    for pl in plans:
        pl.close()

    # ---- loop 4: the decode sequences alone and the recomputation spans alone (same tables, same q rows)
    def sub_call_ms(pick):
        subs = []
        for b in S.batches:
            sel = np.nonzero(pick(b))[0]
            if len(sel) == 0:
                return None
            subs.append(B.HostDesc(b.ctx_len[sel], b.q_len[sel], b.q_start[sel], b.block_tables[sel], b.scale,
                                   total_q_rows=b.total_q_rows, flags=B.IC_FLAG_TRUSTED))
            need = pool.workspace_bytes(subs[-1])   # a part may be split over keys where the whole batch is not
            if need > S.ws.numel():
                S.ws = torch.empty(need, dtype=torch.uint8, device=dev)
        n = max(10, args.steps // 2)
        return wall_ms(lambda i: S.call(i, subs[i & 1]), n, n)

    decode_alone_ms = sub_call_ms(lambda b: b.q_len == 1)
    spans_alone_ms = sub_call_ms(lambda b: b.q_len > 1)

    # ---- loop 5: pack and unpack, each in loops of its own: SWAP_LOOP launches back to back inside ONE HIP event
    # pair on the launch stream, two staging buffers alternating; several such loops, the median loop reported
    swap = {}
    swap_moved = 2.0 * scfg.n_move * scfg.block_bytes if do_swap else 0.0   # read + write, per call
    if do_swap:
        # a second pair of lists (the other way round), for loops in which no call finds its list already on the device
        lists = {"pack": [src, dst], "unpack": [dst, src]}
        calls = {"pack": lambda i, ids: spool.kv_pack_blocks(ids, stagings[i & 1].data_ptr(), sbytes, stream),
                 "unpack": lambda i, ids: spool.kv_unpack_blocks(ids, stagings[i & 1].data_ptr(), sbytes, stream)}

        def loop_ms(fn, pick):
            for i in range(10):
                fn(i, pick(i))
            per_launch = []
            for rep in range(SWAP_REPS):
                e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                e0.record()
                for i in range(SWAP_LOOP):
                    fn(i, pick(i))
                e1.record()
                e1.synchronize()
                per_launch.append(e0.elapsed_time(e1) / SWAP_LOOP)
            return float(np.median(per_launch)), float(min(per_launch))

        for name, fn in calls.items():
            med, best = loop_ms(fn, lambda i: lists[name][0])                 # one list, call after call (a swap's layers)
            med_new, _ = loop_ms(fn, lambda i: lists[name][i & 1])            # a new list every call
            g = swap_moved / (med * 1e-3) / 1e9
            kavg = step_prof[name]["total_ms"] / step_prof[name]["launches"]
            swap[name] = {"moved_bytes": swap_moved, "GBps": round(g, 1), "frac_hbm_peak": round(g / HBM_PEAK_GBPS, 4),
                          "ms_per_call_median": round(med, 5), "ms_per_call_min": round(best, 5),
                          "timing": f"median of {SWAP_REPS} loops of {SWAP_LOOP} back-to-back calls, one HIP event pair around "
                                    "each loop on the launch stream; every call brings the same id list, as the layers of one "
                                    "swap do, so the library uploads it once and a call is the one gather / scatter launch",
                          "new_list_every_call": {"ms_per_call_median": round(med_new, 5),
                                                  "GBps": round(swap_moved / (med_new * 1e-3) / 1e9, 1),
                                                  "frac_hbm_peak": round(swap_moved / (med_new * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4),
                                                  "note": "a call = id-list upload + the launch"},
                          "kernel_avg_ms_in_step": round(kavg, 5),
                          "kernel_GBps_in_step": round(swap_moved / (kavg * 1e-3) / 1e9, 1)}

    # ---- loop 6 (outside the step): kv_write_span of the same batches, the step that precedes the attention call in
    # an iteration; the rows written are random, the attention outputs above were already taken
    append = None
    if not args.no_append:
        kn = [torch.randn((b.total_q_rows, acfg.kv_heads, D), device=dev).to(torch.bfloat16) for b in S.batches]
        vn = [torch.randn((b.total_q_rows, acfg.kv_heads, D), device=dev).to(torch.bfloat16) for b in S.batches]
        n_ap = max(10, args.steps // 2)
        for timed in (False, True):
            if timed:
                pool.prof_begin(2 * n_ap + 8)
            for i in range(n_ap):
                k = i & 1
                pool.kv_write_span(S.descs[k], kn[k].data_ptr(), vn[k].data_ptr(), stream)
            torch.cuda.synchronize()
        ap = pool.prof_end()["append"]
        ap_ms = ap["total_ms"] / ap["launches"]
        ap_bytes = float(np.mean([2.0 * 2 * b.total_q_rows * acfg.kv_heads * D * 2 for b in S.batches]))   # K and V, read + write
        append = {"rows": int(np.mean([b.total_q_rows for b in S.batches])), "moved_bytes": ap_bytes,
                  "avg_ms": round(ap_ms, 5), "min_ms": round(ap["min_ms"], 5),
                  "GBps": round(ap_bytes / (ap_ms * 1e-3) / 1e9, 1),
                  "frac_hbm_peak": round(ap_bytes / (ap_ms * 1e-3) / 1e9 / HBM_PEAK_GBPS, 4)}
        del kn, vn

    step_bytes = S.kv_bytes + 2 * swap_moved
    attn.update({"planned_ms": round(attn_planned_ms, 4),
                 "planned_kv_read_GBps": round(S.kv_bytes / (attn_planned_ms * 1e-3) / 1e9, 1),
                 "decode_kv_bytes": S.dec_bytes,
                 "decode_alone_ms": None if decode_alone_ms is None else round(decode_alone_ms, 4),
                 "decode_alone_GBps": (None if decode_alone_ms is None else
                                       round(S.dec_bytes / (decode_alone_ms * 1e-3) / 1e9, 1)),
                 "spans_alone_ms": None if spans_alone_ms is None else round(spans_alone_ms, 4),
                 "plan": pool.plan_query(S.descs[0])})
    roofline = attn.pop("roofline")

    result = {
        "metric": "mixed paged-attn KV-read GB/s (% HBM peak); swap pack/unpack GB/s",
        "value": round(step_bytes / (ms_per_step * 1e-3) / 1e9, 1),
        "unit": "GB/s",
        "value_definition": "algorithmic bytes of one step (KV bytes read once per sequence + pack read+write + "
                            "unpack read+write) / wall time of the step",
        "n_gpus": 1, "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms_per_step, 4),
        "clock_ramp_s": args.clock_ramp, "clock_ramp_steps": ramp_steps,
        "ms_per_step_with_kernel_events": round(ms_per_step_events, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": f"{acfg.name} attention ({acfg.n_decode} decode + {acfg.n_span}x{acfg.span_len}-row spans, "
                               f"H{H} D{D}, pool {acfg.pool_blocks} blocks)"
                               + (f" + {scfg.name} ({scfg.n_move} of {scfg.pool_blocks} blocks x {scfg.block_bytes // 1024} KiB)" if do_swap else ""),
                   "decode_part_tokens": args.decode_part, "span_part_tokens": args.span_part, "span_kernel": args.span_kernel},
        "attn": attn,
        "step_kernels": kernel_table({k: step_prof[k] for k in ("upload", "row", "group", "tile", "merge", "pack", "unpack")}),
        "roofline": roofline,
    }
    result.update(swap)
    if append:
        result["kv_write_span"] = append
    if not args.no_cpu_baseline:
        result["cpu_baseline"] = cpu_baseline(S.batches[0], S.pool_t, S.q_bits[0], args.cpu_seconds)

    # ---- the other attention configurations, one after the other (each with its own pool): driver-visible throughput
    # of every config, a few dozen calls each
    if args.workload == "mixed_13b" and default_plan and not args.no_other_configs:
        if do_swap:
            spool.close()
            del spool_t, stagings
        S.close()
        del S
        torch.cuda.empty_cache()
        others = {}
        n_other = max(10, min(args.steps, 30))
        for name in ("gptj_decode", "gptj_mixed", "gqa_70b", "long_ctx"):
            cfg = W.ATTN_CONFIGS[name]
            free, _ = torch.cuda.mem_get_info()
            if free < cfg.pool_blocks * cfg.block_bytes + (8 << 30):
                others[name] = {"skipped": f"needs {cfg.pool_blocks * cfg.block_bytes >> 30} GiB of free HBM"}
                continue
            So = AttnSetup(cfg, args, dev)
            clock_ramp(So.call, min(args.clock_ramp, 0.2))
            others[name], _ = attention_report(So, args, n_other, min(10, n_other), True)
            So.close()
            del So
            torch.cuda.empty_cache()
        result["other_configs"] = others
    print(json.dumps(result))


if __name__ == "__main__":
    main()
