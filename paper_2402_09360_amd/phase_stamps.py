"""Phase stamps of the selecting kernels, read from the profiling build of the library.

    python -m paper_2402_09360_amd.build --timestamps
    HIRE_LIB=$PWD/paper_2402_09360_amd/libhire_ts.so python -m paper_2402_09360_amd.phase_stamps --batch 1
    HIRE_LIB=$PWD/paper_2402_09360_amd/libhire_ts.so python -m paper_2402_09360_amd.phase_stamps --softmax

The profiling build (-DHIRE_TIMESTAMPS) makes thread 0 of workgroup 0 store the 100 MHz wall clock and the shader
clock at numbered points of the kernels; this module runs a few FFN steps of the 1B shape (d_model 2048, d_ff
16384, k 819, k' 3276, seeded synthetic weights and tokens), reads the three tables back and prints, per kernel,
the time of every stamp since the kernel's first one.  The stamps show where the time inside ONE workgroup goes;
they do not show launch latency, and a stamp's own store costs a few tens of nanoseconds.
"""
from __future__ import annotations

import argparse
import ctypes as C

import numpy as np
import torch

from . import hire, inputs as I

# stamp number -> what has happened by then (kernels of the batch-1 route, ffn_fast.hip / fast_select.h)
FAST = [
    ("k_fast_score_int4", [(30, "kernel start"), (31, "token loaded, largest |x| known"),
                            (32, "token quantised, sum |xq| known (anchors)"), (33, "integer dot products done"),
                            (34, "keys stored and counted into the window histogram")]),
    ("k_fast_gather", [(10, "kernel start"), (11, "keys, window and token requested and unpacked"),
                       (15, "window walked: threshold bin known"), (12, "workgroup's units of the bin settled"),
                       (13, "shortlisted units known"), (14, "rows read, activations stored and counted")]),
    ("k_fast_w2", [(24, "kernel start"), (20, "window walked: threshold bin known"), (21, "keys sorted into above and bin"),
                   (22, "bin settled"), (26, "selected rows listed"), (27, "second-layer rows read and accumulated"),
                   (28, "reduced over the waves, y written")]),
]
TOKENS = [
    ("k_fast_score_tokens", [(30, "kernel start"), (31, "tokens loaded, largest |x| known"), (32, "tokens quantised"),
                             (33, "integer dot products done"), (34, "keys stored and counted into the windows")]),
    ("k_fast_gather_tokens", [(10, "kernel start"), (11, "windows read, sums of 256 counters"),
                              (15, "windows walked: threshold bins known"), (12, "workgroup's units settled"),
                              (13, "rows noted"), (16, "rows read and multiplied"), (17, "... by all waves"),
                              (14, "activations stored and counted")]),
]
BATCH = [
    ("k_keys_select (top-k' of the keys)",
     [(10, "kernel start"), (11, "keys loaded, window cleared"), (12, "window built and walked: threshold bin known"),
      (13, "bin listed"), (14, "bin ranked: cut known"), (15, "union bits set")]),
    ("k_refine (top-k of the activations)",
     [(40, "kernel start"), (41, "values loaded, window cleared, bound known"),
      (42, "window built and walked: threshold bin known"), (43, "entries above counted, band listed"),
      (44, "band recomputed in fp64"), (45, "band ranked"), (46, "selected entries packed in output order"),
      (47, "outputs written")]),
]
GATHER = [
    ("k_filter_units (filter stage, first workgroup)",
     [(55, "kernel start"), (56, "candidates known"), (57, "all stages done"),
      (58, "norms, stored values, maximum written")]),
]


SOFTMAX_B1 = [
    ("k_sm1_gather (first workgroup)",
     [(20, "kernel start"), (21, "keys, maxima and token requested, window cleared"),
      (22, "maxima counted, window walked: lower bound of the k'-th key known"),
      (23, "own keys at or above the bound found, their logits computed and stored")]),
    ("k_sm1_final",
     [(30, "kernel start (slots requested)"), (31, "superset counted; key bins and logit range known"),
      (32, "surplus keys dropped, logits of the shortlist counted"),
      (34, "bin of the k-th logit found, selected entries listed"), (35, "ranked, indices and logits written"),
      (36, "softmax written")]),
]


def softmax_one_token(steps):
    """Config 4's classifier (256000 x 2048, k 64, k' 1024) at one token: the short kernel sequence."""
    d, N, k, kp = 2048, 256000, 64, 1024
    layer = hire.SoftmaxLayer.with_int4_scorer(hire.bf16_from_bits(I.classifier(4, N, d)))
    out = hire.SoftmaxOutputs(layer, 1, k, kp)
    ws = hire.alloc_workspace(hire.hire_softmax_workspace_bytes(layer, 1, k, kp))
    x = hire.bf16_from_bits(I.tokens(600, 1, d))
    for _ in range(steps):
        hire.hire_softmax_step(layer, x, k, kp, out, ws)
    torch.cuda.synchronize()
    print(f"# phase stamps, softmax step d_model={d} vocab={N} k={k} k'={kp} batch=1, after {steps} steps on one workspace")
    show(SOFTMAX_B1, *table("hire_debug_timestamps_softmax_b1"))


def table(name):
    fn = getattr(hire._lib, name, None)
    if fn is None:
        raise SystemExit(f"{name} is not exported: load the profiling build (HIRE_LIB=.../libhire_ts.so)")
    buf = (C.c_uint64 * 128)()
    fn(buf)
    return np.array(buf[:64], dtype=np.int64), np.array(buf[64:], dtype=np.int64)


def show(kernels, ts, tc):
    for kernel, points in kernels:
        have = [(i, what) for i, what in points if ts[i] > 0]
        if not have:
            continue
        print(kernel)
        t0, prev = ts[have[0][0]], None
        for i, what in have:
            line = f"  [{i:2d}] +{(ts[i] - t0) * 0.01:7.2f} us"
            if prev is not None:
                dt = (ts[i] - ts[prev]) * 0.01
                mhz = f" at {(tc[i] - tc[prev]) / dt:5.0f} MHz" if dt > 0 else ""
                line += f"  (+{dt:5.2f}{mhz})"
            print(f"{line:52s} {what}")
            prev = i


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--batch", type=int, default=1)
    ap.add_argument("--steps", type=int, default=6)
    ap.add_argument("--general", action="store_true", help="batch 1 through the general kernel sequence")
    ap.add_argument("--softmax", action="store_true", help="the softmax step for one token instead of the FFN step")
    args = ap.parse_args()
    if args.softmax:
        softmax_one_token(args.steps)
        return
    d, N, k, kp, B = 2048, 16384, 819, 3276, args.batch
    L = I.ffn_layer(500, d, N)
    layer = hire.FFNLayer.with_int4_scorer(hire.bf16_from_bits(L["w1u"]), hire.bf16_from_bits(L["w2u"]))
    out = hire.FFNOutputs(layer, B, k, kp)
    ws = hire.alloc_workspace(hire.hire_ffn_workspace_bytes(layer, B, k, kp))
    x = hire.bf16_from_bits(I.tokens(600, B, d))
    if args.general:
        hire.hire_force_generic_path(True)
    for _ in range(args.steps):
        hire.hire_ffn_step(layer, x, k, kp, out, ws)
    torch.cuda.synchronize()
    print(f"# phase stamps, FFN step d_model={d} d_ff={N} k={k} k'={kp} batch={B}, after {args.steps} steps on one workspace")
    if B == 1 and not args.general:
        show(FAST, *table("hire_debug_timestamps_fast"))
    elif B <= 4 and not args.general:
        show(TOKENS, *table("hire_debug_timestamps_fast_tokens"))
        show(FAST[2:], *table("hire_debug_timestamps_fast"))
    else:
        show(BATCH, *table("hire_debug_timestamps_batch_select"))
        show(GATHER, *table("hire_debug_timestamps_gather"))


if __name__ == "__main__":
    main()
