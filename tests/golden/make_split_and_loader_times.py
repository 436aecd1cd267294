#!/usr/bin/env python3
"""Writes tests/golden/split_and_loader_times.json: measured launch times of the schedules the library chooses between where a
contraction is split along k (every instance and split factor) and of the convolution loaders (patch-staged, row-staged,
element gather), on one MI355X.  A measurement fixture like instance_times.json, for the parts of the cost model that file
does not reach; tests/test_cost_model_splits_and_loaders.py reads it on the CPU.

Run on an MI355X from the repository root, after building (the file to write may be named):
    python tests/golden/make_split_and_loader_times.py [path]
Protocol per schedule: three sets of operands in turn, 5 ms of launches to settle the clock, then the least of 3 event-bracketed
batches of at least 10 launches.  Schedules the model prices above SKIP_GEMM or SKIP_CONV times its cheapest are not timed.
"""
import json
import os
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.dirname(os.path.abspath(__file__))))
sys.path.insert(0, ROOT)
SKIP_GEMM, SKIP_CONV = 3.0, 10.0      # (the element gather is priced well above the other loaders)
SPLITS = (1, 2, 3, 4, 6, 8, 12, 16)
# dtype, out, M, N, K, transA, transB: few tiles over a deep k, some that are nearly a round, extents off the vectors
GEMMS = [("f16", "f32", 512, 512, 32768, 0, 1), ("f16", "f32", 256, 256, 65536, 0, 0), ("f16", "f32", 1024, 1024, 8192, 0, 1),
         ("f32", "f32", 256, 256, 16384, 0, 1), ("f16", "f32", 768, 3072, 8192, 1, 0), ("bf16", "f32", 640, 384, 12288, 0, 0),
         ("bf16", "bf16", 512, 768, 4096, 0, 1), ("f32", "f32", 512, 512, 2048, 0, 0), ("f16", "f32", 300, 512, 4096, 0, 1),
         ("f16", "f32", 1000, 1000, 2000, 1, 1), ("f16", "f32", 1003, 511, 9001, 0, 0), ("bf16", "f32", 333, 777, 5001, 0, 1),
         ("f32", "f32", 201, 303, 3001, 1, 0), ("f16", "f32", 128, 128, 4096, 0, 0)]
# dtype, n, c, h, w, k, r, stride, pad
CONVS = [("f16", 16, 3, 112, 112, 64, 7, 2, 3), ("f16", 14, 5, 89, 98, 33, 3, 1, 0), ("f16", 14, 100, 96, 48, 128, 3, 2, 1),
         ("f32", 8, 64, 20, 103, 64, 5, 2, 1), ("f32", 18, 33, 55, 98, 128, 1, 1, 1), ("f16", 23, 4, 76, 68, 10, 5, 1, 0),
         ("f32", 14, 128, 60, 96, 64, 3, 3, 1), ("f16", 26, 100, 37, 58, 64, 1, 1, 1), ("f16", 18, 64, 46, 71, 10, 3, 2, 0),
         ("f32", 27, 6, 83, 57, 8, 7, 2, 3), ("f16", 16, 20, 66, 66, 64, 3, 1, 1), ("f32", 8, 12, 56, 56, 64, 3, 1, 1),
         ("f16", 17, 128, 24, 30, 10, 5, 1, 1), ("bf16", 16, 16, 56, 56, 64, 5, 1, 2), ("f16", 6, 16, 57, 47, 48, 7, 1, 3)]


def main():
    import torch
    from paper_2502_11407_amd import binding as gs
    torch_type = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}

    def fresh(shape, dtype):
        return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(-1, 1).to(torch_type[dtype])

    def batch_us(call, launches):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for i in range(launches):
            call(i)
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) * 1e3 / launches

    def time_us(call):
        n = max(10, int(5000.0 / max(batch_us(call, 3), 3.0)))
        batch_us(call, n)
        return round(min(batch_us(call, max(10, n // 5)) for _ in range(3)), 3)

    out = {"device": torch.cuda.get_device_properties(0).name, "command": "python tests/golden/make_split_and_loader_times.py", "shapes": []}
    for shape in GEMMS + CONVS:
        if len(shape) == 7:
            dtype, odt, M, N, K, ta, tb = shape
            p = gs.gemm_problem(dtype, M, N, K, ta, tb, 1, odt)
            x = [(fresh((K, M) if ta else (M, K), dtype), fresh((N, K) if tb else (K, N), dtype)) for _ in range(3)]
            o, splits, ws_of = gs.empty_device((M, N), odt), SPLITS, gs.gemm_workspace

            def run(i, s, ws):
                gs.gemm(p, x[i % 3][0], x[i % 3][1], o, 1.0, 0.0, s, workspace=ws)
        else:
            dtype, n, c, h, w, k, r, stride, pad = shape
            p = gs.conv_problem(dtype, n, c, h, w, k, r, r, stride, pad)
            x = [(fresh((n, c, h, w), dtype), fresh((k, c, r, r), dtype)) for _ in range(3)]
            o, splits, ws_of = gs.empty_device((n, k, (h + 2 * pad - r) // stride + 1, (w + 2 * pad - r) // stride + 1)), (1,), gs.conv_workspace

            def run(i, s, ws):
                gs.conv2d(p, x[i % 3][0], x[i % 3][1], o, s, ws)
        cands = []
        for idx in range(gs.num_instances()):
            s = gs.instance_schedule(idx, p)
            for split in splits if s is not None else ():
                t = gs.Schedule.from_buffer_copy(s)
                t.split_k = split
                us = gs.predict_us(t, p)
                if us > 0 and (split == 1 or gs.workspace_bytes(p, t) > 0):
                    cands.append((us, idx, split, t))
        cheapest = min(u for u, _, _, _ in cands)
        rows = []
        for us, idx, split, s in cands:
            if us > (SKIP_GEMM if len(shape) == 7 else SKIP_CONV) * cheapest:
                continue
            ws = ws_of(p, s)
            try:
                run(0, s, ws)
            except gs.GensorError:                 # vector reads these operands cannot give, or a k tail beside direct staging
                continue
            rows.append([idx, split, time_us(lambda i: run(i, s, ws))])
        rows.sort()
        out["shapes"].append({"shape": list(shape), "rows": rows})
        best = min(rows, key=lambda q: q[2])
        print(shape, "%d schedules, best instance %d split %d %.1f us" % (len(rows), *best), flush=True)
    text = json.dumps(out).replace('{"shape"', '\n{"shape"')
    path = sys.argv[1] if len(sys.argv) > 1 else os.path.join(ROOT, "tests", "golden", "split_and_loader_times.json")
    with open(path, "w") as f:
        f.write(text + "\n")


if __name__ == "__main__":
    main()
