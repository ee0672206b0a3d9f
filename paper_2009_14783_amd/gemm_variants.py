"""Times every tiling of the library's bf16 GEMM kernel on the products of one BERT-base layer (64 x 128 tokens).

    python -m paper_2009_14783_amd.gemm_variants [--iters 50] [--step] [--variants -1,5,9] [--products "fwd ffn1,dx qkv"] [--cube] [--large]
                                                 [--choice]

Stand-alone: each product runs `iters` times back to back on fixed buffers with the epilogue it has in the training
step (bias, bias + residual, bias + GELU with both outputs, GELU' of a saved pre-activation, fp32 accumulate); the
table gives TFLOP/s per variant.  A variant that is not built with a product's epilogue, or cannot take its
contraction length, is served by the library's fallback kernel; the automatic choice is the row `auto`.
--step adds the whole training step (ms per step, 10 warm-up + 30 timed) with the variant forced for every product of the
forward pass and of the activation-gradient chain (the grouped weight-gradient launch keeps its own tiling).
--large takes the products of a BERT-large layer instead (16384 tokens = 32 x 512, and `half`: the 8192 of a forward half-batch).
--choice times the forward and activation-gradient products of widths 512, 768 and 1024 over 264 to 16384 rows with every tiling, operands
rotating over eight copies, and prints what the automatic choice takes beside the fastest tiling.  Tilings 12 and 13 cannot be selected: where the automatic choice
takes one of them, its number and the fastest of the others stand beside its time.
--cube times 8192 x 8192 x 8192 products in the three operand layouts instead (no epilogue; fp32 output for the m-major layout).
--products keeps the named products only (for counter runs under a profiler).
Prints Markdown.  Needs the GPU and the built library; no oracle, no CPU path.
"""
from __future__ import annotations

import argparse
import time

import torch

from . import binding as hs
from . import synth
from .step import Worker

T, H, F = 8192, 768, 3072
# name, a_kmajor, b_kmajor, M, N, K, epilogue (0 none, 1 bias + residual, 2 bias + GELU, 3 GELU'), fp32 output
PRODUCTS = [
    ("fwd qkv", 1, 1, T, 3 * H, H, 0, 0), ("fwd out", 1, 1, T, H, H, 1, 0), ("fwd ffn1", 1, 1, T, F, H, 2, 0), ("fwd ffn2", 1, 1, T, H, F, 1, 0),
    ("dx ffn2", 1, 0, T, F, H, 3, 0), ("dx ffn1", 1, 0, T, H, F, 0, 0), ("dx out", 1, 0, T, H, H, 0, 0), ("dx qkv", 1, 0, T, H, 3 * H, 0, 0),
    ("dW ffn1", 0, 0, F, H, T, 0, 1), ("dW ffn2", 0, 0, H, F, T, 0, 1), ("dW out", 0, 0, H, H, T, 0, 1), ("dW qkv", 0, 0, 3 * H, H, T, 0, 1),
]


def layer_products(rows, H, F, tag=""):
    return [(f"fwd qkv{tag}", 1, 1, rows, 3 * H, H, 0, 0), (f"fwd out{tag}", 1, 1, rows, H, H, 1, 0), (f"fwd ffn1{tag}", 1, 1, rows, F, H, 2, 0),
            (f"fwd ffn2{tag}", 1, 1, rows, H, F, 1, 0)], [(f"dx ffn2{tag}", 1, 0, rows, F, H, 3, 0), (f"dx ffn1{tag}", 1, 0, rows, H, F, 1, 0),
            (f"dx out{tag}", 1, 0, rows, H, H, 0, 0), (f"dx qkv{tag}", 1, 0, rows, H, 3 * H, 1, 0)]


LARGE = layer_products(16384, 1024, 4096)[0] + layer_products(8192, 1024, 4096, " half")[0] + layer_products(16384, 1024, 4096)[1]
# A and B k-major; A k-major, B n-major; A and B m-major
CUBES = [("cube kk", 1, 1, 8192, 8192, 8192, 0, 0), ("cube kn", 1, 0, 8192, 8192, 8192, 0, 0), ("cube nn", 0, 0, 8192, 8192, 8192, 0, 1)]
NAMES = {-1: "auto", 0: "0: 128x128x32, 3/CU", 1: "1: LDS-direct 256x256x64", 2: "2: 32x32, waves split K", 3: "3: LDS-direct 128x192x64, 2/CU",
         4: "4: LDS-direct 32x64x64, 3/CU", 5: "5: 128x128x64, 2/CU", 6: "6: LDS-direct 192x128x64, 2/CU", 7: "7: LDS-direct 64x128x64, 2/CU",
         8: "8: LDS-direct 128x64x64, 2/CU", 9: "9: LDS-direct 128x128x64, 2/CU", 10: "10: LDS-direct 256x128x64", 11: "11: LDS-direct 64x64x64, 3/CU"}


def time_product(prod, iters, bufs):
    name, ak, bk, M, N, K, epi, cf = prod
    A, B, Cb, Cf, C2, aux, bias, ws = bufs
    lda = K if ak else M
    ldb = K if bk else N
    kw = dict(c_f32=cf, beta=1.0 if cf else 0.0)
    if not cf:
        kw.update(epi=epi, bias=None if epi == 3 else bias, aux=aux if epi in (1, 3) else None, ldaux=N if epi in (1, 3) else 0,
                  C2=C2 if epi == 2 else None)
    run = lambda: hs.hs_op_gemm(1, ak, bk, M, N, K, A, lda, B, ldb, Cf if cf else Cb, N, scratch=ws, scratch_bytes=ws.numel(), **kw)
    for _ in range(3):
        run()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    for _ in range(iters):
        run()
    e1.record()
    torch.cuda.synchronize()
    us = e0.elapsed_time(e1) * 1e3 / iters
    return us, 2.0 * M * N * K / us / 1e6


def choice(iters):
    """Markdown: per product and row count the time of the automatic choice, and of the fastest tiling where that is another."""
    rows_of, copies = (264, 520, 1032, 2056, 4104, 8192, 16384), 8
    n = 16384 * 4096
    mk = lambda scale: [(torch.randn(n, device="cuda") * scale).to(torch.bfloat16) for _ in range(copies)]
    As, Bs, Xs = mk(0.5), mk(0.05), mk(1.0)
    Cs, C2 = [torch.empty(n, dtype=torch.bfloat16, device="cuda") for _ in range(copies)], torch.empty(n, dtype=torch.bfloat16, device="cuda")
    bias = torch.zeros(4096, dtype=torch.bfloat16, device="cuda")

    def us(prod, v):
        _, ak, bk, M, N, K, epi, _ = prod
        hs.hs_tune_gemm_variant(v)
        def run(i):
            i %= copies
            hs.hs_op_gemm(1, ak, bk, M, N, K, As[i], K, Bs[i], K if bk else N, Cs[i], N, epi=epi, bias=None if epi == 3 else bias,
                          aux=Xs[i] if epi in (1, 3) else None, ldaux=N if epi in (1, 3) else 0, C2=C2 if epi == 2 else None)
        times = []
        for rep in range(3):
            run(0)
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            for i in range(iters):
                run(i)
            e1.record()
            torch.cuda.synchronize()
            times.append(e0.elapsed_time(e1) * 1e3 / iters)
        return min(times)

    print("| width, product | " + " | ".join(f"{r} rows" for r in rows_of) + " |")
    print("|---|" + "---|" * len(rows_of))
    ratios, lone = [], []      # lone: fastest other tiling over 12 or 13 where these are chosen
    for H in (512, 768, 1024):
        lists = [sum(layer_products(r, H, 4 * H), []) for r in rows_of]
        for j in range(len(lists[0])):
            cells = []
            for r, products in zip(rows_of, lists):
                t = {v: us(products[j], v) for v in [-1] + list(range(12))}
                best = min(range(12), key=lambda v: t[v])
                ratios.append(t[-1] / min(t.values()))
                _, ak, bk, M, N, K, epi, _ = products[j]
                hs.hs_tune_gemm_variant(-1)
                took, _ = hs.hs_gemm_choice(ak, bk, M, N, K, epi=epi)
                if took >= 12:
                    lone.append(t[best] / t[-1])
                cells.append(f"{t[-1]:.1f}" + (f" [{took}]" if took >= 12 else "") +
                             (f" ({t[best]:.1f}: {best})" if t[best] < 0.98 * t[-1] or took >= 12 else ""))
            print(f"| {H}, {lists[0][j][0]} | " + " | ".join(cells) + " |", flush=True)
    hs.hs_tune_gemm_variant(-1)
    print(f"\nus; in brackets the fastest tiling and its time where it is more than 2 % faster, and beside 12 and 13.  Automatic choice over fastest: mean "
          f"{sum(ratios) / len(ratios):.3f}, largest {max(ratios):.2f} over {len(ratios)} products; fastest other tiling over 12 and 13 where these are taken: mean "
          f"{sum(lone) / max(1, len(lone)):.3f} over {len(lone)}.")


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--iters", type=int, default=50)
    ap.add_argument("--step", action="store_true")
    ap.add_argument("--variants", default="", help="comma-separated variant numbers (-1: automatic); default: all")
    ap.add_argument("--products", default="", help="comma-separated product names; default: all")
    ap.add_argument("--cube", action="store_true")
    ap.add_argument("--large", action="store_true")
    ap.add_argument("--choice", action="store_true")
    args = ap.parse_args()
    hs.lib()
    if args.choice:
        return choice(args.iters)
    products = CUBES if args.cube else LARGE if args.large else PRODUCTS
    if args.products:
        products = [p for p in products if p[0] in [q.strip() for q in args.products.split(",")]]
        if not products:
            raise SystemExit("--products: no such product")
    g = torch.Generator(device="cuda").manual_seed(1)
    n = max(p[3] * p[4] for p in products + [("", 0, 0, T, F, 0, 0, 0)])
    n = max(n, max(max(p[3], p[4]) * p[5] for p in products))
    A = (torch.randn(n, generator=g, device="cuda") * 0.5).to(torch.bfloat16)
    B = (torch.randn(n, generator=g, device="cuda") * 0.05).to(torch.bfloat16)
    aux = torch.randn(n, generator=g, device="cuda").to(torch.bfloat16)
    bufs = (A, B, torch.empty(n, dtype=torch.bfloat16, device="cuda"),
            torch.zeros(max([F * 3 * H] + [p[3] * p[4] for p in products if p[7]]), dtype=torch.float32, device="cuda"),
            torch.empty(n, dtype=torch.bfloat16, device="cuda"), aux, torch.zeros(max([F] + [p[4] for p in products]), dtype=torch.bfloat16, device="cuda"),
            torch.empty(96 << 20, dtype=torch.uint8, device="cuda"))
    variants = [int(v) for v in args.variants.split(",")] if args.variants else [-1] + list(range(12))
    for prod in products:      # untimed pass: clocks up, code loaded
        time_product(prod, 3, bufs)
    print("| variant | " + " | ".join(p[0] for p in products) + " | sum (us) |")
    print("|---|" + "---|" * (len(products) + 1))
    for v in variants:
        hs.hs_tune_gemm_variant(v)
        cells, tot = [], 0.0
        for prod in products:
            us, tf = time_product(prod, args.iters, bufs)
            cells.append(f"{tf:.0f}")
            tot += us
        print(f"| {NAMES[v]} | " + " | ".join(cells) + f" | {tot:.0f} |", flush=True)
    hs.hs_tune_gemm_variant(-1)
    if not args.step:
        return
    wl = synth.WORKLOADS[1]
    model = synth.MODELS[wl["model"]]
    cfg = hs.make_cfg(**model)
    theta = synth.init_params(hs.hs_param_layout(cfg), wl["seed"])
    worker = Worker(model, wl["compute"], theta)
    dev = [worker.upload(b) for b in synth.workload_micro_batches(1)]
    print("\n| variant | ms per step |\n|---|---|")
    for v in variants:
        hs.hs_tune_gemm_variant(v)
        for _ in range(10):
            worker.train_step(dev, wl["adam"])
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(30):
            worker.train_step(dev, wl["adam"])
        torch.cuda.synchronize()
        print(f"| {NAMES[v]} | {(time.perf_counter() - t0) / 30 * 1e3:.3f} |", flush=True)
    hs.hs_tune_gemm_variant(-1)


if __name__ == "__main__":
    main()
