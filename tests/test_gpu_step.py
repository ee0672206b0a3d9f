"""End-to-end parity of the training step on the GPU against the CPU oracle, through the C ABI.

Tolerances (relative L2 error per tensor, |a-b|/|b| for scalars; tensors whose reference norm is
below 1e-12 are compared absolutely): 1e-4 in fp32 mode, 2e-2 on losses and gradients in bf16
mode.  Masks and batch indices are compared bit-exactly (tests/test_gpu_ops.py,
tests/test_library_host.py)."""
import math

import numpy as np
import pytest

from oracle import batcher as OB
from oracle import hetseq_oracle as O
from paper_2009_14783_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = {"fp32": 1e-4, "bf16": 2e-2}


@pytest.fixture(scope="module")
def W():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2009_14783_amd import binding
    binding.lib()
    from paper_2009_14783_amd import step
    return step.Worker


def rel(a, b):
    a, b = np.asarray(a, np.float64), np.asarray(b, np.float64)
    nb = np.linalg.norm(b)
    return float(np.linalg.norm(a - b) / nb) if nb > 1e-12 else float(np.linalg.norm(a - b))


ROWWISE = ("emb.word", "emb.pos", "head.dec.b")     # tensors whose rows (entries) belong to single tokens / positions


def compare_flat(layout, got, want, tol, what):
    """Per tensor: relative L2 error below tol.  On top of that, so that one wrong row or entry cannot hide inside a
    large tensor: (1) no single element is off by more than 4 tol of its own size plus 48 tol times the scale of its row
    and column, RMS(row) x RMS(column) / RMS(tensor) (a weight gradient is a sum of outer products, so its rounding noise
    has that rank-one profile, and heavy tails: rounding the weights to bf16 alone moves single elements of the oracle's
    gradient by up to 0.4 of that scale at BERT-base size; at least a quarter of the tensor's RMS, the RMS itself for
    vectors); (2) for the embedding tables and the decoder bias every row (entry)
    that carries real signal (norm above a tenth of the RMS row norm) is held to 2 tol on its own."""
    worst = ("", 0.0)
    for name, off, r, c in layout:
        g = np.asarray(got[off:off + r * c], np.float64)
        w = np.asarray(want[off:off + r * c], np.float64)
        e = rel(g, w)
        if e > worst[1]:
            worst = (name, e)
        assert e < tol, f"{what}: {name} rel err {e:.3e} >= {tol}"
        rms = float(np.sqrt(np.mean(w * w)))
        if rms > 1e-12:
            g2, w2 = g.reshape(r, c), w.reshape(r, c)
            row_rms = np.sqrt(np.mean(w2 * w2, axis=1, keepdims=True))
            col_rms = np.sqrt(np.mean(w2 * w2, axis=0, keepdims=True))
            scale = np.maximum(row_rms * col_rms / rms, 0.25 * rms) if r > 1 else np.full_like(w2, rms)
            excess = (np.abs(g2 - w2) - 4 * tol * np.abs(w2)) / scale
            k = int(np.argmax(excess))
            assert excess.flat[k] < 48 * tol, (f"{what}: {name}[{k // c}, {k % c}] = {g2.flat[k]:.6e}, oracle {w2.flat[k]:.6e}: off by more "
                                               f"than 4 tol of itself + 48 tol x the scale of its row and column ({scale.flat[k]:.3e})")
        if name in ROWWISE:
            rows = (r, c) if r > 1 else (c, 1)
            g2, w2 = g.reshape(rows), w.reshape(rows)
            wn = np.linalg.norm(w2, axis=1)
            floor = 0.1 * float(np.sqrt(np.mean(wn * wn)))
            big = wn > floor
            if big.any():
                err = np.linalg.norm(g2 - w2, axis=1)[big] / wn[big]
                k = int(np.argmax(err))
                assert err[k] < 2 * tol, f"{what}: {name} row {np.flatnonzero(big)[k]} rel err {err[k]:.3e} >= {2 * tol} ({int(big.sum())} rows checked)"
    return worst


def gpu_micro_grad(worker, mb):
    d = worker.upload(mb)
    worker.G.fill_(float("nan")) if d["M"] > 0 else worker.G.zero_()   # accumulate=0 must overwrite everything
    worker.forward_backward(d, worker.G, 0, 0)
    torch.cuda.synchronize()
    return float(worker.loss_buf[0].item()), worker.G.cpu().numpy().copy()


def oracle_micro_grad(ocfg, theta, mb, dtype):
    l, g, _, _ = O.micro_batch_grad(ocfg, theta.astype(dtype), mb["ids"], mb["lens"], mb["mlm_pos"], mb["mlm_label"])
    return float(l), g


# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("compute", ["fp32", "bf16"])
def test_workload0_tiny_step(W, compute):
    """Tiny encoder: forward + backward, normalise by the sample count, one Adam step."""
    wl = synth.WORKLOADS[0]
    model = synth.MODELS["tiny"]
    ocfg = O.ModelCfg(**model)
    theta = synth.init_params(O.param_layout(ocfg), wl["seed"])
    mbs = synth.workload_micro_batches(0)
    worker = W(model, compute, theta)
    layout = O.param_layout(ocfg)
    tol = TOL[compute]
    # gradient of the loss sum
    loss, g = gpu_micro_grad(worker, mbs[0])
    ol, og = oracle_micro_grad(ocfg, theta, mbs[0], np.float64)
    assert abs(loss - ol) / abs(ol) < tol
    compare_flat(layout, g, og, tol, "grad")
    # whole step
    th, m, v = theta.astype(np.float64), np.zeros_like(theta, np.float64), np.zeros_like(theta, np.float64)
    oloss, oG, oD = O.train_step(ocfg, th, m, v, 1, mbs, **wl["adam"])
    D = worker.train_step([worker.upload(mb) for mb in mbs], wl["adam"])
    torch.cuda.synchronize()
    assert D == oD == 4
    assert abs(worker.reported_loss(D) - oloss) / abs(oloss) < tol
    compare_flat(layout, worker.G.cpu().numpy(), oG, tol, "G")
    if compute == "fp32":
        compare_flat(layout, worker.m.cpu().numpy(), m, tol, "m")
        compare_flat(layout, worker.v.cpu().numpy(), v, 2 * tol, "v")
        assert rel(worker.w.cpu().numpy(), th) < 1e-6
        # the update itself: Adam divides by |g|, so elements with a vanishing gradient are sensitive;
        # compare where the reference gradient is well above eps
        big = np.abs(oG) > 1e-4
        dw = worker.w.cpu().numpy().astype(np.float64) - theta
        assert rel(dw[big], (th - theta)[big]) < 1e-3
    else:
        assert torch.equal(worker.w_lowp, worker.w.to(torch.bfloat16))
    worker.close()


def test_fp32_edge_cases_ragged_single_token_no_targets(W):
    """Lengths 1 and L, a micro-batch without any target, an 8-wide padding."""
    model = dict(synth.MODELS["tiny"])
    ocfg = O.ModelCfg(**model)
    theta = synth.init_params(O.param_layout(ocfg), 7)
    theta = (theta * 5).astype(np.float32)                      # stronger non-linearity than the 0.02 init
    layout = O.param_layout(ocfg)
    rng = synth.rng_for(11)
    worker = W(model, "fp32", theta)
    for lens, L in ([1, 8, 3], 8), ([40, 1, 17, 33, 24], 40), ([64], 64):
        mb = synth.make_micro_batch(rng, lens, L, ocfg.vocab, "uniform")
        loss, g = gpu_micro_grad(worker, mb)
        ol, og = oracle_micro_grad(ocfg, theta, mb, np.float64)
        assert abs(loss - ol) / abs(ol) < 1e-4
        compare_flat(layout, g, og, 1e-4, f"lens={lens}")
    # no targets: loss 0 and (with a zeroed buffer) zero gradient
    mb = synth.make_micro_batch(rng, [5, 8], 8, ocfg.vocab, "uniform")
    mb["mlm_pos"] = mb["mlm_pos"][:0]
    mb["mlm_label"] = mb["mlm_label"][:0]
    loss, g = gpu_micro_grad(worker, mb)
    assert loss == 0.0 and not np.any(g)
    worker.close()


@pytest.mark.parametrize("compute", ["fp32", "bf16"])
def test_unequal_micro_batches_dummy_and_fused_accumulation(W, compute):
    """Shares 2 : 6 : 14 with an empty worker in between: G/22 equals the oracle's step, fused
    (gradients added straight into G) and unfused (separate buffer + accumulate) agree."""
    model = dict(synth.MODELS["tiny"])
    ocfg = O.ModelCfg(**model)
    theta = synth.init_params(O.param_layout(ocfg), 21)
    layout = O.param_layout(ocfg)
    rng = synth.rng_for(31)
    mbs = [synth.make_micro_batch(rng, lens, 32, ocfg.vocab, "uniform")
           for lens in ([32, 20], [12, 32, 32, 24, 8, 28], [16] * 14)]
    mbs.insert(1, dict(dummy=True))
    th, m, v = theta.astype(np.float64), np.zeros(theta.size), np.zeros(theta.size)
    oloss, oG, oD = O.train_step(ocfg, th, m, v, 1, mbs, lr=1e-4, eps=1e-6)
    assert oD == 22
    results = []
    for fused in (True, False):
        worker = W(model, compute, theta)
        up = [None if mb.get("dummy") else worker.upload(mb) for mb in mbs]
        D = worker.train_step(up, dict(lr=1e-4, beta1=0.9, beta2=0.999, eps=1e-6), fused=fused)
        torch.cuda.synchronize()
        assert D == 22
        assert abs(worker.reported_loss(D) - oloss) / abs(oloss) < TOL[compute]
        G = worker.G.cpu().numpy()
        compare_flat(layout, G, oG, TOL[compute], f"G fused={fused}")
        results.append(G)
        worker.close()
    compare_flat(layout, results[0], results[1], 1e-5 if compute == "fp32" else 1e-3, "fused vs unfused")


@pytest.mark.parametrize("hidden,vocab,B,L", [(64, 1000, 1, 8), (64, 8, 33, 64), (320, 24, 9, 40), (768, 400, 8, 24), (1024, 24, 17, 16)])
def test_embedding_gradients_over_widths_and_run_lengths(W, hidden, vocab, B, L):
    """Rows that end inside a block of 256 columns, token counts that end inside a chunk, runs of one token over many chunks, sequences
    beyond a multiple of eight."""
    model = dict(synth.MODELS["tiny"], hidden=hidden, n_heads=hidden // 64, ffn=128, vocab=vocab)
    ocfg = O.ModelCfg(**model)
    layout = O.param_layout(ocfg)
    theta = synth.init_params(layout, hidden + vocab)
    mb = synth.make_micro_batch(synth.rng_for(B * L), [max(1, L - 3 * (i % 4)) for i in range(B)], L, vocab, "uniform")
    worker = W(model, "fp32", theta)
    loss, g = gpu_micro_grad(worker, mb)
    worker.close()
    ol, og = oracle_micro_grad(ocfg, theta, mb, np.float64)
    assert abs(loss - ol) / abs(ol) < TOL["fp32"]
    compare_flat(layout, g, og, TOL["fp32"], f"hidden={hidden}")


def test_run_to_run_bit_reproducible(W):
    model = dict(synth.MODELS["tiny"])
    ocfg = O.ModelCfg(**model)
    theta = synth.init_params(O.param_layout(ocfg), 3)
    mb = synth.make_micro_batch(synth.rng_for(2), [64, 50, 64, 64, 9, 64], 64, ocfg.vocab, "zipf")
    worker = W(model, "bf16", theta)
    a = gpu_micro_grad(worker, mb)
    b = gpu_micro_grad(worker, mb)
    assert a[0] == b[0] and a[1].tobytes() == b[1].tobytes()
    worker.close()


# ------------------------------------------------------------------------------------------------
# BERT-base sized workloads (bf16) against the fp32 oracle
# ------------------------------------------------------------------------------------------------
@pytest.fixture(scope="module")
def base():
    model = synth.MODELS["bert_base"]
    ocfg = O.ModelCfg(**model)
    layout = O.param_layout(ocfg)
    return model, ocfg, layout


def test_workload1_bert_base_full_size(W, base):
    model, ocfg, layout = base
    wl = synth.WORKLOADS[1]
    theta = synth.init_params(layout, wl["seed"])
    mb = synth.workload_micro_batches(1)[0]
    assert mb["ids"].shape == (64, 128) and mb["mlm_pos"].size == 1216
    worker = W(model, "bf16", theta)
    loss, g = gpu_micro_grad(worker, mb)
    ol, og = oracle_micro_grad(ocfg, theta, mb, np.float32)
    assert abs(loss / 1216 - math.log(30522)) < 0.2
    assert abs(loss - ol) / abs(ol) < TOL["bf16"]
    worst = compare_flat(layout, g, og, TOL["bf16"], "grad")
    print("workload 1 worst tensor", worst)
    worker.close()


def test_workload1_three_updates_follow_oracle_bf16(W, base):
    """Three whole steps at full size (forward, loss, backward with the update armed inside it, bf16 weight copy): the
    reported loss of every step against the oracle's fp32 loop, and the weights after the third."""
    model, ocfg, layout = base
    wl = synth.WORKLOADS[1]
    theta = synth.init_params(layout, wl["seed"])
    adam = dict(wl["adam"], lr=1e-3)        # ten times the paper's rate, so that three updates move the loss visibly
    worker = W(model, "bf16", theta)
    th, m, v = theta.copy(), np.zeros_like(theta), np.zeros_like(theta)
    got, want = [], []
    for t in range(1, 4):
        mbs = synth.step_micro_batches(wl["seed"], t, [128] * 64, 128, model["vocab"], "zipf")
        D = worker.train_step([worker.upload(mb) for mb in mbs], adam)
        got.append(worker.reported_loss(D))
        oloss, oG, oD = O.train_step(ocfg, th, m, v, t, mbs, **adam)
        want.append(float(oloss))
        print(f"update {t}: loss {got[-1]:.4f} (oracle {want[-1]:.4f})", flush=True)
        assert oD == D and abs(got[-1] - want[-1]) / abs(want[-1]) < TOL["bf16"]
    assert want[2] < want[0] - 0.5                     # the updates do change the model
    # Adam moves every weight by about lr per step whatever the size of its gradient, so where a gradient is within bf16
    # noise of zero the two sides may step in opposite directions: the weights are compared on the scale of the movement
    w_gpu = worker.w.cpu().numpy()
    moved = float(np.linalg.norm(th.astype(np.float64) - theta))
    apart = float(np.linalg.norm(w_gpu.astype(np.float64) - th))
    print(f"weights moved {moved:.3f} (L2), the two sides are {apart:.3f} apart: {apart / moved:.3f} of the movement")
    assert apart < 0.25 * moved
    worker.close()


def test_workload3_unequal_shares_equal_one_batch(W, base):
    """Micro-batches of 8, 24 and 56 sequences summed and divided by 88 against one batch of 88."""
    model, ocfg, layout = base
    wl = synth.WORKLOADS[3]
    theta = synth.init_params(layout, wl["seed"])
    mbs = synth.workload_micro_batches(3)
    assert [mb["n_seq"] for mb in mbs] == [8, 24, 56]
    big = synth.concat_micro_batches(mbs)
    worker = W(model, "bf16", theta)
    n = worker.accumulate_micro_batches([worker.upload(mb) for mb in mbs])
    from paper_2009_14783_amd import binding as hs
    hs.hs_grad_accum_normalize(worker.G, None, worker.P, 0, 88.0)
    torch.cuda.synchronize()
    assert n == 88
    G3 = worker.G.cpu().numpy().copy()
    loss3 = float(worker.loss_buf.sum().item())
    loss1, g1 = gpu_micro_grad(worker, big)
    worker.close()
    assert abs(loss3 - loss1) / abs(loss1) < 1e-3
    compare_flat(layout, G3, g1 / 88.0, 1e-2, "3 micro-batches vs one batch (both GPU)")
    # oracle: the same three shares accumulated and divided by the global sample count
    oG, on, ol = np.zeros_like(theta), 0, 0.0
    for mb in mbs:
        l, g = oracle_micro_grad(ocfg, theta, mb, np.float32)
        oG, on = O.accumulate(oG, on, g, mb["n_seq"])
        ol += l
        print("oracle share done", mb["n_seq"], flush=True)
    assert on == 88
    O.normalize(oG, on)
    assert abs(loss3 - ol) / abs(ol) < TOL["bf16"]
    compare_flat(layout, G3, oG, TOL["bf16"], "G vs oracle")


def test_workload2_variable_length_buckets(W, base):
    """Batches formed by the library's batcher under the 16384-real-token cap, bit for bit the oracle's.  Against the
    oracle: the whole first batch (shortest bucket, most sequences), the whole last one (longest bucket, partial), and
    for every padded length in between the first eight sequences of that bucket's first batch."""
    from paper_2009_14783_amd import binding as hs
    model, ocfg, layout = base
    wl = synth.WORKLOADS[2]
    rng = synth.rng_for(wl["seed"])
    lengths = synth.draw_lengths(rng, 4096, 64, 512)
    seq, offs, pads = hs.hs_make_batches(lengths, 64, 16384, 0)
    oseq, ooffs, opads = OB.make_batches(lengths, 64, 16384, 0)
    assert seq.tolist() == oseq and offs.tolist() == ooffs and pads.tolist() == opads
    theta = synth.init_params(layout, wl["seed"])
    worker = W(model, "bf16", theta)
    nb = len(pads)
    assert sorted(set(pads.tolist())) == [64 * k for k in range(1, 9)]
    first_of = {int(L): int(np.flatnonzero(pads == L)[0]) for L in sorted(set(pads.tolist()))}
    cases = [(0, None), (nb - 1, None)] + [(j, 8) for L, j in first_of.items() if j not in (0, nb - 1)]
    for j, take in cases:
        lens = lengths[seq[offs[j]:offs[j + 1]]]
        assert lens.sum() <= 16384 and lens.max() <= pads[j] and lens.min() > pads[j] - 64
        if take:
            lens = lens[:take]
        mb = synth.make_micro_batch(synth.rng_for(wl["seed"] + 100 + j), lens, int(pads[j]), ocfg.vocab, "zipf")
        loss, g = gpu_micro_grad(worker, mb)
        ol, og = oracle_micro_grad(ocfg, theta, mb, np.float32)
        print(f"batch {j}: B={len(lens)} L={pads[j]} loss {loss:.2f} (oracle {ol:.2f})", flush=True)
        assert abs(loss - ol) / abs(ol) < TOL["bf16"]
        compare_flat(layout, g, og, TOL["bf16"], f"batch {j} (B={len(lens)}, L={pads[j]})")
    worker.close()


def test_workload4_bert_large_shape(W):
    """BERT-large at L = 512.  Against the oracle, element by element: 2 layers with 4 sequences, then the whole
    24-layer model with 16 ragged sequences (every gradient tensor; about a minute of oracle time).  The full
    4 x 32-sequence step on top: loss near ln V and accumulation of 4 micro-batches equal to 4 x one of them when the
    same micro-batch is repeated."""
    model = dict(synth.MODELS["bert_large"])
    small = dict(model, n_layers=2)
    ocfg = O.ModelCfg(**small)
    layout = O.param_layout(ocfg)
    theta = synth.init_params(layout, 1238)
    mb = synth.make_micro_batch(synth.rng_for(1238), [512, 300, 512, 77], 512, ocfg.vocab, "zipf")
    worker = W(small, "bf16", theta)
    loss, g = gpu_micro_grad(worker, mb)
    worker.close()
    ol, og = oracle_micro_grad(ocfg, theta, mb, np.float32)
    assert abs(loss - ol) / abs(ol) < TOL["bf16"]
    compare_flat(layout, g, og, TOL["bf16"], "bert-large layers")
    # Full depth: all 24 layers, sixteen ragged sequences at L = 512, every gradient tensor.  At this depth rounding the
    # WEIGHTS to bf16 alone, with exact arithmetic otherwise, already moves the oracle's own gradient by about 2e-2
    # (printed below), which no bf16 kernel can undo; the kernels are responsible for the gradient of the function they
    # are given, so the 2e-2 bar is applied against the oracle at the bf16-rounded weights the GPU path really uses, and
    # the distance to the oracle at the fp32 weights is held to that bar plus the measured effect of the rounding.
    full_cfg = O.ModelCfg(**model)
    full_layout = O.param_layout(full_cfg)
    theta = synth.init_params(full_layout, 1238)
    lens16 = [512, 300, 512, 77, 512, 409, 512, 181, 512, 64, 256, 512, 333, 512, 129, 480]
    mb16 = synth.make_micro_batch(synth.rng_for(1239), lens16, 512, full_cfg.vocab, "zipf")
    worker = W(model, "bf16", theta)
    loss, g = gpu_micro_grad(worker, mb16)
    theta_r = worker.w_lowp.float().cpu().numpy()                      # the weights the forward and backward passes read
    assert np.array_equal(theta_r, torch.from_numpy(theta).to(torch.bfloat16).float().numpy())
    print("24 layers: oracle at the rounded weights running", flush=True)
    olr, ogr = oracle_micro_grad(full_cfg, theta_r, mb16, np.float32)
    print(f"24 layers, 16 sequences: loss {loss:.2f} (oracle at the rounded weights {olr:.2f}); oracle at the fp32 weights running", flush=True)
    ol, og = oracle_micro_grad(full_cfg, theta, mb16, np.float32)
    assert abs(loss - olr) / abs(olr) < TOL["bf16"] and abs(loss - ol) / abs(ol) < TOL["bf16"]
    worst = compare_flat(full_layout, g, ogr, TOL["bf16"], "bert-large, 24 layers, oracle at the rounded weights")
    drift = max(rel(ogr[off:off + r * c], og[off:off + r * c]) for _, off, r, c in full_layout)
    far = max(rel(g[off:off + r * c], og[off:off + r * c]) for _, off, r, c in full_layout)
    print(f"24 layers: worst tensor against the oracle at the rounded weights {worst}; bf16 rounding of the weights alone moves the "
          f"oracle's gradient by up to {drift:.3e} per tensor; GPU against the oracle at the fp32 weights: up to {far:.3e}", flush=True)
    assert far < TOL["bf16"] + drift
    del og, ogr
    # full size
    mbs = synth.workload_micro_batches(4)
    up = worker.upload(mbs[0])
    n = worker.accumulate_micro_batches([up, up, up, up])
    torch.cuda.synchronize()
    assert n == 128
    G4 = worker.G.cpu().numpy().copy()
    loss4 = float(worker.loss_buf.sum().item())
    loss1, g1 = gpu_micro_grad(worker, mbs[0])
    worker.close()
    assert abs(loss1 / mbs[0]["mlm_pos"].size - math.log(30522)) < 0.3
    assert abs(loss4 - 4 * loss1) / abs(4 * loss1) < 1e-5
    compare_flat(full_layout, G4, 4.0 * g1, 1e-5, "4 accumulated passes vs 4 x one pass")


@pytest.mark.gpu
@pytest.mark.parametrize("compute", ["fp32", "bf16"])
def test_update_inside_backward_gives_the_bits_of_the_separate_calls(W, compute):
    """Normalise + Adam armed for the last micro-batch's backward pass (per parameter group, beside the
    rest of the pass) against hs_grad_accum_normalize + hs_adam_step after it: identical state, two updates in a row,
    unequal micro-batches and workers without data in between."""
    from paper_2009_14783_amd import binding as hs
    Worker = W
    model = dict(n_layers=3, hidden=128, n_heads=2, ffn=512, vocab=1000, max_pos=64, ln_eps=1e-12)
    cfg = hs.make_cfg(**model)
    theta = synth.init_params(hs.hs_param_layout(cfg), 31)
    rng = synth.rng_for(77)
    mbs = [synth.make_micro_batch(rng, lens, 64, model["vocab"], "uniform") for lens in ([64, 30, 7], [64] * 5, [12])]
    adam = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)
    states = []
    for in_backward in (False, True):
        wk = Worker(model, compute, theta)
        dev = [None, wk.upload(mbs[0]), wk.upload(mbs[1]), dict(dummy=True), wk.upload(mbs[2]), None]
        for _ in range(2):
            D = wk.train_step(dev, adam, update_in_backward=in_backward)
        torch.cuda.synchronize()
        assert D == 9 and wk.t == 2
        states.append({k: getattr(wk, k).clone() for k in ("w", "m", "v", "G")} | ({"w_lowp": wk.w_lowp.clone()} if compute == "bf16" else {}))
        wk.close()
    for k in states[0]:
        assert torch.equal(states[0][k], states[1][k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("compute", ["fp32", "bf16"])
@pytest.mark.parametrize("B", [32, 33])
def test_backward_on_both_sides_of_the_few_rows_limit(W, B, compute):
    """2048 rows (gradients of up to three layers handed to the second stream at a time) and 2112 (layer by layer, two
    buffer sets), five layers so that the last hand-over is a partial one: the gradient is the sum over the two halves of the batch, and
    the update armed inside the pass gives the bits of the separate calls."""
    model = dict(n_layers=5, hidden=128, n_heads=2, ffn=256, vocab=500, max_pos=64, ln_eps=1e-12)
    layout = O.param_layout(O.ModelCfg(**model))
    theta = synth.init_params(layout, 5)
    rng = synth.rng_for(6)
    lens = [int(x) for x in rng.integers(1, 65, B)]
    mb = synth.make_micro_batch(rng, lens, 64, model["vocab"], "uniform")
    cut = B // 2
    n = int(np.searchsorted(mb["mlm_pos"], cut * 64))
    halves = [dict(mb, ids=mb["ids"][:cut], lens=mb["lens"][:cut], mlm_pos=mb["mlm_pos"][:n], mlm_label=mb["mlm_label"][:n]),
              dict(mb, ids=mb["ids"][cut:], lens=mb["lens"][cut:], mlm_pos=mb["mlm_pos"][n:] - cut * 64, mlm_label=mb["mlm_label"][n:])]
    adam = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)
    wk = W(model, compute, theta)
    _, whole = gpu_micro_grad(wk, mb)
    parts = [gpu_micro_grad(wk, h)[1].astype(np.float64) for h in halves]
    compare_flat(layout, whole, parts[0] + parts[1], TOL[compute], "whole against halves")
    wk.close()
    states = []
    for in_backward in (False, True):
        wk = W(model, compute, theta)
        wk.train_step([wk.upload(mb)], adam, update_in_backward=in_backward)
        torch.cuda.synchronize()
        states.append({k: getattr(wk, k).clone() for k in ("w", "m", "v", "G")})
        wk.close()
    for k in states[0]:
        assert torch.equal(states[0][k], states[1][k]), k


@pytest.mark.gpu
@pytest.mark.parametrize("compute", ["fp32", "bf16"])
@pytest.mark.parametrize("B,L", [(3, 24), (11, 48), (9, 232)])
def test_grouped_gradients_on_ragged_tiles(W, B, L, compute):
    """Widths of 192 and 320 and 72, 528 and 2088 rows: the grouped weight and bias gradients end inside a tile in both directions and
    their contraction inside a k-tile."""
    model = dict(n_layers=2, hidden=192, n_heads=3, ffn=320, vocab=520, max_pos=256, ln_eps=1e-12)
    ocfg = O.ModelCfg(**model)
    theta = synth.init_params(O.param_layout(ocfg), 8)
    rng = synth.rng_for(9)
    mb = synth.make_micro_batch(rng, [L] + [int(x) for x in rng.integers(1, L + 1, B - 1)], L, model["vocab"], "uniform")
    worker = W(model, compute, theta)
    loss, g = gpu_micro_grad(worker, mb)
    ol, og = oracle_micro_grad(ocfg, theta, mb, np.float64)
    assert abs(loss - ol) / abs(ol) < TOL[compute]
    compare_flat(O.param_layout(ocfg), g, og, TOL[compute], "grad")
    worker.close()


@pytest.mark.gpu
def test_grouped_gradients_on_ragged_wide_tiles(W):
    """Widths of 448 and 8256 and 2016 rows, three layers handed over together: the grouped launch takes its 256 x 256 tiles, which end inside
    both widths, and adds the bias gradients in them."""
    model = dict(n_layers=3, hidden=448, n_heads=7, ffn=8256, vocab=200, max_pos=96, ln_eps=1e-12)
    ocfg = O.ModelCfg(**model)
    theta = synth.init_params(O.param_layout(ocfg), 12)
    rng = synth.rng_for(13)
    mb = synth.make_micro_batch(rng, [96] + [int(x) for x in rng.integers(1, 97, 20)], 96, model["vocab"], "uniform")
    worker = W(model, "bf16", theta)
    loss, g = gpu_micro_grad(worker, mb)
    ol, og = oracle_micro_grad(ocfg, theta, mb, np.float32)
    assert abs(loss - ol) / abs(ol) < TOL["bf16"]
    compare_flat(O.param_layout(ocfg), g, og, TOL["bf16"], "grad")
    worker.close()


@pytest.mark.gpu
@pytest.mark.parametrize("hidden,ffn", [(320, 1088), (448, 1088)])
def test_grouped_gradients_on_ragged_middle_tiles(W, hidden, ffn):
    """1032 rows and three layers handed over together: the grouped launch takes 128 x 128 tiles at widths of 320 and 1088 and 256 x 128 tiles
    at 448 and 1088, which end inside the widths in both directions, and adds the bias gradients in them; written, then added to."""
    model = dict(n_layers=3, hidden=hidden, n_heads=hidden // 64, ffn=ffn, vocab=200, max_pos=24, ln_eps=1e-12)
    ocfg = O.ModelCfg(**model)
    theta = synth.init_params(O.param_layout(ocfg), 12)
    rng = synth.rng_for(14)
    mb = synth.make_micro_batch(rng, [24] + [int(x) for x in rng.integers(1, 25, 42)], 24, model["vocab"], "uniform")
    worker = W(model, "bf16", theta)
    loss, g = gpu_micro_grad(worker, mb)
    ol, og = oracle_micro_grad(ocfg, theta, mb, np.float32)
    assert abs(loss - ol) / abs(ol) < TOL["bf16"]
    compare_flat(O.param_layout(ocfg), g, og, TOL["bf16"], "grad")
    worker.forward_backward(worker.upload(mb), worker.G, 1, 0)
    torch.cuda.synchronize()
    compare_flat(O.param_layout(ocfg), worker.G.cpu().numpy() - g, og, TOL["bf16"], "added")
    worker.close()


@pytest.mark.gpu
@pytest.mark.parametrize("compute", ["fp32", "bf16"])
@pytest.mark.parametrize("layers", [1, 2, 9])
def test_backward_gives_the_same_bits_in_every_workspace_it_accepts(W, layers, compute):
    """A batch of few rows in the workspace of its own size, of larger batches and in the smallest that is accepted: how many layers the
    backward pass hands over at once (and so how its buffer sets are used again) follows the workspace, the results do not.
    One byte less is refused before anything is launched."""
    from paper_2009_14783_amd import binding as hs
    model = dict(n_layers=layers, hidden=256, n_heads=4, ffn=1024, vocab=500, max_pos=64, ln_eps=1e-12)
    theta = synth.init_params(O.param_layout(O.ModelCfg(**model)), 5)
    rng = synth.rng_for(6)
    mb = synth.make_micro_batch(rng, [int(x) for x in rng.integers(1, 65, 16)], 64, model["vocab"], "uniform")
    adam = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)
    wk = W(model, compute, theta)
    d = wk.upload(mb)
    own = hs.hs_workspace_bytes(wk.cfg, 16, 64, d["M"])
    assert own <= hs.hs_workspace_bytes(wk.cfg, 33, 64, d["M"]) <= hs.hs_workspace_bytes(wk.cfg, 64, 64, d["M"])
    wk.forward_backward(d, wk.G, 0, 0)
    lo, hi = 0, own                        # the smallest accepted size: refused calls launch nothing
    while hi - lo > 1:
        mid = (lo + hi) // 2
        try:
            hs.hs_encoder_bwd(wk.ctx, wk.w_compute, wk._acts, d["ids"], d["lens"], 16, 64, wk._dhidden, wk.G, 0, wk._ws, mid)
            hi = mid
        except hs.HsError as e:
            assert e.status == 3
            lo = mid
    torch.cuda.synchronize()
    wk.close()
    states = []
    for size in [hi + (own - hi) * k // 6 for k in range(7)] + [4 * own]:
        wk = W(model, compute, theta)
        d = wk.upload(mb)
        wk._ws = torch.full((max(size, own),), 255, dtype=torch.uint8, device="cuda")
        for armed in (False, True):        # the head's calls need more than the smallest size: only the backward pass is given it
            w = wk.w_compute
            hs.hs_encoder_fwd(wk.ctx, w, d["ids"], d["lens"], d["lens_host"], 16, 64, wk._acts, wk._hidden, wk._ws, wk._ws.numel())
            hs.hs_mlm_loss(wk.ctx, w, wk._hidden, d["mlm_pos"], d["mlm_label"], d["M"], 16, 64, wk.loss_buf, wk._dhidden, wk.G, 0, wk._ws,
                           wk._ws.numel())
            if armed:
                hs.hs_arm_update(wk.ctx, wk.w, wk.m, wk.v, wk.G, wk.w_lowp, 16.0, adam["lr"], adam["beta1"], adam["beta2"], adam["eps"], 0.01, 1)
            hs.hs_encoder_bwd(wk.ctx, w, wk._acts, d["ids"], d["lens"], 16, 64, wk._dhidden, wk.G, 0, wk._ws, size)
            torch.cuda.synchronize()
            states.append((armed, {k: getattr(wk, k).clone() for k in ("w", "m", "v", "G")}))
        wk.close()
    for armed, s in states[2:]:
        for k in s:
            assert torch.equal(s[k], states[int(armed)][1][k]), (armed, k)
