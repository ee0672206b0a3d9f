"""Packed rows (hs_set_lengths): passes over the real positions only against passes over the padded batch."""
import numpy as np
import pytest
import torch

from paper_2009_14783_amd import binding as hs
from paper_2009_14783_amd import synth
from paper_2009_14783_amd.step import PairWorker, Worker

pytestmark = pytest.mark.gpu

# Both passes form the same sums of the same bf16 values; the products run in other tiles and the weight gradients add their rows in another
# order, so that single activations round the other way (2^-9 each): the bound of every bf16 gradient against the oracle.
TOL = 2e-2


def rel(a, b):
    a, b = a.double(), b.double()
    return float((a - b).norm() / b.norm().clamp_min(1e-12))


def real_and_padding(hidden, lens, L):
    h = hidden.view(len(lens), L, -1)
    real = torch.cat([h[b, :n] for b, n in enumerate(lens)])
    pad = torch.cat([h[b, n:] for b, n in enumerate(lens)])
    return real.float(), pad.float()


# lengths of 1 and of L, tiles and 128-row blocks that end inside a sequence, one sequence, passes in one part and in two halves (4096 real
# rows and more) whose cut is not the middle sequence, both attention backward kernels, one width per register plan of the LayerNorm backward
@pytest.mark.parametrize("hidden,B,L,lens,p", [
    (256, 6, 128, [1, 128, 33, 97, 64, 2], 0.0), (256, 6, 128, [1, 128, 33, 97, 64, 2], 0.1), (128, 1, 64, [5], 0.1), (256, 5, 256, [256, 1, 129, 128, 40], 0.1),
    (768, 70, 96, None, 0.1), (512, 40, 200, None, 0.0), (1024, 3, 56, [56, 7, 55], 0.1)])
def test_encoder_pass_over_real_rows(hidden, B, L, lens, p):
    model = dict(n_layers=2, hidden=hidden, n_heads=hidden // 64, ffn=2 * hidden, vocab=1000, max_pos=256, ln_eps=1e-12)
    lens = lens or [max(1, L - (b * b) // 40) for b in range(B)]
    theta = synth.init_params(hs.hs_param_layout(hs.make_cfg(**model)), 71)
    mb = synth.make_micro_batch(synth.rng_for(72), lens, L, model["vocab"], "zipf")
    wk = Worker(model, "bf16", theta)
    d = wk.upload(dict(mb, drop=dict(p=p, seed=9, stream=3) if p else None))
    out = []
    for use in (dict(d, lens_host=None), d):      # without lengths on the host: padded rows
        wk.G.fill_(float("nan"))
        wk._hidden.fill_(float("nan"))
        wk.forward_backward(use, wk.G, 0, 0)
        torch.cuda.synchronize()
        out.append((float(wk.loss_buf[0]), wk.G.clone(), *real_and_padding(wk._hidden[:B * L * hidden], lens, L)))
    (l0, g0, h0, _), (l1, g1, h1, pad) = out
    assert abs(l0 - l1) / abs(l0) < 1e-3 and rel(h1, h0) < TOL, (l0, l1, rel(h1, h0))
    assert bool((pad == 0).all())
    for name, off, r, c in hs.hs_param_layout(hs.make_cfg(**model)):
        assert rel(g1[off:off + r * c], g0[off:off + r * c]) < TOL, name
    wk.forward_backward(d, wk.G, 0, 0)            # the same bits again
    torch.cuda.synchronize()
    assert torch.equal(wk.G, g1)
    wk.close()


@pytest.mark.parametrize("B,Ls,Lt,p", [(5, 24, 32, 0.0), (3, 136, 72, 0.1), (130, 32, 40, 0.1)])
def test_pair_pass_over_real_rows(B, Ls, Lt, p):
    model = dict(n_enc=2, n_dec=2, hidden=128, n_heads=2, ffn=256, vocab=500, max_pos=160)
    sl, tl = [max(1, Ls - 3 * (b % 9)) for b in range(B)], [max(1, Lt - 5 * (b % 7)) for b in range(B)]
    sl[0], tl[-1] = 1, 1
    layout = hs.hs_s2s_param_layout(hs.make_s2s_cfg(**model))
    wk = PairWorker(model, "bf16", synth.init_params(layout, 73))
    mb = synth.make_pair_batch(synth.rng_for(74), sl, tl, Ls, Lt, model["vocab"], "uniform")
    d = wk.upload(dict(mb, drop=dict(p=p, seed=8, stream=5) if p else None))
    out = []
    for use in (dict(d, packable=False), d):
        wk.G.fill_(float("nan"))
        wk._out.fill_(float("nan"))
        wk.forward_backward(use, wk.G, 0, 0)
        torch.cuda.synchronize()
        out.append((float(wk.loss_buf[0]), wk.G.clone(), *real_and_padding(wk._out[:B * Lt * 128], tl, Lt)))
    (l0, g0, h0, _), (l1, g1, h1, pad) = out
    assert abs(l0 - l1) / abs(l0) < 1e-3 and rel(h1, h0) < TOL
    assert bool((pad == 0).all())
    # per stack and not per tensor: a ReLU gate within rounding of zero that falls the other way moves a small tensor by more than the bound
    for stack in ("emb", "enc0", "enc1", "dec0", "dec1"):
        at = [slice(off, off + r * c) for name, off, r, c in layout if name.startswith(stack)]
        assert rel(torch.cat([g1[s] for s in at]), torch.cat([g0[s] for s in at])) < TOL, stack
    wk.close()


def test_gradient_rows_of_the_padding_are_not_read():
    model = dict(n_layers=1, hidden=128, n_heads=2, ffn=256, vocab=200, max_pos=64, ln_eps=1e-12)
    wk = Worker(model, "bf16", synth.init_params(hs.hs_param_layout(hs.make_cfg(**model)), 75))
    lens, L = [64, 9, 30], 64
    d = wk.upload(synth.make_micro_batch(synth.rng_for(76), lens, L, 200, "uniform"))
    wk.forward_backward(d, wk.G, 0, 0)
    torch.cuda.synchronize()
    want = wk.G.clone()
    hs.hs_set_lengths(wk.ctx, d["lens_host"], 3, L)
    hs.hs_encoder_fwd(wk.ctx, wk.w_compute, d["ids"], d["lens"], None, 3, L, wk._acts, wk._hidden, wk._ws, wk._ws_bytes)
    hs.hs_mlm_loss(wk.ctx, wk.w_compute, wk._hidden, d["mlm_pos"], d["mlm_label"], d["M"], 3, L, wk.loss_buf, wk._dhidden, wk.G, 0, wk._ws, wk._ws_bytes)
    dh = wk._dhidden[:3 * L * 128].view(3, L, 128)
    for b, n in enumerate(lens):
        dh[b, n:] = float("nan")
    hs.hs_encoder_bwd(wk.ctx, wk.w_compute, wk._acts, d["ids"], d["lens"], 3, L, wk._dhidden, wk.G, 0, wk._ws, wk._ws_bytes)
    torch.cuda.synchronize()
    assert torch.equal(wk.G, want)
    wk.close()


def same_state(a, b, names):
    for k in names:
        assert torch.equal(getattr(a, k), getattr(b, k)), k


# 33000 x 128 parameters and more: the embedding's rows that the last micro-batch does not hold are updated in front of its backward pass, up to 4096 rows
@pytest.mark.parametrize("compute,B,L", [("bf16", 5, 24), ("bf16", 34, 128), ("fp32", 3, 32)])
def test_embedding_rows_updated_in_two_parts_give_the_bits_of_one(compute, B, L):
    model = dict(n_layers=2, hidden=128, n_heads=2, ffn=256, vocab=33001, max_pos=128, ln_eps=1e-12)
    theta = synth.init_params(hs.hs_param_layout(hs.make_cfg(**model)), 77)
    a, b = Worker(model, compute, theta), Worker(model, compute, theta)
    adam = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8, weight_decay=0.01)
    for t in range(2):
        mbs = [synth.make_micro_batch(synth.rng_for(78 + 2 * t + i), [max(1, L - 3 * (k % 7)) for k in range(B)], L, model["vocab"], "zipf") for i in range(2)]
        mbs[1]["ids"][0, :2] = [0, model["vocab"] - 1]
        a.train_step([a.upload(mb) for mb in mbs], adam)
        b.train_step([b.upload(mb) for mb in mbs], adam, update_in_backward=False)
        torch.cuda.synchronize()
        same_state(a, b, ("w", "m", "v", "G") + (("w_lowp",) if compute == "bf16" else ()))
    a.close(); b.close()


@pytest.mark.parametrize("compute,B,Ls,Lt", [("bf16", 4, 24, 32), ("bf16", 130, 32, 40), ("fp32", 3, 16, 24)])
def test_pair_step_of_a_large_model_gives_the_bits_of_the_separate_update(compute, B, Ls, Lt):
    model = dict(n_enc=2, n_dec=2, hidden=128, n_heads=2, ffn=256, vocab=33001, max_pos=64)
    theta = synth.init_params(hs.hs_s2s_param_layout(hs.make_s2s_cfg(**model)), 79)
    a, b = PairWorker(model, compute, theta), PairWorker(model, compute, theta)
    adam = dict(lr=1e-3, beta1=0.9, beta2=0.98, eps=1e-9)
    for t in range(2):
        lens = lambda L, k: [max(1, L - k * (i % 5)) for i in range(B)]
        mbs = [synth.make_pair_batch(synth.rng_for(80 + 2 * t + i), lens(Ls, 3), lens(Lt, 4), Ls, Lt, model["vocab"], "zipf") for i in range(2)]
        D = a.train_step([a.upload(mb) for mb in mbs], adam)
        for i, mb in enumerate(mbs):
            b.forward_backward(b.upload(mb), b.G, i, i)
        hs.hs_normalize_adam_step(b.w, b.m, b.v, b.G, b.w_lowp, b.P, D, adam["lr"], adam["beta1"], adam["beta2"], adam["eps"], 0.0, t + 1)
        torch.cuda.synchronize()
        same_state(a, b, ("w", "m", "v", "G") + (("w_lowp",) if compute == "bf16" else ()))
    a.close(); b.close()


def with_guards(wk, *names):
    """Replaces the worker's byte arenas by ones with 1 MiB of a pattern behind them; returns a check that it is all there."""
    ends = []
    for name in names:
        old = getattr(wk, name)
        n = old.numel() * old.element_size()
        new = torch.full((n + (1 << 20),), 0xA5, dtype=torch.uint8, device="cuda")
        setattr(wk, name, new if old.dtype == torch.uint8 else new.view(old.dtype))
        ends.append(new[n:])
    return lambda: all(bool((e == 0xA5).all()) for e in ends)


# `lens` on the device that no longer are the lengths the host was told, with a larger and a smaller sum, in one part and in two halves: NaN and not
# plausible numbers, every buffer kept, and the right lengths give the right bits again
@pytest.mark.parametrize("B,L", [(6, 64), (48, 128)])
@pytest.mark.parametrize("p", [0.0, 0.1])
def test_lengths_on_the_device_that_are_not_the_host_s(B, L, p):
    model = dict(n_layers=2, hidden=128, n_heads=2, ffn=256, vocab=500, max_pos=128, ln_eps=1e-12)
    wk = Worker(model, "bf16", synth.init_params(hs.hs_param_layout(hs.make_cfg(**model)), 81))
    lens = [max(1, L - (b % 5) * 6) for b in range(B)]
    assert (sum(lens) >= 4096) == (B == 48)
    d = wk.upload(dict(synth.make_micro_batch(synth.rng_for(82), lens, L, 500, "uniform"), drop=dict(p=p, seed=9, stream=3) if p else None))
    kept = with_guards(wk, "_acts", "_ws", "_hidden", "_dhidden")
    wk.forward_backward(d, wk.G, 0, 0)
    torch.cuda.synchronize()
    want, right = wk.G.clone(), d["lens"].clone()
    assert bool(torch.isfinite(want).all())
    for wrong in (torch.full_like(right, L), torch.ones_like(right), right.clamp(max=L // 2), torch.where(torch.arange(B, device="cuda") < B // 2, L, right)):
        d["lens"].copy_(wrong)
        wk.G.zero_()
        wk.forward_backward(d, wk.G, 0, 0)
        torch.cuda.synchronize()
        assert kept() and bool(torch.isnan(wk.G).any())
    d["lens"].copy_(right)
    wk.forward_backward(d, wk.G, 0, 0)
    torch.cuda.synchronize()
    assert kept() and torch.equal(wk.G, want)
    wk.close()


@pytest.mark.parametrize("B,Ls,Lt", [(5, 32, 24), (130, 40, 48)])
def test_pair_lengths_on_the_device_that_are_not_the_host_s(B, Ls, Lt):
    model = dict(n_enc=2, n_dec=2, hidden=128, n_heads=2, ffn=256, vocab=500, max_pos=160)
    wk = PairWorker(model, "bf16", synth.init_params(hs.hs_s2s_param_layout(hs.make_s2s_cfg(**model)), 83))
    sl, tl = [max(1, Ls - 3 * (b % 6)) for b in range(B)], [max(1, Lt - 2 * (b % 7)) for b in range(B)]
    d = wk.upload(synth.make_pair_batch(synth.rng_for(84), sl, tl, Ls, Lt, 500, "uniform"))
    kept = with_guards(wk, "_acts", "_ws", "_out", "_dout")
    wk.forward_backward(d, wk.G, 0, 0)
    torch.cuda.synchronize()
    want = wk.G.clone()
    assert bool(torch.isfinite(want).all())
    for side, L in (("src_lens", Ls), ("tgt_lens", Lt)):
        right = d[side].clone()
        for wrong in (torch.full_like(right, L), torch.ones_like(right), right.clamp(max=L // 2)):
            d[side].copy_(wrong)
            wk.G.zero_()
            wk.forward_backward(d, wk.G, 0, 0)
            torch.cuda.synchronize()
            assert kept() and bool(torch.isnan(wk.G).any())
        d[side].copy_(right)
    wk.forward_backward(d, wk.G, 0, 0)
    torch.cuda.synchronize()
    assert kept() and torch.equal(wk.G, want)
    wk.close()


@pytest.mark.parametrize("compute", ["bf16", "fp32"])
def test_targets_in_the_padding_keep_the_padded_rows(compute):
    """A target at a padded position has a hidden state and a gradient in the padded passes; packed rows have none."""
    model = dict(n_layers=2, hidden=128, n_heads=2, ffn=256, vocab=200, max_pos=64, ln_eps=1e-12)
    wk = Worker(model, compute, synth.init_params(hs.hs_param_layout(hs.make_cfg(**model)), 85))
    mb = synth.make_micro_batch(synth.rng_for(86), [64, 9, 30], 64, 200, "uniform")
    mb["mlm_pos"] = np.array([3, 64 + 8, 64 + 9, 64 + 40, 128 + 29], np.int32)      # the third and the fourth are padding
    mb["mlm_label"] = np.arange(5, dtype=np.int32)
    d = wk.upload(mb)
    out = []
    for use in (dict(d, lens_host=None), d):
        wk.G.fill_(float("nan"))
        wk.forward_backward(use, wk.G, 0, 0)
        torch.cuda.synchronize()
        out.append((wk.loss_buf[:1].clone(), wk.G.clone()))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1]) and bool(torch.isfinite(out[0][1]).all())
    wk.close()


def test_packable_batches():
    model = dict(n_layers=1, hidden=128, n_heads=2, ffn=256, vocab=200, max_pos=64, ln_eps=1e-12)
    wk = Worker(model, "bf16", synth.init_params(hs.hs_param_layout(hs.make_cfg(**model)), 87))
    def packable(lens, pos):
        mb = dict(ids=np.ones((len(lens), 16), np.int32), lens=np.array(lens, np.int32), mlm_pos=np.array(pos, np.int32), mlm_label=np.zeros(len(pos), np.int32))
        return wk.upload(mb)["packable"]
    assert packable([16, 5], [0, 15, 16, 20]) and packable([1, 1], []) and packable([1, 1], [0, 16])
    assert not packable([16, 5], [0, 21]) and not packable([16, 5], [32]) and not packable([16, 16], [32]) and not packable([16, 5], [-1])
    assert not packable([], [])
    wk.close()


@pytest.mark.parametrize("vocab,by_size", [(33001, True), (500, False)])
def test_pair_step_has_the_form_that_it_was_asked_for(monkeypatch, vocab, by_size):
    """update_in_backward: True and False force the form at any size, None goes by it; the same bits in every form."""
    model = dict(n_enc=1, n_dec=1, hidden=128, n_heads=2, ffn=256, vocab=vocab, max_pos=64)
    theta = synth.init_params(hs.hs_s2s_param_layout(hs.make_s2s_cfg(**model)), 88)
    mb = synth.make_pair_batch(synth.rng_for(89), [16, 9], [24, 5], 16, 24, vocab, "zipf")
    arm, armed, out = hs.hs_arm_update, [], []
    monkeypatch.setattr(hs, "hs_arm_update", lambda *a: (armed.append(1), arm(*a)))
    for form, want in ((True, True), (False, False), (None, by_size)):
        wk = PairWorker(model, "bf16", theta)
        armed.clear()
        wk.train_step([wk.upload(mb)], dict(lr=1e-3, beta1=0.9, beta2=0.98, eps=1e-9), update_in_backward=form)
        torch.cuda.synchronize()
        assert bool(armed) == want
        out.append((wk.w.clone(), wk.m.clone(), wk.v.clone(), wk.G.clone(), wk.w_lowp.clone()))
        wk.close()
    for other in out[1:]:
        assert all(torch.equal(a, b) for a, b in zip(out[0], other))


# a pass over 4096 real rows and more runs as two halves, whose cut (19 of 40) is not the middle sequence: masks numbered from the second half's first
# sequence in the attention, by position in the products and the embedding
@pytest.mark.parametrize("hidden,B,L,step", [(512, 40, 200, 40), (256, 70, 96, 150)])
def test_encoder_halves_over_real_rows_with_dropout(hidden, B, L, step):
    lens = [max(1, L - (b * b) // step) for b in range(B)]
    assert 4096 <= sum(lens) < B * L
    first = np.concatenate([[0], np.cumsum(lens)])
    assert int(np.argmin(abs(2 * first - first[-1]))) != B // 2
    test_encoder_pass_over_real_rows(hidden, B, L, lens, 0.1)


def replays_equal_eager(step, state, refill, eager, n=4):
    """Captures step(); every replay, with state restored and refill(k) in front, must leave what eager(k) leaves."""
    saved = [t.clone() for t in state]
    step()                                             # streams, events and tables that the first call makes
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for k in range(n):
        for t, s in zip(state, saved):
            t.copy_(s)
        refill(k)
        graph.replay()
        torch.cuda.synchronize()
        got = [t.clone() for t in state]
        for a, b in zip(got, eager(k)):
            assert bool(torch.isfinite(a).all()) and torch.equal(a, b), k


STATE = ("w", "m", "v", "G", "w_lowp")


@pytest.mark.parametrize("B,L", [(6, 64), (48, 128)])
def test_captured_step_reads_the_lengths_of_its_replay(B, L):
    """A captured step keeps the padded rows: its replays take ids and lengths that are on the device by then.  One part and two halves."""
    model = dict(n_layers=2, hidden=128, n_heads=2, ffn=256, vocab=33001, max_pos=128, ln_eps=1e-12)
    theta = synth.init_params(hs.hs_param_layout(hs.make_cfg(**model)), 90)
    adam = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-8)
    batch = lambda k: dict(synth.make_micro_batch(synth.rng_for(91 + k), [max(1, L - (3 + k) * (b % 7)) for b in range(B)], L, 33001, "zipf"),
                           mlm_pos=np.arange(B, dtype=np.int32) * L, mlm_label=np.arange(B, dtype=np.int32), drop=dict(p=0.1, seed=9, stream=3))
    a, b = Worker(model, "bf16", theta), Worker(model, "bf16", theta)
    d = a.upload(batch(0))
    assert d["packable"]
    def refill(k):
        new = a.upload(batch(k))
        for name in ("ids", "lens"):
            d[name].copy_(new[name])
    def step():
        a.t = 0
        a.train_step([d], adam)
    def eager(k):
        b.t = 0
        for t, s in zip((b.w, b.m, b.v, b.w_lowp), first):
            t.copy_(s)
        b.train_step([dict(b.upload(batch(k)), lens_host=None)], adam)
        torch.cuda.synchronize()
        return [getattr(b, n) for n in STATE]
    first = [b.w.clone(), b.m.clone(), b.v.clone(), b.w_lowp.clone()]
    replays_equal_eager(step, [getattr(a, n) for n in STATE], refill, eager)
    a.close(); b.close()


# without the target lengths on the host every position goes through the projection, and replays may have others; with them the number of rows is captured
@pytest.mark.parametrize("B,Ls,Lt", [(5, 24, 32), (130, 32, 40)])
@pytest.mark.parametrize("host_lens", [False, True])
def test_captured_pair_step_reads_the_lengths_of_its_replay(B, Ls, Lt, host_lens):
    model = dict(n_enc=2, n_dec=2, hidden=128, n_heads=2, ffn=256, vocab=33001, max_pos=64)
    theta = synth.init_params(hs.hs_s2s_param_layout(hs.make_s2s_cfg(**model)), 92)
    adam = dict(lr=1e-3, beta1=0.9, beta2=0.98, eps=1e-9)
    def batch(k):
        sl, tl = [max(1, Ls - (2 + k) * (b % 5)) for b in range(B)], [max(1, Lt - (3 + (0 if host_lens else k)) * (b % 6)) for b in range(B)]
        return dict(synth.make_pair_batch(synth.rng_for(93 + k), sl, tl, Ls, Lt, 33001, "zipf"), drop=dict(p=0.1, seed=8, stream=5))
    keep = (lambda d: d) if host_lens else (lambda d: dict(d, tgt_lens_host=None))
    a, b = PairWorker(model, "bf16", theta), PairWorker(model, "bf16", theta)
    d = keep(a.upload(batch(0)))
    assert d["packable"]
    def refill(k):
        new = a.upload(batch(k))
        for name in ("src", "src_lens", "tgt_in", "tgt_out", "tgt_lens"):
            d[name].copy_(new[name])
    def step():
        a.t = 0
        a.train_step([d], adam, denom=1000)
    def eager(k):
        b.t = 0
        for t, s in zip((b.w, b.m, b.v, b.w_lowp), first):
            t.copy_(s)
        b.train_step([dict(keep(b.upload(batch(k))), packable=False)], adam, denom=1000)
        torch.cuda.synchronize()
        return [getattr(b, n) for n in STATE]
    first = [b.w.clone(), b.m.clone(), b.v.clone(), b.w_lowp.clone()]
    replays_equal_eager(step, [getattr(a, n) for n in STATE], refill, eager)
    a.close(); b.close()
