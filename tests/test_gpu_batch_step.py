"""All layers of a batched decode step in one kernel against the launches per op (option 3 = 0).  The oracle tests of the batched path run both."""
import pytest
import torch

import paper_2410_12513_amd as P
from synth import CONFIGS, ModelDesc, make_prompt, make_router, make_weights
from synth.generators import to_device
from tests.gpu_util import build

pytestmark = pytest.mark.gpu
torch.set_grad_enabled(False)

# Both form the same products of bf16 weights with 16-bit-split activations and add them in fp32, in another order.  That is 1e-6 of a sum, but now and
# then a key or value falls on the other side of its bf16 rounding: 2^-8 of one element, which reaches a logit as one of hundreds of terms of
# its size (logits of size 4: 2^-8 * 4 / sqrt(256) = 1e-3 a flip at most; a few of them at a time).
TOLERANCE = 3e-3
OPT_BATCH_STEP = 12                                              # 1: the one kernel wherever it can run, also where it is not the faster way


def _steps(ctx, desc, masks, n, first):
    B = len(masks[0])
    lg, tk = torch.zeros(B, desc.vocab, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda")
    tin, out = torch.zeros(B, dtype=torch.int32, device="cuda"), []
    for s in range(n):
        for b, m in enumerate(masks[s * len(masks) // n]):
            ctx.set_mask(b, m)
        tin.copy_(torch.tensor([(first + 7 * s + 13 * b) % desc.vocab for b in range(B)], dtype=torch.int32))
        ctx.decode_step(tin, lg, tk)
        ctx.sync()                                               # raises if a wait between workgroups gave up
        assert tk.tolist() == lg.argmax(dim=1).tolist()
        out.append(lg.clone())
    return torch.stack(out)


# (layers, width, heads, KV heads, head dimension, FFN width), contexts.  Workgroups without a row (32 units for 256 of them), with one or two units and with half
# tiles (288, 544), pairs of waves without a share of K, a last pass that is not whole (2304, 4352); 4, 8 and 16 slots, all used or not; one and several splits;
# contexts at the edges of pages and tiles; a split of more tiles than page ids are fetched ahead for; more items of attention than compute units; contexts that
# need two splits whatever else there is.
@pytest.mark.parametrize("shape,lens", [
    ((3, 256, 4, 2, 64, 256), [1, 16, 63, 64]),
    ((3, 256, 4, 1, 64, 512), [5, 900]),
    ((2, 768, 6, 2, 128, 1280), [15, 700, 33, 64, 1400]),
    ((3, 2304, 8, 4, 64, 4352), [20 + 170 * b for b in range(9)]),
    ((2, 512, 8, 2, 128, 2304), [3 + 11 * b for b in range(16)]),
    ((2, 1536, 12, 4, 64, 2560), [2047, 40, 9]),
    ((2, 2048, 8, 4, 128, 2048), [30] * 8),
    ((3, 2048, 4, 1, 64, 512), [1000, 30, 700]),              # (waves that merge splits and have no share of the output projection's K)
    ((2, 512, 32, 16, 64, 512), [4310] + [20 + b for b in range(15)]),      # (16 items a KV head: one split each, the first of 68 tiles)
    ((2, 512, 64, 32, 64, 512), [33 + 9 * b for b in range(16)]),           # (512 items)
    ((2, 256, 4, 2, 64, 256), [16390, 50]),
], ids=str)
@pytest.mark.parametrize("graph", [1, 0])
def test_one_kernel_agrees_with_launches_per_op(shape, lens, graph):
    desc, B, L, n = ModelDesc(*shape, 1003, dtype="bf16"), len(lens), shape[0], 8
    w, r = to_device(make_weights(desc, 5), "cuda"), make_router(desc, 5).cuda()
    ids = torch.cat([make_prompt(desc.vocab, k, 5 + b) for b, k in enumerate(lens)]).cuda()
    # every layer; a layer for some of the sequences; fewer layers (the exchange begins anew), most sequences without any
    some = [[int(i == 0 or (i + b) % 2) for i in range(L)] for b in range(B)]
    few = [[m if i == L - 1 else 0 for i, m in enumerate(row)] for row in some]
    masks = [[[1] * L] * B, some, few]
    out, kv = [], []
    for path in (0, -1):
        ctx = P.FirstContext(desc, w, r, max_batch=B, max_seq_len=max(lens) + n + 1)
        ctx.set_option(1, graph)
        ctx.set_option(3, path)
        ctx.set_option(OPT_BATCH_STEP, 1)
        for first in (3, 400):                                   # (a new prompt: every layer again)
            ctx.prefill_route(ids, lens)
            out.append(_steps(ctx, desc, masks, n, first))
            kv.append([ctx.kv_read(b, i, lens[b], 3) for b in range(B) for i in range(L)])
        ctx.close()
    for i in (0, 1):
        assert float((out[i] - out[2 + i]).abs().max()) <= TOLERANCE
        assert not torch.equal(out[i], out[2 + i])               # (the same bits would come of the same kernels)
        for x, y in zip(kv[i], kv[2 + i]):
            for p, q in zip(x, y):                               # (bf16 roundings that fall on the other side)
                assert float((p.double() - q.double()).norm() / p.double().norm()) <= 2 ** -8


def test_batched_and_single_steps_on_streams_of_their_own():
    """Kernels that each need the whole chip, and small fp32 models' between them, which then have no room, a few microseconds behind each other: each context has
    the bits that it has alone."""
    def contexts():
        out = []
        for model, lens in (("step_hd128", [40, 21, 300]), ("step_hd64", [70]), ("mini_fp32", [60]), ("step_g2", [90] * 5), ("mini_fp32", [31])):
            desc, _, _, ctx = build(model, 11, max_batch=len(lens), max_seq_len=400)
            ctx.set_option(OPT_BATCH_STEP, 1)
            ctx.prefill_route(torch.cat([make_prompt(desc.vocab, k, 5 + b) for b, k in enumerate(lens)]).cuda(), lens)
            for b in range(len(lens)):
                ctx.set_mask(b, [1] * desc.n_layers)
            out.append((ctx, torch.full((len(lens),), 9, dtype=torch.int32, device="cuda"), torch.zeros(40, len(lens), desc.vocab, device="cuda")))
        torch.cuda.synchronize()
        return out
    alone = contexts()
    for ctx, tok, hist in alone:
        for lg in hist:
            ctx.decode_step(tok, lg, tok)
        ctx.sync()
    together = contexts()
    for i in range(40):
        for ctx, tok, hist in together:
            ctx.decode_step(tok, hist[i], tok)
    for (ctx, tok, hist), (c, t, ref) in zip(together, alone):
        ctx.sync()
        assert torch.equal(hist, ref) and torch.equal(tok, t)
        ctx.close()
        c.close()


def test_a_captured_step_takes_the_launches_per_op():
    desc = CONFIGS["step_hd64"]
    lens, stream = [50, 20, 33], torch.cuda.Stream()
    w, r = to_device(make_weights(desc, 5), "cuda"), make_router(desc, 5).cuda()
    ids, out = torch.cat([make_prompt(desc.vocab, k, b) for b, k in enumerate(lens)]).cuda(), []
    for captured in (False, True):
        ctx = P.FirstContext(desc, w, r, max_batch=3, max_seq_len=100, stream=stream)
        ctx.set_option(1, 0)
        ctx.set_option(OPT_BATCH_STEP, 1)
        torch.cuda.synchronize()
        ctx.prefill_route(ids, lens)
        for b in range(3):
            ctx.set_mask(b, [1] * desc.n_layers)
        tok, lg, hist = torch.full((3,), 9, dtype=torch.int32, device="cuda"), torch.zeros(3, desc.vocab, device="cuda"), []
        torch.cuda.synchronize()
        if captured:
            g = torch.cuda.CUDAGraph()
            with torch.cuda.graph(g, stream=stream):
                ctx.decode_step(tok, lg, tok)
        else:
            ctx.set_option(3, 0)
        for _ in range(4):
            if captured:
                with torch.cuda.stream(stream):
                    g.replay()
            else:
                ctx.decode_step(tok, lg, tok)
            stream.synchronize()
            hist.append(lg.clone())
            torch.cuda.synchronize()
        if not captured:
            ctx.sync()
        out.append(torch.stack(hist))
        ctx.close()
    assert torch.equal(*out)


@pytest.mark.parametrize("sampled", [False, True])
@pytest.mark.parametrize("shape,lens", [((3, 256, 4, 1, 64, 512), [5, 900, 40]), ((2, 768, 6, 2, 128, 1280), [15, 700, 33, 64, 1400])], ids=str)
def test_a_wait_that_gives_up_stops_everything_until_it_is_reported(shape, lens, sampled):
    """A poll limit of 0, set from the host: every first unsuccessful poll gives up and every workgroup leaves.  Until the error has been reported, once, later steps
    change no logits, no tokens and no lengths; after a new prompt the context has the bits of an untouched twin."""
    desc, B = ModelDesc(*shape, 1003, dtype="bf16"), len(lens)
    w, r = to_device(make_weights(desc, 6), "cuda"), make_router(desc, 6).cuda()
    ids = torch.cat([make_prompt(desc.vocab, k, 6 + b) for b, k in enumerate(lens)]).cuda()
    u = torch.linspace(0.1, 0.9, B, device="cuda")
    hist = []
    for provoke in (False, True):
        ctx = P.FirstContext(desc, w, r, max_batch=B, max_seq_len=max(lens) + 20)
        ctx.set_option(OPT_BATCH_STEP, 1)
        lg, tk, tin = torch.zeros(B, desc.vocab, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda"), torch.full((B,), 9, dtype=torch.int32, device="cuda")

        def step():
            if sampled:
                ctx.decode_step_sampled(tin, u, 1.0, 10, lg, tk)
            else:
                ctx.decode_step(tin, lg, tk)

        def prompt():
            ctx.prefill_route(ids, lens)
            for b in range(B):
                ctx.set_mask(b, [1] * desc.n_layers)
        prompt()
        for graph in (1, 0) if provoke else ():
            ctx.set_option(1, graph)
            for _ in range(3):                                   # (an odd number: the next launch takes the other set of words)
                step()
            ctx.sync()
            lg.fill_(-77.)
            tk.fill_(-7)
            ctx.set_option(10, 0)
            for _ in range(3):
                step()
            torch.cuda.synchronize()
            assert bool((lg == -77.).all()) and bool((tk == -7).all())
            with pytest.raises(P.FirstError) as e:
                ctx.sync()
            assert e.value.code == -4 and "gave up" in str(e.value)
            assert [ctx.seq_len(b) for b in range(B)] == [k + 3 for k in lens]
            prompt()
        ctx.set_option(1, 1)
        hist.append([])
        for _ in range(6):
            step()
            ctx.sync()
            hist[-1].append((lg.clone(), tk.clone()))
        ctx.close()
    for (la, ta), (lb, tb) in zip(*hist):
        assert torch.equal(la, lb) and torch.equal(ta, tb)


def test_as_many_sets_of_buffers_as_before_keep_their_graphs():
    """Seventeen output buffers in turn, which meet both sets of exchange words: once each has been through both, a step neither captures nor waits for
    the stream.  The stream is busy when the steps are enqueued, and still is when they have been."""
    desc, lens, stream, n = ModelDesc(2, 256, 4, 2, 64, 512, 1003, dtype="bf16"), [20, 33, 7], torch.cuda.Stream(), 17
    w, r = to_device(make_weights(desc, 7), "cuda"), make_router(desc, 7).cuda()
    ctx = P.FirstContext(desc, w, r, max_batch=3, max_seq_len=120, stream=stream)
    ctx.set_option(OPT_BATCH_STEP, 1)
    torch.cuda.synchronize()
    ctx.prefill_route(torch.cat([make_prompt(desc.vocab, k, b) for b, k in enumerate(lens)]).cuda(), lens)
    for b in range(3):
        ctx.set_mask(b, [1] * desc.n_layers)
    tok, lg, out = torch.full((3,), 9, dtype=torch.int32, device="cuda"), torch.zeros(n, 3, desc.vocab, device="cuda"), torch.zeros(n, 3, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    for i in range(2 * n):
        ctx.decode_step(tok, lg[i % n], out[i % n])
    ctx.sync()
    busy = torch.cuda.Event()
    with torch.cuda.stream(stream):
        torch.cuda._sleep(200_000_000)
        busy.record(stream)
    for i in range(n):
        ctx.decode_step(tok, lg[i], out[i])
    assert not busy.query()
    ctx.sync()
    assert ctx.seq_len(0) == lens[0] + 3 * n
    ctx.close()


def test_sequences_and_layers_that_come_and_go():
    """Sixteen sequences, three, nine, sixteen again in one context, with more and with fewer layers kept than before: the exchange lies elsewhere every time, and
    only what was written is emptied in between."""
    desc, steps = ModelDesc(6, 512, 8, 4, 64, 768, 1003, dtype="bf16"), 5
    w, r = to_device(make_weights(desc, 8), "cuda"), make_router(desc, 8).cuda()
    out = []
    for path in (0, -1):
        ctx = P.FirstContext(desc, w, r, max_batch=16, max_seq_len=420)
        ctx.set_option(3, path)
        ctx.set_option(OPT_BATCH_STEP, 1)
        for turn, B in enumerate((16, 3, 9, 16, 2)):
            lens = [5 + 37 * ((b + turn) % 11) for b in range(B)]
            ctx.prefill_route(torch.cat([make_prompt(desc.vocab, k, turn + b) for b, k in enumerate(lens)]).cuda(), lens)
            kept = ((2, 1), (6, 4), (5, 3), (3, 3), (6, 1))[turn]  # layers that somebody keeps, at first and later
            masks = [[[int(i < k and (b == 0 or i == 0 or (i + b) % 3 != 1)) for i in range(6)] for b in range(B)] for k in kept]
            out.append(_steps(ctx, desc, masks, steps, 11 * turn))
        ctx.close()
    for a, b in zip(out[:5], out[5:]):
        assert float((a - b).abs().max()) <= TOLERANCE and not torch.equal(a, b)


@pytest.mark.parametrize("width,ffn,heads,lens,first", [
    (512, 1536, 8, [40, 300, 9], 2),                             # 14 us to gain, 9 a layer
    (2560, 1024, 20, [40, 300, 9], 7),                           # 320 units of rows on 256 compute units: 2 a layer
    (2560, 1024, 20, [900, 700, 800], 3),                        # ... and 3 more where sequences are split
], ids=str)
def test_few_layers_take_the_launches(width, ffn, heads, lens, first):
    """From `first` kept layers on a step has the bits of the one kernel, with fewer those of the launches per op."""
    if torch.cuda.get_device_properties(0).multi_processor_count != 256:
        pytest.skip("the numbers of layers are those of 256 compute units")
    desc, B = ModelDesc(8, width, heads, heads // 4, 64, ffn, 1003, dtype="bf16"), len(lens)
    w, r = to_device(make_weights(desc, 9), "cuda"), make_router(desc, 9).cuda()
    ids = torch.cat([make_prompt(desc.vocab, k, 9 + b) for b, k in enumerate(lens)]).cuda()
    masks, out = [[[int(i < k) for i in range(8)]] * B for k in (8, first, first - 1)], []
    for path, force in ((0, 0), (-1, 0), (-1, 1)):
        ctx = P.FirstContext(desc, w, r, max_batch=B, max_seq_len=max(lens) + 10)
        ctx.set_option(3, path)
        ctx.set_option(OPT_BATCH_STEP, force)
        kept = []
        for m in masks:
            ctx.prefill_route(ids, lens)
            kept.append(_steps(ctx, desc, [m], 3, 5))
        out.append(kept)
        ctx.close()
    launches, auto, one = out
    assert all(not torch.equal(a, b) for a, b in zip(launches, one))
    assert [torch.equal(a, b) for a, b in zip(auto, one)] == [True, True, False] and torch.equal(auto[2], launches[2])


def test_sampled_steps_draw_from_the_logits_of_the_one_kernel():
    desc, lens = ModelDesc(3, 512, 8, 2, 64, 768, 1003, dtype="bf16"), [40, 300, 9, 65, 20]
    w, r, B = to_device(make_weights(desc, 10), "cuda"), make_router(desc, 10).cuda(), len(lens)
    ids = torch.cat([make_prompt(desc.vocab, k, 10 + b) for b, k in enumerate(lens)]).cuda()
    u, out = torch.linspace(0.05, 0.95, B, device="cuda"), []
    for path in (0, -1):
        ctx = P.FirstContext(desc, w, r, max_batch=B, max_seq_len=320)
        ctx.set_option(3, path)
        ctx.set_option(OPT_BATCH_STEP, 1)
        ctx.prefill_route(ids, lens)
        for b in range(B):
            ctx.set_mask(b, [1] * desc.n_layers)
        lg, cand, drawn = torch.zeros(B, desc.vocab, device="cuda"), torch.zeros(B, 10, dtype=torch.int32, device="cuda"), torch.zeros(B, 10, dtype=torch.int32, device="cuda")
        tk, again = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda")
        for s in range(6):
            fed = torch.tensor([(3 + 7 * s + 13 * b) % desc.vocab for b in range(B)], dtype=torch.int32, device="cuda")
            ctx.decode_step_sampled(fed, u, 0.8, 10, lg, tk, cand)
            ctx.sync()
            P.sample_top_k_static(lg, u, 0.8, 10, again, drawn)
            torch.cuda.synchronize()
            assert torch.equal(tk, again) and torch.equal(cand, drawn)
            out.append(lg.clone())
        ctx.close()
    assert float((torch.stack(out[:6]) - torch.stack(out[6:])).abs().max()) <= TOLERANCE and not torch.equal(out[0], out[6])
