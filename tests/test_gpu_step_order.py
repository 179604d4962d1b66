"""Contexts on streams of their own whose decode steps wait between workgroups: steps enqueued a few microseconds behind each other, without a
synchronisation between them, give each context the bits that it has alone.  Persistent steps need the whole chip, those of small fp32 models
64 places beside them, or, where a persistent kernel's LDS leaves none, the chip without it."""
import threading

import pytest
import torch

import paper_2410_12513_amd as P
from synth import CONFIGS, ModelDesc, make_prompt, make_router, make_weights
from synth.generators import to_device

pytestmark = pytest.mark.gpu
torch.set_grad_enabled(False)

STEPS, PROMPT = 60, 90


SMALL = ModelDesc(3, 256, 4, 2, 64, 696, 1001, dtype="fp32")
NO_ROOM = ModelDesc(1, 2048, 128, 32, 128, 14336, 1000, dtype="bf16")        # 146 KB of LDS a workgroup


def _context(model, seed, stream=None):
    desc = model if isinstance(model, ModelDesc) else CONFIGS[model]
    ctx = P.FirstContext(desc, to_device(make_weights(desc, seed), "cuda"), make_router(desc, seed).cuda(), max_batch=1,
                         max_seq_len=PROMPT + STEPS + 1, stream=stream)
    if desc.dtype == "bf16":
        ctx.set_option(3, 1)                            # the persistent kernel or an error
    tok = torch.zeros(1, dtype=torch.int32, device="cuda")
    prompt = make_prompt(desc.vocab, PROMPT, seed).cuda()
    torch.cuda.synchronize()
    ctx.prefill_route(prompt, [PROMPT], token=tok)
    ctx.set_mask(0, [1] * desc.n_layers)
    hist = torch.zeros(STEPS, 1, desc.vocab, device="cuda")
    torch.cuda.synchronize()
    return ctx, tok, hist


def _steps(ctx, tok, hist, use_graph):
    ctx.set_option(1, use_graph)
    for out in hist:
        ctx.decode_step(tok, out, tok)


@pytest.mark.parametrize("use_graph", [1, 0])
@pytest.mark.parametrize("streams", ["private", "caller's", "threads"])
@pytest.mark.parametrize("models", [[("step_hd128", 21), ("step_hd64", 22), ("step_hd128", 23)],
                                    [("step_hd128", 21)] + [(SMALL, 30 + i) for i in range(6)],
                                    [(NO_ROOM, 26), (SMALL, 30), (SMALL, 31), ("step_hd64", 22)]], ids=["persistent", "beside", "no room"])
def test_steps_of_contexts_on_different_streams(use_graph, streams, models):
    alone = []
    for model, seed in models:
        ctx, tok, hist = _context(model, seed)
        _steps(ctx, tok, hist, use_graph)
        ctx.sync()
        alone.append((int(tok[0]), hist))
        ctx.close()
    own = [torch.cuda.Stream() if streams == "caller's" else None for _ in models]
    together = [_context(m, s, st) for (m, s), st in zip(models, own)]
    if streams == "threads":
        threads = [threading.Thread(target=_steps, args=(*c, use_graph)) for c in together]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    else:
        for ctx, _, _ in together:
            ctx.set_option(1, use_graph)
        for i in range(STEPS):
            for ctx, tok, hist in together:
                ctx.decode_step(tok, hist[i], tok)
    for (ctx, tok, hist), (last, ref) in zip(together, alone):
        ctx.sync()                                      # raises if a wait between workgroups gave up
        assert int(tok[0]) == last and torch.equal(hist, ref)
        ctx.close()


def test_a_context_that_comes_while_another_one_decodes():
    """The first context's steps leave no events as long as it is alone: those under way when the second one comes are waited for too."""
    ref = []
    for seed in (24, 25):
        ctx, tok, hist = _context("step_hd128", seed)
        _steps(ctx, tok, hist, 0)
        ctx.sync()
        ref.append(hist)
        ctx.close()
    a, tok_a, hist_a = _context("step_hd128", 24, torch.cuda.Stream())
    a.set_option(1, 0)
    for out in hist_a[:STEPS // 2]:
        a.decode_step(tok_a, out, tok_a)
    b, tok_b, hist_b = _context("step_hd128", 25, torch.cuda.Stream())
    b.set_option(1, 0)
    for i in range(STEPS // 2):
        a.decode_step(tok_a, hist_a[STEPS // 2 + i], tok_a)
        b.decode_step(tok_b, hist_b[i], tok_b)
    a.sync()
    assert torch.equal(hist_a, ref[0])
    a.close()
    for out in hist_b[STEPS // 2:]:                     # alone again
        b.decode_step(tok_b, out, tok_b)
    b.sync()
    assert torch.equal(hist_b, ref[1])
    b.close()
