"""The whole-step kernel of small full-precision models against the oracle and against the per-op kernels: row lengths of one, two, four
and more pieces, rows that do not divide among the waves, head dimensions and groups, contexts at the edges of the key tiles and of the
waves' rounds, pages of other sizes, masks, batches, and a wait that gives up."""
import pytest
import torch

import paper_2410_12513_amd as P
from oracle import first_oracle as O
from synth import make_prompt
from synth.generators import ModelDesc
from tests.gpu_util import build, logits_close, top2_gap

pytestmark = pytest.mark.gpu
torch.set_grad_enabled(False)

HD64 = ModelDesc(3, 256, 4, 2, 64, 696, 1001, dtype="fp32")
HD128 = ModelDesc(3, 512, 4, 1, 128, 1032, 500, dtype="fp32")
WIDE = ModelDesc(3, 512, 8, 8, 64, 2048, 77, dtype="fp32")
NARROW = ModelDesc(3, 72, 2, 1, 64, 96, 67, dtype="fp32")
VOCAB = ModelDesc(2, 256, 4, 2, 64, 696, 16384, dtype="fp32")
OPT_DECODE_PATH, OPT_STEP_POLL_LIMIT, OPT_SMALL_EPOCH = 3, 10, 11


def _prefilled(desc, prompts, seed, page=16, room=16, path=-1, max_seq_len=None):
    n = [p.numel() for p in prompts]
    _, w, r, ctx = build(None, seed, desc=desc, max_batch=len(prompts), max_seq_len=max_seq_len or max(n) + room, page=page)
    ctx.set_option(OPT_DECODE_PATH, path)
    tok = torch.zeros(len(prompts), dtype=torch.int32, device="cuda")
    ctx.prefill_route(torch.cat(prompts).cuda(), n, token=tok)
    return w, r, ctx, tok


def _waits_between_workgroups(ctx, tok):
    """Does a step of this context take the whole-step kernel?  Only that one has waits that a poll limit of 0 makes give up."""
    ctx.set_option(OPT_STEP_POLL_LIMIT, 0)
    ctx.decode_step(tok, None, tok.clone())
    try:
        ctx.sync()
    except P.FirstError as e:
        assert e.code == -4 and "gave up" in str(e)
        return True
    ctx.set_option(OPT_STEP_POLL_LIMIT, -1)
    return False


@pytest.mark.parametrize("desc,n,mask,page,max_seq_len", [
    (HD64, 1, [1, 1, 1], 16, None), (HD64, 30, [1, 0, 1], 16, None), (HD64, 127, [1, 1, 1], 16, None), (HD64, 290, [0, 1, 1], 24, None),
    (HD128, 14, [1, 1, 1], 16, None), (HD128, 63, [1, 0, 1], 8, None), (HD128, 140, [1, 1, 0], 16, None), (WIDE, 40, [1, 1, 1], 16, None),
    (NARROW, 33, [1, 1, 1], 16, None), (HD64, 20, [0, 0, 0], 16, None), (HD64, 20, [1, 1, 1], 16, 2056),
    (HD64, 2040, [1, 1, 1], 16, 2048), (HD128, 2040, [0, 1, 1], 16, 2048), (VOCAB, 25, [1, 1], 16, None),
    (VOCAB.with_(vocab=16385), 25, [1, 1], 16, None)])
def test_steps_match_the_oracle_and_the_per_op_kernels(desc, n, mask, page, max_seq_len):
    prompt = make_prompt(desc.vocab, n, 91)
    w, r, ctx, tok = _prefilled(desc, [prompt], 91, page, max_seq_len=max_seq_len)
    _, _, ops, _ = _prefilled(desc, [prompt], 91, page, path=0)
    st = O.prefill_route(desc, w, r, prompt)
    assert int(tok[0]) == st.token or top2_gap(st.logits) < 4e-4
    for c in (ctx, ops):
        c.set_mask(0, mask)
    st.set_mask(mask)
    fed = torch.tensor([st.token], dtype=torch.int32, device="cuda")
    lg, lo, out = torch.zeros(1, desc.vocab, device="cuda"), torch.zeros(1, desc.vocab, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    for step in range(6):
        ctx.decode_step(fed, lg if step != 2 else None, out)
        ops.decode_step(fed, lo, out.clone())
        ctx.sync(), ops.sync()
        ref, ref_tok = O.decode_step(desc, w, st, int(fed[0]))
        if step != 2:
            ok, worst, rel = logits_close(lg[0], ref, "fp32")
            assert ok, (step, worst, rel)
            # the same products, other orders of fp32 sums: a few units in the last place of each of some thousand terms
            assert float((lg - lo).norm() / lo.norm()) <= 1e-5
        if top2_gap(ref) > 4e-4:
            assert int(out[0]) == ref_tok
        fed[0] = ref_tok
    assert ctx.seq_len(0) == n + 6
    h, ho = ctx.get_hidden(), ops.get_hidden()
    assert torch.equal(h, ho) if not any(mask) else float((h - ho).norm() / ho.norm()) <= 1e-5
    for i, keep in enumerate(mask):
        for a, b in zip(ctx.kv_read(0, i, 0, n + 6 if keep else n), ops.kv_read(0, i, 0, n + 6 if keep else n)):
            assert float((a - b).norm()) <= 1e-5 * float(b.norm())
    if any(mask):                                       # (without a layer only one workgroup waits, for the others' candidates)
        assert _waits_between_workgroups(ctx, fed) == ((max_seq_len or 0) <= 2048 and desc.vocab <= 16384)
    assert not _waits_between_workgroups(ops, fed)
    ctx.close(), ops.close()


def test_a_batch_has_the_bits_of_each_sequence_alone():
    prompts = [make_prompt(HD64.vocab, n, 92 + n) for n in (9, 150, 40)]
    masks = [[1, 0, 1], [1, 1, 1], [0, 1, 0]]
    _, _, ctx, tok = _prefilled(HD64, prompts, 92)
    lg = torch.zeros(3, HD64.vocab, device="cuda")
    for b, m in enumerate(masks):
        ctx.set_mask(b, m)
    first, hist = tok.clone(), []
    for _ in range(5):
        ctx.decode_step(tok, lg, tok)
        ctx.sync()
        hist.append((tok.clone(), lg.clone()))
    for b, (p, m) in enumerate(zip(prompts, masks)):
        _, _, one, t = _prefilled(HD64, [p], 92, max_seq_len=166)
        assert int(t[0]) == int(first[b])
        one.set_mask(0, m)
        l1 = torch.zeros(1, HD64.vocab, device="cuda")
        for tokens, logits in hist:
            one.decode_step(t, l1, t)
            one.sync()
            assert int(t[0]) == int(tokens[b]) and torch.equal(l1[0], logits[b])
        one.close()
    ctx.close()


@pytest.mark.parametrize("mask", [[1, 1, 1], [0, 1, 0]])
def test_the_exchange_counter_passes_its_largest_value(mask):
    """Three steps from every place before the end of the counter's 32 bits from which one of their first two exchanges passes it: the same
    logits, hidden states and keys as from the counter's start."""
    n, per_step = 40, 5 * sum(mask) + 1
    prompt = make_prompt(HD64.vocab, n, 93)
    _, _, ctx, tok = _prefilled(HD64, [prompt], 93)
    ctx.set_mask(0, mask)
    fed = torch.tensor([[3], [700], [41]], dtype=torch.int32, device="cuda")
    lg, outs = torch.zeros(3, 1, HD64.vocab, device="cuda"), {}
    for back in [0] + list(range(1, 2 * per_step + 2)):
        ctx.set_option(OPT_SMALL_EPOCH, -back)                  # 2^32 - back
        ctx.set_seq_len(0, n)
        lg.zero_()
        for t, out in zip(fed, lg):
            ctx.decode_step(t, out, tok)
        ctx.sync()
        outs[back] = (lg.clone(), ctx.get_hidden().clone(), torch.stack(ctx.kv_read(0, 1, n, 3)))
        assert all(torch.equal(a, b) for a, b in zip(outs[back], outs[0])), back
    ctx.close()


def test_a_wait_that_gives_up_ends_the_launch_and_is_reported_once():
    """A poll limit of 0, set from the host: every first unsuccessful poll gives up and every workgroup leaves."""
    prompt = make_prompt(HD64.vocab, 50, 94)
    outs = []
    for provoke in (False, True):
        _, _, ctx, tok = _prefilled(HD64, [prompt], 94)
        if provoke:
            ctx.set_option(OPT_STEP_POLL_LIMIT, 0)
            ctx.decode_step(tok, None, tok.clone())
            with pytest.raises(P.FirstError) as e:
                ctx.sync()
            assert e.value.code == -4 and "gave up" in str(e.value)
            ctx.sync()
            ctx.prefill_route(prompt.cuda(), [50], token=tok)
        lg, hist = torch.zeros(1, HD64.vocab, device="cuda"), []
        for _ in range(6):
            ctx.decode_step(tok, lg, tok)
            ctx.sync()
            hist.append((int(tok[0]), lg.clone()))
        outs.append(hist)
        ctx.close()
    for (ta, la), (tb, lb) in zip(*outs):
        assert ta == tb and torch.equal(la, lb)


@pytest.mark.parametrize("heads,kv_heads,hd,width", [(1, 1, 64, 256), (3, 1, 64, 200), (4, 4, 64, 256), (2, 1, 128, 256), (3, 3, 128, 72), (4, 2, 64, 264), (5, 5, 64, 256)])
@pytest.mark.parametrize("n", [1, 63, 300])
def test_output_projection_by_head_and_by_row(heads, kv_heads, hd, width, n):
    """One to four heads and a thread an element: every group of workgroups has a head's columns of the output projection (1, 3 heads: groups that do not
    divide the 64 workgroups or the rows); 264 wide or five heads: the heads' outputs go round.  Against the launches per op: the same fp32 products, other orders of
    sums (a few units in the last place of some thousand terms)."""
    desc = ModelDesc(2, width, heads, kv_heads, hd, 264, 300, dtype="fp32")
    prompt = make_prompt(desc.vocab, n, 95)
    ctxs = [_prefilled(desc, [prompt], 95, path=p)[2] for p in (-1, 0)]
    tok, lg = torch.zeros(1, dtype=torch.int32, device="cuda"), [torch.zeros(1, desc.vocab, device="cuda") for _ in ctxs]
    for c in ctxs:
        c.set_mask(0, [1, 1])
    for step in range(4):
        tok.fill_(7 + 50 * step)
        for c, out in zip(ctxs, lg):
            c.decode_step(tok, out, tok.clone())
            c.sync()
        assert float((lg[0] - lg[1]).norm() / lg[1].norm()) <= 1e-5
    assert _waits_between_workgroups(ctxs[0], tok) and not _waits_between_workgroups(ctxs[1], tok)
    for c in ctxs:
        c.close()
