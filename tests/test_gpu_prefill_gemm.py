"""The prompt pass's projections at the edges of their tiles, K steps and slices: prefill and soft-skip forward (which gives every
row) of a one-layer model against the oracle, three times over (the slices of K meet in memory in any order and must give
the same bits each time)."""
import pytest
import torch

from oracle import first_oracle as O
from oracle import training_forward as TF
from synth import make_prompt, make_router, make_weights
from synth.generators import ModelDesc, to_device

# widths that are not multiples of the K step (64): Q/K/V, gate / up and down end in a partial step (the output projection's K is
# always a number of whole heads)
RAGGED = ModelDesc(1, 520, 6, 2, 64, 1416, 500)
# the same with K in four segments; at 256 compute units 100, 300, 500, 807 and 1500 rows take the four tiles, with four slices of K,
# two or none (200 rows: 64 x 128 with four)
RAGGED_WIDE = ModelDesc(1, 3080, 18, 3, 128, 2312, 500)
# a K long enough for many slices, and an N for the widest tile
WIDE = ModelDesc(1, 1024, 8, 4, 128, 4096, 700)


MATRICES = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")


def _shift(w, names=MATRICES):
    """The same weights with the matrices called names at addresses that are not multiples of 16 bytes."""
    def moved(v):
        buf = torch.empty(v.numel() + 4, dtype=v.dtype, device=v.device)
        buf[4:].copy_(v.reshape(-1))
        return buf[4:].view(v.shape)

    out = dict(w, layers=[{k: moved(v) if k in names else v for k, v in lw.items()} for lw in w["layers"]])
    for k in ("embed", "lm_head"):
        out[k] = moved(w[k]) if k in names else w[k]
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("desc,n,shifted", [(RAGGED, 1, False), (RAGGED, 31, False), (RAGGED, 33, False), (RAGGED, 65, True), (RAGGED, 129, False),
                                            (RAGGED, 500, False), (WIDE, 32, False), (WIDE, 200, False), (WIDE, 200, True), (WIDE, 257, False),
                                            (WIDE, 1100, False), (RAGGED_WIDE, 100, False), (RAGGED_WIDE, 200, False), (RAGGED_WIDE, 300, False), (RAGGED_WIDE, 500, False), (RAGGED_WIDE, 807, False), (RAGGED_WIDE, 1500, False)])
def test_prefill_projections_at_tile_edges(desc, n, shifted):
    import paper_2410_12513_amd as P
    w, r, prompt = make_weights(desc, 11), make_router(desc, 11), make_prompt(desc.vocab, n, 11)
    wg = to_device(w, "cuda")
    ctx = P.FirstContext(desc, _shift(wg) if shifted else wg, r.cuda(), max_batch=1, max_seq_len=n + 1)
    ref = O.prefill_route(desc, w, r, prompt)
    soft = TF.soft_forward(desc, w, r, prompt)[0]
    ids, runs = prompt.cuda(), []
    for _ in range(3):
        hidden, logits, rho = torch.zeros(1, desc.d_model, device="cuda"), torch.zeros(1, desc.vocab, device="cuda"), torch.zeros(1, 1, device="cuda")
        rows, terms = torch.zeros(n, desc.d_model, device="cuda"), torch.zeros(1, 4, device="cuda")
        ctx.prefill_route(ids, [n], rho=rho, hidden=hidden, logits=logits)
        ctx.soft_forward(ids, [n], ids, 0.0, 0.0, terms, hidden=rows)
        runs.append((hidden[0].cpu(), logits[0].cpu(), rows.cpu()))
    ctx.close()
    for h, l, rows in runs:
        # activations carry 16 bits into the products (2^-17 each); what is left is K, V values that round to the other
        # neighbouring bf16 (2^-9 of a value, few of them): well below 1.5e-3 of the stream, while one 32 x 32 block of a
        # projection that misses a slice of K is 1e-2 and more
        assert float((h.double() - ref.hidden).norm() / ref.hidden.norm()) <= 1.5e-3
        assert float((l.double() - ref.logits.double()).norm() / ref.logits.double().norm()) <= 1.5e-3
        assert float(((rows.double() - soft).norm(dim=1) / soft.norm(dim=1)).max()) <= 1.5e-3
        assert all(torch.equal(x, y) for x, y in zip((h, l, rows), runs[0]))


# widths that are no multiples of the large tiles nor of their K steps; at 256 compute units: 256 x 256 tiles in gate / up (700 rows) and
# in Q/K/V (1300); then the down projection's 128 x 192 and 128 x 256 tiles with four slices of K (330, 390 rows) and two (700, 900)
MANY_HEADS = ModelDesc(1, 1032, 64, 8, 128, 9000, 500)
LONG_DOWN = ModelDesc(1, 3080, 4, 2, 64, 8200, 500)
DOWN = ModelDesc(1, 3080, 4, 2, 64, 4104, 500)


@pytest.mark.gpu
@pytest.mark.parametrize("desc,n", [(MANY_HEADS, 700), (MANY_HEADS, 1300), (LONG_DOWN, 330), (LONG_DOWN, 390), (DOWN, 700), (LONG_DOWN, 900)])
def test_prefill_projections_in_large_tiles(desc, n):
    test_prefill_projections_at_tile_edges(desc, n, False)


@pytest.mark.gpu
@pytest.mark.parametrize("names", [("embed", "lm_head"), ("wo",), ("w_up",)])
def test_a_matrix_off_16_bytes_leaves_the_other_products_alone(names):
    """The loads that need 16 bytes are a matter of the matrices of one launch.  K and V of the first layer do not see the output
    projection nor the MLP, and the last hidden state does not see the LM head: they keep their bits, also where the launch they
    come from sums K in segments and the kernel for unaligned matrices does not (2048 columns of input)."""
    import paper_2410_12513_amd as P
    desc = ModelDesc(1, 2048, 4, 2, 64, 2304, 500)
    w, r, prompt = to_device(make_weights(desc, 12), "cuda"), make_router(desc, 12).cuda(), make_prompt(desc.vocab, 70, 12)
    got = []
    for ws in (w, _shift(w, names)):
        hidden = torch.zeros(1, desc.d_model, device="cuda")
        ctx = P.FirstContext(desc, ws, r, max_batch=1, max_seq_len=80)
        ctx.prefill_route(prompt.cuda(), [70], hidden=hidden)
        got.append((hidden.cpu(),) + tuple(t.cpu() for t in ctx.kv_read(0, 0, 0, 70)))
        ctx.close()
    (h0, k0, v0), (h1, k1, v1) = got
    assert torch.equal(k0, k1) and torch.equal(v0, v1)
    if "lm_head" in names:
        assert torch.equal(h0, h1)
    else:      # the shifted launch: other sums of fp32 products, 2^-17 of an activation each
        assert float((h0 - h1).norm() / h0.norm()) <= 1e-5
