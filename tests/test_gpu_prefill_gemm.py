"""The prompt pass's projections at the edges of their tiles, K steps and slices: prefill of a one-layer model against the
oracle, three times over (the slices of K meet in memory in any order and must give the same bits each time)."""
import pytest
import torch

from oracle import first_oracle as O
from synth import make_prompt, make_router, make_weights
from synth.generators import ModelDesc, to_device

# widths that are not multiples of the K step (64), so every contraction ends in a partial step
RAGGED = ModelDesc(1, 520, 6, 2, 64, 1416, 500)
# a K long enough for many slices, and an N for the widest tile
WIDE = ModelDesc(1, 1024, 8, 4, 128, 4096, 700)


def _shift(w):
    """The same matrices at addresses that are not multiples of 16 bytes."""
    out = dict(w, layers=[])
    for lw in w["layers"]:
        moved = {}
        for k, v in lw.items():
            if v.dtype == torch.bfloat16:
                buf = torch.empty(v.numel() + 4, dtype=v.dtype, device=v.device)
                buf[4:].copy_(v.reshape(-1))
                v = buf[4:].view(v.shape)
            moved[k] = v
        out["layers"].append(moved)
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("desc,n,shifted", [(RAGGED, 1, False), (RAGGED, 31, False), (RAGGED, 33, False), (RAGGED, 65, True), (RAGGED, 129, False),
                                            (RAGGED, 500, False), (WIDE, 32, False), (WIDE, 200, False), (WIDE, 257, False), (WIDE, 1100, False)])
def test_prefill_projections_at_tile_edges(desc, n, shifted):
    import paper_2410_12513_amd as P
    w, r, prompt = make_weights(desc, 11), make_router(desc, 11), make_prompt(desc.vocab, n, 11)
    wg = to_device(w, "cuda")
    ctx = P.FirstContext(desc, _shift(wg) if shifted else wg, r.cuda(), max_batch=1, max_seq_len=n + 1)
    ref = O.prefill_route(desc, w, r, prompt)
    runs = []
    for _ in range(3):
        hidden, logits, rho = torch.zeros(1, desc.d_model, device="cuda"), torch.zeros(1, desc.vocab, device="cuda"), torch.zeros(1, 1, device="cuda")
        ctx.prefill_route(prompt.cuda(), [n], rho=rho, hidden=hidden, logits=logits)
        runs.append((hidden[0].cpu(), logits[0].cpu()))
    ctx.close()
    for h, l in runs:
        # activations carry 16 bits into the products (2^-17 each); what is left is K, V values that round to the other
        # neighbouring bf16 (2^-9 of a value, few of them): well below 1.5e-3 of the stream, while one 32 x 32 block of a
        # projection that misses a slice of K is 1e-2 and more
        assert float((h.double() - ref.hidden).norm() / ref.hidden.norm()) <= 1.5e-3
        assert float((l.double() - ref.logits.double()).norm() / ref.logits.double().norm()) <= 1.5e-3
        assert torch.equal(h, runs[0][0]) and torch.equal(l, runs[0][1])
