"""Passes of at most 512 workgroups at 192 x 192 exchange whole values between the
lanes of a line, larger ones real and imaginary parts in turn: the same bits from a
batch and its pieces, and from reconstructions alone and grouped, on both sides of
the line (6 column blocks a tile, fewer with a band limit; 6 row blocks)."""
import numpy as np
import pytest

from paper_2505_14372_amd import api, synth

from _cases import Case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _case(M, S, B, seed, **kw):
    scan = int(np.ceil(np.sqrt(B)))
    wl = synth.make_small(N=192, M=M, S=S, scan=scan, step=2, seed=seed, loss="poisson", eps=0.8, amp_noise=0.2, **kw)
    return Case(wl, batch=np.arange(B))


@pytest.mark.parametrize("M,pieces,bandlimit", [(1, (85, 1, 4), 2.0 / 3.0), (1, (40, 86), 0.0), (3, (29, 28, 30), 0.0)])
def test_forward_pieces_equal_the_whole(M, pieces, bandlimit):
    c = _case(M, 3, sum(pieces), 4, bandlimit=bandlimit)
    d = c.device()
    prob = c.problem()
    whole, _ = prob.forward(d["probe"], d["obj"], d["pos"], d["batch"])
    parts = [prob.forward(d["probe"], d["obj"], d["pos"], b.contiguous())[0] for b in d["batch"].split(pieces)]
    prob.check()
    assert torch.equal(whole, torch.cat(parts))


@pytest.mark.parametrize("parts", [[(1, 2, 50), (1, 3, 60)], [(2, 3, 20), (3, 2, 25)]])
def test_grouped_requests_have_the_bits_of_their_steps_alone(parts):
    opt = api.Optimizer(kind="adam", lr_object=1e-3, lr_probe=1e-3, lr_pos=1e-2)
    entries, alone = [], []
    for q, (M, S, B) in enumerate(parts):
        c = _case(M, S, B, 20 + q)
        d = c.device()
        prob = c.problem()
        prob.set_reduction("ordered")
        one, many = (api.ReconState(d["probe"].clone(), d["obj"].clone(), d["pos"].clone()) for _ in range(2))
        alone.append((one, prob.reconstruct_step(one, d["pats"], d["batch"], opt)))
        entries.append((prob, many, d["pats"], d["batch"], opt, torch.zeros(1, dtype=torch.float64, device="cuda")))
    tiles = sum(M * B for M, _, B in parts)
    api.Group(192, sum(B for *_, B in parts), tiles, sum(M * S * B for M, S, B in parts)).step(entries)
    torch.cuda.synchronize()
    for (one, loss), entry in zip(alone, entries):
        assert loss.item() == entry[5].item()
        for f in ("object", "probe", "positions"):
            assert torch.equal(getattr(one, f), getattr(entry[1], f)), f
