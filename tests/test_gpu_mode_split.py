"""The forward row pass takes one mode a workgroup in launches of at most 320
workgroups of whole items (row blocks per tile x positions), all modes of an item
in larger ones: the same bits either way, alone or beside a request with another
number of modes."""
import numpy as np
import pytest

from paper_2505_14372_amd import api, synth

from _cases import Case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _case(N, M, S, scan, seed=4):
    return Case(synth.make_small(N=N, M=M, S=S, scan=scan, step=2, seed=seed, loss="poisson", eps=0.8, amp_noise=0.2))


@pytest.mark.parametrize("N,M,pieces", [(192, 3, (53, 1, 10)), (192, 2, (54, 9, 1)), (256, 3, (20, 5, 11)),
                                        (256, 2, (21, 1, 14))])
def test_forward_pieces_equal_the_whole(N, M, pieces):
    """(192 x 192: 6 row blocks, 53 positions the most of a split launch;
    256 x 256: 16 row blocks, 20 positions.)"""
    c = _case(N, M, 3, 8)
    d = c.device()
    prob = c.problem()
    batch = d["batch"][:sum(pieces)].contiguous()
    whole, _ = prob.forward(d["probe"], d["obj"], d["pos"], batch)
    parts = [prob.forward(d["probe"], d["obj"], d["pos"], b.contiguous())[0] for b in batch.split(pieces)]
    prob.check()
    assert torch.equal(whole, torch.cat(parts))


@pytest.mark.parametrize("N", [192, 256])
def test_grouped_requests_with_other_mode_counts(N):
    """Grouped, the launch is large enough to keep whole items together (or, at
    256 x 256, not); each request alone is split, or has one mode."""
    cases = [_case(N, 3, 3, 4, 6), _case(N, 1, 2, 7, 7)]
    opt = api.Optimizer(kind="adam", lr_object=1e-3, lr_probe=1e-3, lr_pos=1e-2)
    states = []
    for grouped in (False, True):
        entries = []
        for c in cases:
            d = c.device()
            prob = c.problem()
            prob.set_reduction("ordered")
            st = api.ReconState(d["probe"].clone(), d["obj"].clone(), d["pos"].clone())
            entries.append((prob, st, d["pats"], d["batch"], opt, torch.zeros(1, dtype=torch.float64, device="cuda")))
        if grouped:
            n = [len(c.batch) for c in cases]
            grp = api.Group(N, sum(n), 3 * n[0] + n[1], 9 * n[0] + 2 * n[1])
            grp.step(entries)
        else:
            for prob, st, pats, b, o, loss in entries:
                prob.reconstruct_step(st, pats, b, o, loss=loss)
        torch.cuda.synchronize()
        states.append(entries)
    for alone, grouped in zip(*states):
        for f in ("object", "probe", "positions"):
            assert torch.equal(getattr(alone[1], f), getattr(grouped[1], f)), f
        assert alone[5].item() == grouped[5].item()
