"""The probe-spectrum sum takes a thread per pixel where there are many pixels and
few items, else sixteen: each request of a group that is summed the one way has the
bits of its step alone, which is summed the other way (or the same, from 262144
pixels on). Item counts around the sixteen interleaved sums and their fours; final
passes that leave the sums themselves (256 x 256, 4 modes and more)."""
import pytest

from paper_2505_14372_amd import api, synth

from _cases import Case, max_rel, rel_l2

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _case(N, M, B, seed):
    scan = 5
    return Case(synth.make_small(N=N, M=M, S=1, scan=scan, step=2, seed=seed, loss="poisson", eps=0.8, amp_noise=0.2),
                batch=list(range(B)))


@pytest.mark.parametrize("N,strategy,parts", [
    (64, "auto", [(2, 3), (1, 1), (3, 8), (2, 5), (1, 16), (5, 17), (4, 10)]),
    (64, "two_pass", [(2, 3), (1, 1), (3, 8), (2, 5), (1, 16), (5, 17), (4, 10)]),
    (128, "auto", [(1, 2), (2, 15), (3, 21)]), (192, "auto", [(1, 7), (2, 18)]),
    (256, "auto", [(1, 9), (2, 12)]), (256, "auto", [(5, 3), (4, 17), (1, 20)])])
def test_requests_of_a_group_have_the_bits_of_their_steps_alone(N, strategy, parts):
    opt = api.Optimizer(kind="sgd", lr_object=1e-4, lr_probe=1e-3, lr_pos=1e-4)
    entries, alone = [], []
    for q, (M, B) in enumerate(parts):
        c = _case(N, M, B, 50 + q)
        d = c.device()
        prob = c.problem()
        prob.set_strategy(strategy)
        prob.set_reduction("ordered")
        one, many = (api.ReconState(d["probe"].clone(), d["obj"].clone(), d["pos"].clone(), adam=False) for _ in range(2))
        alone.append((one, prob.reconstruct_step(one, d["pats"], d["batch"], opt)))
        entries.append((prob, many, d["pats"], d["batch"], opt, torch.zeros(1, dtype=torch.float64, device="cuda")))
        assert not torch.equal(one.probe, d["probe"])
    tiles = sum(M * B for M, B in parts)
    api.Group(N, sum(B for _, B in parts), tiles, tiles).step(entries)
    torch.cuda.synchronize()
    for (one, loss), entry in zip(alone, entries):
        assert loss.item() == entry[5].item()
        for f in ("object", "probe", "positions"):
            assert torch.equal(getattr(one, f), getattr(entry[1], f)), f


@pytest.mark.parametrize("N,M,B", [(192, 8, 6), (256, 2, 21), (256, 5, 19)])
def test_probe_gradient_matches_oracle(N, M, B):
    c = _case(N, M, B, 60)
    d = c.device()
    ref = c.oracle_grad()
    _, _, gP, _ = c.problem().loss_and_grad(d["probe"], d["obj"], d["pos"], d["pats"], d["batch"])
    got = gP.cpu().numpy()
    assert rel_l2(got, ref["g_probe"]) < 1e-3 and max_rel(got, ref["g_probe"]) < 1e-3
