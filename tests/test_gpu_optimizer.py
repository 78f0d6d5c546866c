"""The optimiser launch of a step: every variable's update in one launch, against the update formulas in float64 from the gradients of loss_and_grad.
Buffers at 16-byte boundaries and off them, counts that are no multiple of four,
the step count on the host and on the device, a frozen probe, SGD, and grouped
steps whose requests share one state."""
import numpy as np
import pytest

from paper_2505_14372_amd import api, synth

from _cases import Case

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

U = 2.0 ** -24
VARS = (("object", "lr_object"), ("probe", "lr_probe"), ("positions", "lr_pos"))


def _case(N, seed=3):
    return Case(synth.make_small(N=N, M=2, S=2, scan=3, step=3, seed=seed, loss="poisson", eps=0.8, amp_noise=0.2))


def _off(t, by):
    """A copy of t that starts `by` elements into its storage."""
    s = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    s[by:] = t.reshape(-1)
    return s[by:].view(t.shape)


def _state(d, by, device_step, step):
    st = api.ReconState(_off(d["probe"], by), _off(d["obj"], by), _off(d["pos"], by), device_step=device_step)
    gen = torch.Generator(device="cpu").manual_seed(7)
    for name in ("m_object", "m_probe", "m_pos", "v_object", "v_probe", "v_pos"):
        t = getattr(st, name)
        r = torch.randn(t.shape, generator=gen) * 0.1
        setattr(st, name, _off((r.square() if name[0] == "v" else r).to(t.device), by))
    if device_step:
        st.step_dev.fill_(step)
    else:
        st.step = step
    return st


def _real(t):
    return (torch.view_as_real(t) if t.is_complex() else t).detach().cpu().numpy().astype(np.float64).ravel()


def _read(st):
    return {v: (_real(getattr(st, v)), _real(getattr(st, "m_" + v.replace("positions", "pos"))),
                _real(getattr(st, "v_" + v.replace("positions", "pos")))) for v, _ in VARS}


def _adam(x, g, lr, t, o):
    """Updated (th, m, v) and the float32 rounding bound of each: at most 16
    roundings between the first moment and the update, two in each product sum."""
    th, m0, v0 = x
    m, v = o.beta1 * m0 + (1 - o.beta1) * g, o.beta2 * v0 + (1 - o.beta2) * g * g
    d = lr / (1 - o.beta1 ** t) / (np.sqrt(v / (1 - o.beta2 ** t)) + o.eps)
    em = 4 * U * (np.abs(o.beta1 * m0) + np.abs((1 - o.beta1) * g))
    new = th - d * m
    return (new, m, v), (2 * U * np.abs(new) + d * (em + 16 * U * np.abs(m)), em, 8 * U * v)


@pytest.mark.parametrize("N,strategy,by,device_step,kind,lr_probe",
                         [(64, "auto", 0, False, "adam", 2e-3), (64, "auto", 1, True, "adam", 2e-3),
                          (128, "auto", 0, True, "adam", 2e-3), (128, "auto", 1, False, "adam", 0.0),
                          (128, "two_pass", 0, False, "adam", 2e-3), (192, "auto", 1, False, "adam", 2e-3),
                          (64, "auto", 1, False, "sgd", 2e-3), (192, "auto", 0, False, "sgd", 0.0)])
def test_updates_follow_the_formulas(N, strategy, by, device_step, kind, lr_probe):
    c = _case(N)
    d = c.device()
    prob = c.problem()
    prob.set_strategy(strategy)
    opt = api.Optimizer(kind=kind, lr_object=1e-3, lr_probe=lr_probe, lr_pos=5e-2)
    st = _state(d, by, device_step, 3)
    before = _read(st)
    _, gO, gP, gX = prob.loss_and_grad(st.probe, st.object, st.positions, d["pats"], d["batch"], dense_pos=True)
    prob.reconstruct_step(st, d["pats"], d["batch"], opt)
    prob.check()
    assert st.steps_done() == (4 if kind == "adam" else 3)
    after = _read(st)
    for (var, lr_name), g in zip(VARS, (gO, gP, gX)):
        lr, g = getattr(opt, lr_name), _real(g)
        th = before[var][0]
        if lr == 0.0:
            want, tol = before[var], (0.0, 0.0, 0.0)
        elif kind == "sgd":
            want = (th - lr * g,) + before[var][1:]
            tol = (U * (np.abs(want[0]) + 2 * np.abs(lr * g)), 0.0, 0.0)
        else:
            want, tol = _adam(before[var], g, lr, 4, opt)
        for k in range(3):
            assert np.all(np.abs(after[var][k] - want[k]) <= tol[k]), (var, k)


@pytest.mark.parametrize("N", [64, 192])
def test_grouped_requests_that_share_a_state_update_it_in_turn(N):
    """Every gradient is taken before the first update; the updates of one state
    (and its count) then follow one another."""
    c = _case(N)
    d = c.device()
    probs = [c.problem(), c.problem()]
    batches = [d["batch"][:4].contiguous(), d["batch"][4:].contiguous()]
    opt = api.Optimizer(kind="adam", lr_object=1e-3, lr_probe=2e-3, lr_pos=5e-2)
    st = _state(d, 0, True, 0)
    x = _read(st)
    tol = {v: [0.0, 0.0, 0.0] for v, _ in VARS}
    losses = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in probs]
    grads = [p.loss_and_grad(st.probe, st.object, st.positions, d["pats"], b, dense_pos=True)[1:]
             for p, b in zip(probs, batches)]
    grp = api.Group(N, 9, 18, 36)
    grp.step([(p, st, d["pats"], b, opt, loss) for p, b, loss in zip(probs, batches, losses)])
    torch.cuda.synchronize()
    assert st.steps_done() == 2
    after = _read(st)
    for t, gs in enumerate(grads, 1):
        for (var, lr_name), g in zip(VARS, gs):
            x[var], e = _adam(x[var], _real(g), getattr(opt, lr_name), t, opt)
            # the errors of the first update pass on, by factors of at most one
            # (moments) and 4 (their share in the second step of the variable)
            tol[var] = [tol[var][0] + e[0], tol[var][1] + e[1], tol[var][2] + e[2]]
    for var, _ in VARS:
        assert np.all(np.abs(after[var][0] - x[var][0]) <= 4 * tol[var][0]), var
        for k in (1, 2):
            assert np.all(np.abs(after[var][k] - x[var][k]) <= 2 * tol[var][k]), (var, k)


@pytest.mark.parametrize("N,paths", [(64, ("auto", "two_pass")), (128, ("two_pass", "auto"))])
def test_grouped_requests_of_other_paths_that_share_a_state(N, paths):
    """The same when the requests of one state run on different kernels, in
    either order: losses and gradients are those of the state before the step."""
    c = _case(N)
    d = c.device()
    probs = [c.problem(), c.problem()]
    for p, path in zip(probs, paths):
        p.set_strategy(path)
    batches = [d["batch"][:4].contiguous(), d["batch"][4:].contiguous()]
    opt = api.Optimizer(kind="sgd", lr_object=1e-3, lr_probe=1e-3, lr_pos=1e-3)
    st = api.ReconState(d["probe"].clone(), d["obj"].clone(), d["pos"].clone(), adam=False)
    before = {v: _real(getattr(st, v)) for v, _ in VARS}
    losses = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in probs]
    grads = [p.loss_and_grad(st.probe, st.object, st.positions, d["pats"], b, dense_pos=True)
             for p, b in zip(probs, batches)]
    grp = api.Group(N, 9, 18, 36)
    grp.step([(p, st, d["pats"], b, opt, loss) for p, b, loss in zip(probs, batches, losses)])
    torch.cuda.synchronize()
    for loss, g in zip(losses, grads):
        assert loss.item() == g[0].item()
    for k, (var, lr_name) in enumerate(VARS, 1):
        lr, x, size = getattr(opt, lr_name), before[var], 0.0
        for g in (_real(g[k]) for g in grads):
            x, size = x - lr * g, size + np.abs(lr * g)
        # a product and a difference are rounded for each request
        tol = 2 * U * (np.abs(before[var]) + 2 * size)
        assert np.all(np.abs(_real(getattr(st, var)) - x) <= tol), var


@pytest.mark.parametrize("N,strategy,reduction", [(64, "auto", "atomic"), (64, "auto", "ordered"),
                                                  (128, "two_pass", "ordered"), (192, "auto", "atomic")])
def test_grouped_entries_of_one_context_add_their_gradients(N, strategy, reduction):
    """Two batches of one reconstruction through one context, beside another
    reconstruction: object and position gradients are the sum over both, and each
    entry's update takes it; the other one is not touched by it."""
    c, other = _case(N), _case(N, seed=9)
    d, e = c.device(), other.device()
    prob, prob2 = c.problem(), other.problem()
    for p in (prob, prob2):
        p.set_strategy(strategy)
        p.set_reduction(reduction)
    opt = api.Optimizer(kind="sgd", lr_object=1e-3, lr_probe=0.0, lr_pos=1e-3)
    make = lambda x: api.ReconState(x["probe"].clone(), x["obj"].clone(), x["pos"].clone(), adam=False)  # noqa: E731
    st, alone, beside = make(d), make(e), make(e)
    want = {v: _real(getattr(st, v)) for v in ("object", "positions")}
    _, gO, _, gX = prob.loss_and_grad(st.probe, st.object, st.positions, d["pats"], d["batch"], dense_pos=True)
    step = {"object": 2e-3 * _real(gO), "positions": 2e-3 * _real(gX)}
    loss = lambda: torch.zeros(1, dtype=torch.float64, device="cuda")  # noqa: E731
    prob2.reconstruct_step(alone, e["pats"], e["batch"], opt)
    grp = api.Group(N, 18, 36, 72)
    grp.step([(prob, st, d["pats"], d["batch"][:4].contiguous(), opt, loss()),
              (prob2, beside, e["pats"], e["batch"], opt, loss()),
              (prob, st, d["pats"], d["batch"][4:].contiguous(), opt, loss())])
    torch.cuda.synchronize()
    for v, delta in step.items():
        got = _real(getattr(st, v)) - want[v]
        # the parity bound of a gradient, and the rounding of the two updates
        assert np.linalg.norm(got + delta) <= 1e-3 * np.linalg.norm(delta) + 4 * U * np.linalg.norm(want[v]), v
    for v, _ in VARS:
        a, b = _real(getattr(alone, v)), _real(getattr(beside, v))
        assert np.array_equal(a, b), v
