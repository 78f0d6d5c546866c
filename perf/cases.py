"""The calls whose speed matters here, as a user's reconstruction program makes them.

One pass is one call of the package's public entry points on a group of probe
positions: simulated patterns (`Problem.forward`), loss and gradients
(`Problem.loss_and_grad`, or `autograd.multislice_loss` with its backward), or a
whole group step (`Problem.reconstruct_step` with Adam, SGD or ePIE,
`Problem.lsqml_step`, `Group.step` for several reconstructions in shared
launches). Sizes run from a handful of 64 x 64 windows of one mode and one slice
to the 256 x 256, 8-mode, 30-slice group of 512 positions that the repository's
benchmark times.

The data are those of a reconstruction in progress: patterns are Poisson counts
of the model's own intensities at a true probe and object, the state is an
estimate some way off the truth, Adam's moments are those of a run some tens of
steps old. The simulation and `exact` are the model written out in plain torch;
neither uses the package.
"""
from __future__ import annotations

import math

import torch

from paper_2505_14372_amd import api
from paper_2505_14372_amd.autograd import multislice_loss

DX, WAVELENGTH, BANDLIMIT = 0.2, 0.019688, 2.0 / 3.0   # Angstrom, 300 kV, of Nyquist
OBJ_MARGIN = 8          # object pixels around the scanned windows
NAMES = ("forward", "grad", "autograd", "adam", "sgd", "epie", "lsqml", "group")

# engine: the entry point; N, M, S: window side, modes, slices; B: positions of
# the group, taken as rows of `cols` positions at `step` pixels pitch; dz: gap in
# Angstrom; eps: the noise model's; reduction: how the object gradient is summed;
# every: every how many slices an entry wave is stored.
DEFAULT = dict(engine="adam", N=64, M=1, S=1, B=16, cols=16, step=4, dz=2.0, dose=1e5, phi=0.1, loss="poisson", eps=0.8,
               reduction="atomic", every=1)


def _case(name, **kw):
    return dict(DEFAULT, name=name, **kw)


def listed():
    return [
        # a few simulated patterns, for a look at a probe or an object: the smallest call
        _case("preview_64", engine="forward", N=64, M=1, S=1, B=16, cols=4),
        # the single-slice, single-mode step of conventional ptychography (the benchmark's spoa64)
        _case("step_64", engine="adam", N=64, M=1, S=1, B=256, step=4, dose=1e4, phi=0.3, loss="amplitude", eps=1e-3),
        # a small multislice reconstruction as it runs on its own on the server: bit-reproducible sum
        _case("step_64_m2_s8", engine="adam", N=64, M=2, S=8, B=225, cols=15, step=6, reduction="ordered"),
        # two modes at 128 through torch.autograd, an odd group left over at the end of an epoch
        _case("autograd_128_m2_s5", engine="autograd", N=128, M=2, S=5, B=77, cols=11, step=8, loss="anscombe", eps=1e-3),
        # four reconstructions of different depth sharing a launch on the server
        _case("group_128", engine="group", N=128, M=2, S=6, B=64, cols=8, step=8, reduction="ordered"),
        # loss and gradients of a whole 32 x 32 scan for an outside optimiser (the benchmark's ms128_m4_s8)
        _case("grad_128_m4_s8", engine="grad", N=128, M=4, S=8, B=1024, cols=32, step=8),
        # the same scan's Adam step as the benchmark takes it
        _case("step_128_m4_s8", engine="adam", N=128, M=4, S=8, B=1024, cols=32, step=8, reduction="ordered"),
        # conventional 3PIE on a modest group
        _case("epie_128_m3_s4", engine="epie", N=128, M=3, S=4, B=200, cols=20, step=8, loss="amplitude", eps=1e-3),
        # simulated patterns of a thick specimen at 192
        _case("forward_192_m3_s12", engine="forward", N=192, M=3, S=12, B=100, cols=10, step=11),
        # the benchmark's ms192_m6_s20 step
        _case("step_192_m6_s20", engine="adam", N=192, M=6, S=20, B=256, cols=64, step=11, reduction="ordered"),
        # a small group at the largest window: latency more than throughput
        _case("grad_256_m3_s10", engine="grad", N=256, M=3, S=10, B=24, cols=6, step=8, dz=1.0, dose=1e6),
        # the benchmark's headline step: 512 positions of a 128-wide scan
        _case("step_256_m8_s30", engine="adam", N=256, M=8, S=30, B=512, cols=128, step=8, dz=1.0, dose=1e6),
    ]


def _tiles(c):
    return c["B"] * c["M"] * c["S"] * c["N"] ** 2


def draw(rng):
    """One more case: any window size, modes, slices and group size of the range,
    no more work than the headline step."""
    most = 512 * 8 * 30 * 256 ** 2
    while True:
        c = dict(DEFAULT)
        c["N"] = rng.choice((64, 128, 192, 256))
        c["M"] = rng.randint(1, 8)
        c["S"] = int(round(math.exp(rng.uniform(0.0, math.log(30.0)))))
        c["B"] = int(round(math.exp(rng.uniform(math.log(4.0), math.log(1024.0)))))
        c["cols"] = max(1, int(round(math.sqrt(c["B"]) * rng.uniform(0.7, 2.0))))
        c["step"] = rng.randint(3, 12)
        c["engine"] = rng.choice(("forward", "grad", "grad", "autograd", "adam", "adam", "adam", "adam", "sgd", "epie", "lsqml",
                                  "group"))
        c["loss"], c["eps"] = rng.choice((("poisson", 0.8), ("poisson", 0.8), ("amplitude", 1e-3), ("anscombe", 1e-3),
                                          ("gaussian", 0.0)))
        c["reduction"] = "ordered" if c["engine"] == "group" else rng.choice(("atomic", "ordered"))
        c["dz"], c["phi"] = rng.choice((1.0, 2.0, 4.0)), rng.choice((0.05, 0.1, 0.3))
        c["dose"] = rng.choice((1e4, 1e5, 1e6))
        c["every"] = rng.choice((1, 1, 1, 1, 1, 1, 2, 3)) if c["engine"] != "group" else 1
        if c["engine"] == "group":
            c["B"] = min(c["B"], 256)
        if _tiles(c) * len(_parts(c)) <= most:
            return c


def _parts(c):
    """(modes, slices, positions) of each reconstruction of a case: one, but for
    a group, whose members differ in depth and size."""
    if c["engine"] != "group":
        return [(c["M"], c["S"], c["B"])]
    M, S, B = c["M"], c["S"], c["B"]
    return [(M, S, B), (max(1, M - 1), max(1, S // 2), B), (M, max(1, S - 1), max(1, B // 2)), (1, 1, max(1, B // 3))]


def _shape(c, B):
    rows = -(-B // c["cols"])
    return (c["N"] + 2 * OBJ_MARGIN + (rows - 1) * c["step"], c["N"] + 2 * OBJ_MARGIN + (c["cols"] - 1) * c["step"])


def work(c):
    """Each array a pass needs read once and each result written once, and the
    FFT arithmetic of the method: 2 S transforms of N x N per mode and position
    forward, as many again in the adjoint, 5 n log2 n flops each."""
    n2, total, flops = c["N"] ** 2, 0.0, 0.0
    for M, S, B in _parts(c):
        H, W = _shape(c, B)
        obj, probe, pats = 8.0 * S * H * W, 8.0 * M * n2, 4.0 * B * n2
        fft = 5.0 * n2 * math.log2(n2)
        if c["engine"] == "forward":
            total += obj + probe + pats + 8.0 * B
            flops += B * M * 2 * S * fft
            continue
        # state read, gradient or new state written
        total += 2 * (obj + probe) + pats + 16.0 * B
        if c["engine"] in ("adam", "group"):
            total += 4 * (obj + probe)      # two moments of the variable's size, read and written
        if c["engine"] == "lsqml":
            total += 2 * obj
        flops += B * M * 4 * S * fft
    return {"bytes": total, "flops": flops}


# ---------------------------------------------------------------- inputs

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _freq(n, dtype=torch.float64):
    return torch.fft.fftfreq(n, d=1.0 / n, device="cuda", dtype=dtype)


def _probe(c, M, defocus):
    """M mutually orthogonal modes from a round aperture with a defocus phase."""
    N = c["N"]
    k = _freq(N)
    ky, kx = k[:, None], k[None, :]
    r2 = ky * ky + kx * kx
    R = N / 4.0
    spec = (r2 <= R * R) * torch.exp(-1j * defocus * r2 / (R * R))
    w = torch.tensor([1.0] if M == 1 else [0.6] + [0.4 * 0.6 ** m for m in range(1, M)], dtype=torch.float64)
    w = w / w.sum()
    modes = []
    for m in range(M):
        th = 2 * math.pi * m / M
        s = spec * torch.exp(-2j * math.pi * (ky * 0.5 * math.sin(th) + kx * 0.5 * math.cos(th) * (1 + m)) / N) if m else spec
        p = torch.fft.ifft2(s)
        for _ in range(2):
            for q in modes:
                p = p - (q.conj() * p).sum() / (q.conj() * q).sum() * q
        modes.append(p)
    return torch.stack([p / p.abs().square().sum().sqrt() * (w[m].item() * c["dose"]) ** 0.5 for m, p in enumerate(modes)])


def _object(S, H, W, phi, g):
    """Phase slices: smoothed noise between 0 and phi."""
    ky, kx = torch.fft.fftfreq(H, device="cuda")[:, None], torch.fft.fftfreq(W, device="cuda")[None, :]
    low = torch.exp(-2 * (math.pi * 2.0) ** 2 * (ky * ky + kx * kx))
    out = torch.empty((S, H, W), dtype=torch.float32, device="cuda")
    for i in range(S):
        f = torch.fft.ifft2(torch.fft.fft2(torch.rand((H, W), generator=g, device="cuda")) * low).real
        out[i] = (f - f.min()) / (f.max() - f.min()) * phi
    return out


def _inputs(c, part, seed):
    """Arrays of one reconstruction, from the seed alone (on the GPU)."""
    M, S, B = part
    g = _gen(seed)
    H, W = _shape(c, B)
    j = torch.arange(B, device="cuda")
    pos = torch.stack([j // c["cols"], j % c["cols"]], 1).double() * c["step"] + OBJ_MARGIN
    pos = pos + (torch.rand((B, 2), generator=g, device="cuda", dtype=torch.float64) - 0.5)
    phase = _object(S, H, W, c["phi"], g)
    probe_true = _probe(c, M, 0.5).to(torch.complex64)
    truth = torch.polar(torch.ones_like(phase), phase)
    pats = torch.empty((B, c["N"], c["N"]), dtype=torch.float32, device="cuda")
    m = _Model(c, part, probe_true, truth, pos.float(), torch.float32)
    for b in m.blocks():
        pats[b] = torch.poisson(m.intensities(b), generator=g)
    est = torch.polar(1.0 - 0.05 * torch.rand((S, H, W), generator=g, device="cuda"), 0.6 * phase)
    return dict(probe=_probe(c, M, 0.3).to(torch.complex64), obj=est, pats=pats,
                pos=(pos + 1.0 * (torch.rand((B, 2), generator=g, device="cuda", dtype=torch.float64) - 0.5)).float(),
                batch=torch.arange(B, dtype=torch.int32, device="cuda"), seed=seed)


def _moments(a, g):
    """Adam moments of a run some steps old: gradients of the size these inputs have."""
    def pair(t, scale):
        s = torch.view_as_real(t).shape if t.is_complex() else t.shape
        r = lambda: torch.rand(s, generator=g, device="cuda")  # noqa: E731
        return scale * 0.3 * (r() - 0.5), (scale * (0.3 + r())) ** 2
    size = a["probe"].abs().square().mean().sqrt().item()
    return dict(object=pair(a["obj"], 0.5 * size * size), probe=pair(a["probe"], 0.5 * size * len(a["pos"]) ** 0.5),
                pos=pair(a["pos"], 0.05 * size * size * a["probe"].shape[-1]))


RATE = dict(adam=dict(lr_object=1e-4, lr_probe=1e-4, lr_pos=1e-5), sgd=dict(lr_object=1e-7, lr_probe=1e-7, lr_pos=0.0),
            epie=dict(lr_object=0.05, lr_probe=0.05, lr_pos=0.0))
STEPS_DONE = 25


def _problem(c, part, lsqml=False):
    M, S, B = part
    H, W = _shape(c, B)
    p = api.Problem(c["N"], M, S, H, W, B, dz=[c["dz"]] * (S - 1), dx=DX, wavelength=WAVELENGTH, bandlimit=BANDLIMIT,
                    loss=c["loss"], eps=c["eps"], sigma=_sigma(c), max_batch=0 if c["engine"] == "group" else B,
                    checkpoint_every=c["every"], lsqml=lsqml)
    p.set_reduction(c["reduction"])
    return p


def _sigma(c):
    return max(1.0, math.sqrt(c["dose"]) / c["N"])


def _state(c, a):
    st = api.ReconState(a["probe"].clone(), a["obj"].clone(), a["pos"].clone(), adam=c["engine"] in ("adam", "group"))
    if c["engine"] in ("adam", "group"):
        m = _moments(a, _gen(a["seed"] + 991))
        (st.m_object, st.v_object), (st.m_probe, st.v_probe), (st.m_pos, st.v_pos) = m["object"], m["probe"], m["pos"]
        st.step = STEPS_DONE
    return st


def prepare(c, seed):
    e = c["engine"]
    parts = _parts(c)
    many = [_inputs(c, p, seed * 16 + q) for q, p in enumerate(parts)]
    s = dict(engine=e, case=c, a=many[0])
    loss = lambda: torch.zeros(1, dtype=torch.float64, device="cuda")  # noqa: E731
    if e == "group":
        probs = [_problem(c, p) for p in parts]
        s["states"] = [_state(c, a) for a in many]
        s["entries"] = [(p, st, a["pats"], a["batch"], api.Optimizer(kind="adam", **RATE["adam"]), loss())
                        for p, st, a in zip(probs, s["states"], many)]
        s["group"] = api.Group(c["N"], sum(B for _, _, B in parts), sum(M * B for M, _, B in parts),
                               sum(M * S * B for M, S, B in parts))
        return s
    s["prob"] = _problem(c, parts[0], lsqml=e == "lsqml")
    s["loss"] = loss()
    if e == "autograd":
        s["leaves"] = [many[0][k].clone().requires_grad_(True) for k in ("obj", "probe", "pos")]
    elif e in RATE:
        s["state"], s["opt"] = _state(c, many[0]), api.Optimizer(kind=e, **RATE[e])
    elif e == "lsqml":
        s["state"] = _state(c, many[0])
        M, S, B = parts[0]
        H, W = _shape(c, B)
        s["illum"] = api.IllumSums(S, H, W, c["N"])
        # the sums of an earlier iteration: the probe's flux over the scanned area
        size = many[0]["probe"].abs().square().mean().item() * c["M"] * (c["N"] / c["step"]) ** 2
        g = _gen(seed + 77)
        s["illum"].obj_cur += size * (0.5 + torch.rand((S, H, W), generator=g, device="cuda"))
        s["illum"].probe_cur += B * (0.5 + torch.rand((c["N"], c["N"]), generator=g, device="cuda"))
        s["illum"].end_iteration()
    return s


def _state_out(st, loss):
    # the loss is a float64 total of float32 partial sums: it comes back at the accuracy it has
    out = dict(loss=loss.float(), object=st.object, probe=st.probe, pos=st.positions)
    if st.m_object is not None:
        out.update(m_object=st.m_object, m_probe=st.m_probe, m_pos=st.m_pos, v_object=st.v_object, v_probe=st.v_probe,
                   v_pos=st.v_pos)
    return out


def run(s):
    e, a = s["engine"], s["a"]
    if e == "forward":
        return s["prob"].forward(a["probe"], a["obj"], a["pos"], a["batch"])[0]
    if e == "grad":
        loss, g_o, g_p, g_x = s["prob"].loss_and_grad(a["probe"], a["obj"], a["pos"], a["pats"], a["batch"], loss=s["loss"])
        return dict(loss=loss.float(), object=g_o, probe=g_p, pos=g_x)
    if e == "autograd":
        for t in s["leaves"]:
            t.grad = None
        loss = multislice_loss(*s["leaves"], s["prob"], a["pats"], a["batch"])
        loss.backward()
        o, p, x = s["leaves"]
        return dict(loss=loss.detach().float(), object=o.grad, probe=p.grad, pos=x.grad)
    if e in RATE:
        s["prob"].reconstruct_step(s["state"], a["pats"], a["batch"], s["opt"], loss=s["loss"])
        return _state_out(s["state"], s["loss"])
    if e == "lsqml":
        s["prob"].lsqml_step(s["state"], s["illum"], a["pats"], a["batch"], loss=s["loss"])
        return dict(_state_out(s["state"], s["loss"]), illum_obj=s["illum"].obj_cur, illum_probe=s["illum"].probe_cur)
    s["group"].step(s["entries"])
    return [_state_out(st, entry[5]) for st, entry in zip(s["states"], s["entries"])]


# ---------------------------------------------------------------- the model in plain torch

class _Model:
    """Forward model, loss and adjoint of one group, over blocks of positions."""

    def __init__(self, c, part, probe, obj, pos, real):
        self.c, (self.M, self.S, self.B) = c, part
        self.N, self.real = c["N"], real
        self.cplx = torch.complex64 if real == torch.float32 else torch.complex128
        self.probe, self.obj = probe.to(self.cplx), obj.to(self.cplx)
        x = pos.double()
        n = torch.floor(x + 0.5)
        self.n, d = n.long(), x - n
        N = self.N
        self.f = _freq(N) / N
        ramp = lambda t: torch.polar(torch.ones_like(t), t).to(self.cplx)  # noqa: E731
        self.ry = ramp(-2 * math.pi * self.f[None, :] * d[:, :1])
        self.rx = ramp(-2 * math.pi * self.f[None, :] * d[:, 1:])
        k = _freq(N)
        q2 = (k[:, None] / (N * DX)) ** 2 + (k[None, :] / (N * DX)) ** 2
        keep = k[:, None] ** 2 + k[None, :] ** 2 <= (BANDLIMIT * N / 2) ** 2 * (1 + 1e-9)
        self.H = (keep * ramp(-math.pi * WAVELENGTH * c["dz"] * q2)).to(self.cplx)
        self.phat = torch.fft.fft2(self.probe, norm="ortho")

    def blocks(self):
        most = max(1, int(2 ** 33 / (8 if self.real == torch.float32 else 16) / (self.M * (self.S + 4) * self.N ** 2)))
        for b in range(0, self.B, most):
            yield torch.arange(b, min(b + most, self.B), device="cuda")

    def patch(self, i, b):
        r = torch.arange(self.N, device="cuda")
        return self.obj[i][(self.n[b, :1] + r)[:, :, None], (self.n[b, 1:] + r)[:, None, :]]

    def ramps(self, b):
        return (self.ry[b][:, :, None] * self.rx[b][:, None, :])[:, None]

    def waves(self, b, keep):
        psi = torch.fft.ifft2(self.phat[None] * self.ramps(b), norm="ortho")
        entry = []
        for i in range(self.S):
            if keep:
                entry.append(psi)
            phi = psi * self.patch(i, b)[:, None]
            if i < self.S - 1:
                psi = torch.fft.ifft2(torch.fft.fft2(phi) * self.H)
        return entry, torch.fft.fft2(phi, norm="ortho")

    def intensities(self, b):
        return self.waves(b, False)[1].abs().square().sum(1)

    def gradients(self, pats):
        """loss, object, probe and position gradients (dL/dRe + i dL/dIm)."""
        c, N = self.c, self.N
        total = torch.zeros((), dtype=torch.float64, device="cuda")
        g_o, g_ph = torch.zeros_like(self.obj), torch.zeros_like(self.phat)
        g_x = torch.zeros((self.B, 2), dtype=self.real, device="cuda")
        r = torch.arange(N, device="cuda")
        for b in self.blocks():
            entry, far = self.waves(b, True)
            intensity, count = far.abs().square().sum(1), pats[b].to(self.real)
            eps = c["eps"]
            if c["loss"] == "poisson":
                some = count > 0
                ell = torch.where(some, intensity - count - count * (torch.log(intensity + eps) - torch.log(count + eps)), intensity)
                w = 2 * (1 - count / (intensity + eps))
            elif c["loss"] == "gaussian":
                ell = (intensity - count) ** 2 / (2 * _sigma(c) ** 2)
                w = 2 * (intensity - count) / _sigma(c) ** 2
            else:
                off = 0.375 if c["loss"] == "anscombe" else 0.0
                root, want = torch.sqrt(intensity + off), torch.sqrt(count + off)
                ell, w = (root - want) ** 2 / 2, 1 - want / (eps + root)
            total += ell.sum(dtype=torch.float64)
            g = torch.fft.ifft2(w[:, None] * far, norm="ortho")
            for i in range(self.S - 1, -1, -1):
                o = self.patch(i, b)
                part = (entry[i].conj() * g).sum(1)
                flat = ((self.n[b, :1] + r)[:, :, None] * self.obj.shape[2] + (self.n[b, 1:] + r)[:, None, :]).reshape(-1)
                view = torch.view_as_real(g_o[i]).view(-1, 2)
                view.index_add_(0, flat, torch.view_as_real(part).reshape(-1, 2))
                g = o.conj()[:, None] * g
                if i > 0:
                    g = torch.fft.ifft2(torch.fft.fft2(g) * self.H.conj())
            ghat, R = torch.fft.fft2(g, norm="ortho"), self.ramps(b)
            z = (ghat.conj() * (self.phat[None] * R)).imag.sum(1)
            g_x[b, 0] = 2 * math.pi * (z.sum(2) * self.f.to(self.real)).sum(1)
            g_x[b, 1] = 2 * math.pi * (z.sum(1) * self.f.to(self.real)).sum(1)
            g_ph += (ghat * R.conj()).sum(0)
        return total, g_o, torch.fft.ifft2(g_ph, norm="ortho"), g_x


def _exact_step(c, part, a, model):
    loss, g_o, g_p, g_x = model.gradients(a["pats"])
    out = dict(loss=loss.reshape(1))
    rate = RATE["sgd" if c["engine"] == "sgd" else "adam"]
    mom = _moments(a, _gen(a["seed"] + 991)) if c["engine"] != "sgd" else None
    for key, t, g, lr in (("object", a["obj"], g_o, rate["lr_object"]), ("probe", a["probe"], g_p, rate["lr_probe"]),
                          ("pos", a["pos"], g_x, rate["lr_pos"])):
        cplx = t.is_complex()
        g = torch.view_as_real(g).contiguous() if cplx else g
        th = torch.view_as_real(t).double() if cplx else t.double()
        if mom is None:
            new = th - lr * g
        else:
            m, v = (x.double() for x in mom[key])
            m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
            step = STEPS_DONE + 1
            new = th - lr / (1 - 0.9 ** step) * m / (v.sqrt() / math.sqrt(1 - 0.999 ** step) + 1e-8)
            out["m_" + key], out["v_" + key] = m, v
        out[key] = torch.view_as_complex(new.contiguous()) if cplx else new
    return out


def exact(c, seed):
    """What `run` returns on a new state, in 64 bits. The ePIE and LSQML updates
    (engines with normalisers of their own) are left to the comparison with the
    start."""
    e = c["engine"]
    if e in ("epie", "lsqml"):
        return None
    out = []
    for q, part in enumerate(_parts(c)):
        a = _inputs(c, part, seed * 16 + q)
        m = _Model(c, part, a["probe"], a["obj"], a["pos"], torch.float64)
        if e == "forward":
            return torch.cat([m.intensities(b) for b in m.blocks()])
        if e in ("grad", "autograd"):
            loss, g_o, g_p, g_x = m.gradients(a["pats"])
            return dict(loss=loss.reshape(1) if e == "grad" else loss, object=g_o, probe=g_p, pos=g_x)
        out.append(_exact_step(c, part, a, m))
    return out if e == "group" else out[0]
