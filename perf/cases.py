"""The work whose speed is measured: calls of the library's public entry points
over the range of sizes that its configurations, tests and benchmark use.

  listed()             the named cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  plan and inputs on the GPU
  run(state)           one call, its outputs
  work(case)           bytes and floating-point operations of one call
  exact(case, seed)    the outputs in 64 bits, by plain torch

A case's "call" is one of
  grad     Plan.holo_grad: objective and both gradients
  loss     holo_loss, forward and backward through autograd
  fwd      Plan.holo_fwd over the angles k0 .. k1 of the plan
  adj      Plan.holo_adj over the angles k0 .. k1 of the plan
  cg       Plan.holo_cg: `iters` conjugate-gradient iterations
  batch2d  Plan2D.holo2d_grad over a batch of single-angle problems

Objectives are double-precision sums over single-precision fields; run() hands
them on in the fields' precision, which is how accurate they are.
"""

import math

import numpy as np
import torch

from paper_2407_20304_amd import holo, synth

DEV = "cuda"
LERP_FLOP = 8.0          # one complex linear interpolation added to a sum


def _tomo(name, call, H, W, angles, nd=4, **more):
    c = {"name": name, "call": call, "H": H, "W": W, "angles": angles, "nd": nd, "chunk": 64,
         "shift": False, "pshift": False, "functional": "amplitude", "projector": "joseph",
         "pad": 1, "k0": 0, "k1": angles, "iters": 0}
    c.update(more)
    return c


def listed():
    return [
        # The smallest workload (64^3, 90 angles in one chunk): a first binning
        # level or a quick look, where launches and idle CUs count.
        _tomo("grad_64_a90", "grad", 64, 64, 90, chunk=90),
        # The small reconstruction (256^3, 360 angles) as a training loop calls
        # it: the differentiable loss and its backward.
        _tomo("loss_256_a360", "loss", 256, 256, 360),
        # The headline workload: 1024^3 volume, 1800 angles in chunks of 64.
        _tomo("grad_1024_a1800", "grad", 1024, 1024, 1800),
        # A wide, thin slab: the 2048-wide detector of 900 angles (chunks of
        # 32), 128 of its slices.
        _tomo("grad_slab128x2048_a900", "grad", 128, 2048, 900, chunk=32),
        # Predicted frames of part of a scan on a 3 * 2^a detector with jitter
        # shifts, three planes: checking a model against data.
        _tomo("fwd_192x384_k64", "fwd", 192, 384, 360, nd=3, shift=True, k0=101, k1=165),
        # Vector-Jacobian product of one 150-angle chunk of a 900-angle scan:
        # the object and probe update of an own solver.
        _tomo("adj_512_k150", "adj", 512, 512, 900, k0=150, k1=300),
        # The Fourier-slice projector in place of the ray sums.
        _tomo("grad_fourier_512_a450", "grad", 512, 512, 450, projector="fourier"),
        # Padded propagation (fields of view that the probe overfills), with
        # object shifts.
        _tomo("grad_padded_256_a180", "grad", 256, 256, 180, pad=2, shift=True),
        # Scans with a moving probe, intensity data, an odd number of angles
        # and a rectangular detector.
        _tomo("grad_pshift_512x384_a121", "grad", 512, 384, 121, nd=2, shift=True, pshift=True,
              functional="intensity"),
        # Two solver iterations on a binned problem: objectives, gradients and
        # vector updates with the line search's host decisions between them.
        _tomo("cg_128_a180", "cg", 128, 128, 180, iters=2),
        # The batched single-angle workload: 96 problems of 128 to 512 px.
        {"name": "batch96_mixed", "call": "batch2d", "n": 96, "sizes": "mixed", "nd": 4,
         "functional": "amplitude"},
        # One small single-angle problem: the latency of a serving loop.
        {"name": "batch1_128", "call": "batch2d", "n": 1, "sizes": "128", "nd": 4,
         "functional": "amplitude"},
    ]


SIZES = (64, 128, 192, 256, 384, 512)


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Calls and options in about the proportions of their use; edges from the
    supported ones, angles log-uniform, the whole bounded by a fraction of the
    headline workload."""
    call = rng.choice(["grad", "grad", "grad", "loss", "fwd", "adj", "cg", "batch2d", "batch2d"])
    nd = rng.choice([1, 2, 3, 4, 4, 4, 5])
    functional = rng.choice(["amplitude", "amplitude", "intensity", "conventional"])
    if call == "batch2d":
        size = rng.choice(["mixed", "mixed", "64", "192", "256", "512", "1024"])
        most = {"64": 512, "192": 128, "256": 96, "512": 32, "1024": 8}.get(size, 96)
        return {"call": call, "n": _log_uniform(rng, 1, most), "sizes": size, "nd": nd,
                "functional": functional}
    while True:
        H, W = rng.choice(SIZES), rng.choice(SIZES + (1024, 2048))
        angles = _log_uniform(rng, 8, 720)
        if angles * W * W * H <= 1.5e11 and angles * nd * H * W <= 6e8:
            break
    if call == "cg" and angles * W * W * H > 2e10:
        H = W = 128
    c = _tomo("", call, H, W, angles, nd=nd, shift=rng.random() < 0.4)
    del c["name"]
    if call in ("fwd", "adj"):
        c["k0"] = rng.randrange(0, angles - 3)
        c["k1"] = rng.randrange(c["k0"] + 1, min(angles, c["k0"] + 150) + 1)
        return c
    if call == "cg":
        c["iters"] = rng.choice([1, 2])
        return c
    c["functional"] = functional
    option = rng.choice(["", "", "", "pshift", "pad", "fourier"])
    if option == "pshift":
        c["pshift"] = True
    elif option == "pad" and W <= 1024:
        c["pad"] = 2
    elif option == "fourier" and W <= 512:
        c["projector"] = "fourier"
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _mags(nd):
    if nd <= len(synth.MAG_REL):
        return tuple(synth.MAG_REL[:nd])
    return tuple(float(m) for m in np.linspace(1.0, 1.5, nd))


def _theta(n):
    return np.arange(n, dtype=np.float64) * (np.pi / n)


def _shifts(case, seed, which):
    if not case[which]:
        return None
    return synth.random_shifts(case["angles"], case["nd"], 8 * seed + (3 if which == "pshift" else 2))


def _waves(gen, n, count=8):
    """A sum of `count` sinusoids along n pixels, at most 1 in size."""
    r = torch.rand((3, count, 1), generator=gen, device=DEV)
    x = torch.arange(n, device=DEV, dtype=torch.float32)[None, :]
    s = (r[0] * torch.sin(2 * math.pi * (x / (2.0 + 30.0 * r[1]) + r[2]))).sum(0)
    return s / s.abs().max()


def _probe(gen, H, W):
    """Gaussian beam with line structure across and down and a smooth phase."""
    x = (torch.arange(W, device=DEV, dtype=torch.float32) - W / 2) / (0.375 * W)
    y = (torch.arange(H, device=DEV, dtype=torch.float32) - H / 2) / (0.375 * H)
    sx, sy, tx, ty = _waves(gen, W), _waves(gen, H), _waves(gen, W), _waves(gen, H)
    c = torch.rand(4, generator=gen, device=DEV)
    amp = torch.exp(-0.5 * (x[None, :] ** 2 + y[:, None] ** 2)) * (1 + 0.05 * sx[None, :] + 0.05 * sy[:, None])
    phase = (torch.sin(2 * x[None, :] * c[0] + 6 * c[1]) * torch.cos(2 * y[:, None] * c[2] + 6 * c[3])
             + 0.15 * tx[None, :] + 0.15 * ty[:, None])
    return torch.polar(amp, phase)


def _phase_object(gen, n, count=10):
    """psi = exp((i - 0.01) phi), phi of `count` ellipses drawn over each other."""
    r = torch.rand((6, count), generator=gen, device=DEV).tolist()
    y = (torch.arange(n, device=DEV, dtype=torch.float32) - n / 2)[:, None]
    x = (torch.arange(n, device=DEV, dtype=torch.float32) - n / 2)[None, :]
    phi = torch.zeros((n, n), device=DEV)
    for i in range(count):
        cx, cy = (0.6 * r[0][i] - 0.3) * n, (0.6 * r[1][i] - 0.3) * n
        ax, ay = (0.05 + 0.2 * r[2][i]) * n, (0.05 + 0.2 * r[3][i]) * n
        c, s = math.cos(math.pi * r[4][i]), math.sin(math.pi * r[4][i])
        xr, yr = (x - cx) * c + (y - cy) * s, -(x - cx) * s + (y - cy) * c
        phi = torch.where((xr / ax) ** 2 + (yr / ay) ** 2 <= 1.0, torch.full_like(phi, r[5][i]), phi)
    return torch.polar(torch.exp(-0.01 * phi), phi)


def _data(case, n_frames, H, W, seed):
    """Hologram-like data: amplitudes, or intensities for that functional."""
    a = synth.synthetic_amplitudes(n_frames, 1, H, W, seed, device=DEV)[:, 0]
    return a.square_() if case["functional"] == "intensity" else a


def _tomo_inputs(case, seed):
    H, W, n, nd = case["H"], case["W"], case["angles"], case["nd"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    s = {"u": synth.ellipsoid_volume(W, H, seed, device=DEV), "q": _probe(gen, H, W)}
    if case["call"] in ("grad", "loss", "cg"):
        s["amp"] = _data(case, n * nd, H, W, 4 * seed + 1).reshape(n, nd, H, W)
        s["amp_ref"] = _data(case, 1, H, W, 4 * seed + 2)[0]
    if case["call"] == "adj":
        k = case["k1"] - case["k0"]
        s["w"] = torch.randn((k, nd, H, W), generator=gen, device=DEV, dtype=torch.complex64)
    return s


def _batch_sizes(case):
    if case["sizes"] == "mixed":
        return synth.batch_sizes(case["n"])
    return [int(case["sizes"])] * case["n"]


def _batch_inputs(case, seed):
    sizes, nd = _batch_sizes(case), case["nd"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    # fringes differ per frame, the probe and object per instance
    amp = {n: _data(case, nd * sizes.count(n), n, n, 4 * seed + n).reshape(-1, nd, n, n)
           for n in sorted(set(sizes))}
    ref = {n: _data(case, sizes.count(n), n, n, 4 * seed + n + 1) for n in sorted(set(sizes))}
    seen = {n: 0 for n in amp}
    parts = {"psi": [], "q": [], "amp": [], "amp_ref": []}
    for n in sizes:
        parts["psi"].append(_phase_object(gen, n).reshape(-1))
        parts["q"].append(_probe(gen, n, n).reshape(-1))
        parts["amp"].append(amp[n][seen[n]].reshape(-1))
        parts["amp_ref"].append(ref[n][seen[n]].reshape(-1))
        seen[n] += 1
    return {k: torch.cat(v) for k, v in parts.items()}


def _plan(case, seed):
    p = holo.Plan(case["H"], case["W"], _theta(case["angles"]), _mags(case["nd"]), synth.M0,
                  synth.FRESNEL0, synth.KAPPA, shift=_shifts(case, seed, "shift"),
                  chunk=case["chunk"])
    if case["functional"] != "amplitude":
        p.set_functional(case["functional"])
    if case["projector"] != "joseph":
        p.set_projector(case["projector"])
    if case["pad"] != 1:
        p.set_padding(case["pad"])
    if case["pshift"]:
        p.set_probe_shifts(_shifts(case, seed, "pshift"))
    return p


def _step0(F, gu, gq):
    """First trial step of the solver: the power of two next to F / ||g||^2."""
    gg = sum(float(torch.linalg.vector_norm(g)) ** 2 for g in (gu, gq))
    return 2.0 ** round(math.log2(F / gg))


def prepare(case, seed):
    seed = int(seed) % (1 << 27)
    s = {"case": case}
    if case["call"] == "batch2d":
        s.update(_batch_inputs(case, seed))
        s["plan"] = holo.Plan2D(_batch_sizes(case), _mags(case["nd"]), synth.M0, synth.FRESNEL0)
        if case["functional"] != "amplitude":
            s["plan"].set_functional(case["functional"])
        s["plan"].workspace(s["psi"].device)
        return s
    s.update(_tomo_inputs(case, seed))
    s["plan"] = _plan(case, seed)
    s["plan"].workspace(s["u"].device)
    if case["call"] == "cg":
        F, gu, gq = s["plan"].holo_grad(s["u"], s["q"], s["amp"], s["amp_ref"])
        s["step0"] = _step0(F.item(), gu, gq)
    if case["call"] == "loss":
        s["u"].requires_grad_(True)
        s["q"].requires_grad_(True)
    return s


def run(s):
    case, p = s["case"], s["plan"]
    call = case["call"]
    if call == "batch2d":
        F, g_psi, g_q = p.holo2d_grad(s["psi"], s["q"], s["amp"], s["amp_ref"])
        return {"F": F.float(), "g_psi": g_psi, "g_q": g_q}
    u, q = s["u"], s["q"]
    if call == "grad":
        F, g_u, g_q = p.holo_grad(u, q, s["amp"], s["amp_ref"])
        return {"F": F.float(), "g_u": g_u, "g_q": g_q}
    if call == "loss":
        u.grad = q.grad = None
        F = holo.holo_loss(u, q, s["amp"], s["amp_ref"], p)
        F.backward()
        return {"F": F.detach().float(), "g_u": u.grad, "g_q": q.grad}
    if call == "fwd":
        return {"v": p.holo_fwd(u, q, case["k0"], case["k1"])}
    if call == "adj":
        g_u, g_q = p.holo_adj(u, q, s["w"], case["k0"], case["k1"])
        return {"g_u": g_u, "g_q": g_q}
    u, q, F_hist, steps, halvings = p.holo_cg(u, q, s["amp"], s["amp_ref"], case["iters"], s["step0"])
    return {"u": u, "q": q, "F": F_hist.astype(np.float32), "halvings": halvings}


# ---------------------------------------------------------------------------
# What a call cannot do without
# ---------------------------------------------------------------------------

def _fft_flop(H, W):
    """One propagation of a frame: a 2-D transform, the transfer, its inverse."""
    return 10.0 * H * W * math.log2(H * W) + 6.0 * H * W


def work(case):
    nd = case["nd"]
    if case["call"] == "batch2d":
        px = [n * n for n in _batch_sizes(case)]
        flops = sum((4 * nd + 2) * _fft_flop(math.isqrt(p), math.isqrt(p)) for p in px)
        return {"bytes": sum(px) * (8 + 8 + 4 * nd + 4 + 8 + 8), "flops": flops}
    H, W = case["H"], case["W"]
    k = case["k1"] - case["k0"]
    vol, frame = 8.0 * H * W * W, 8.0 * H * W
    if case["projector"] == "fourier":     # slice transforms, 8 x 8 taps per polar sample
        ray = H * (10.0 * 4 * W * W * math.log2(2 * W) + k * W * (64 * 4 + 5 * math.log2(W)))
    else:
        ray = LERP_FLOP * k * W * W * H
    prop = _fft_flop(H * case["pad"], W * case["pad"])
    grad_bytes = 2 * vol + 2 * frame + 4.0 * H * W * (k * nd + 1)
    grad_flops = 2 * ray + (2 * k * nd + 2 * nd + 2) * prop
    obj_flops = ray + (k * nd + nd + 1) * prop
    if case["call"] == "fwd":
        return {"bytes": vol + frame * (1 + k * nd), "flops": ray + (k * nd + nd) * prop}
    if case["call"] == "adj":
        return {"bytes": 2 * vol + frame * (2 + k * nd), "flops": 2 * ray + (k * nd + 2 * nd) * prop}
    if case["call"] == "cg":
        it = case["iters"]
        return {"bytes": 2 * vol + 2 * frame + 4.0 * H * W * (k * nd + 1),
                "flops": (it + 1) * grad_flops + it * obj_flops}
    return {"bytes": grad_bytes, "flops": grad_flops}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, from the definitions of include/holo.h
# ---------------------------------------------------------------------------

C128, F64 = torch.complex128, torch.float64


def _transfer(n, rho):
    k = torch.fft.fftfreq(n, device=DEV, dtype=F64) * n
    ph = -math.pi * rho / (synth.FRESNEL0 * n * n) * k * k
    return torch.polar(torch.ones_like(ph), ph)


def _propagate(f, rho, pad=1):
    H, W = f.shape[-2:]
    y0, x0 = (pad - 1) * H // 2, (pad - 1) * W // 2
    g = torch.fft.fft2(torch.nn.functional.pad(f, (x0, x0, y0, y0)) if pad > 1 else f)
    g = torch.fft.ifft2(g * (_transfer(pad * H, rho)[:, None] * _transfer(pad * W, rho)[None, :]))
    return g[..., y0:y0 + H, x0:x0 + W]


def _axis(f, dim, pos, periodic):
    """Linear interpolation of f (K, H, W) along dim at pos (K, n); zero
    outside the grid unless it is periodic."""
    n = f.shape[dim]
    i = torch.floor(pos)
    w = pos - i
    out = 0
    for e in (0, 1):
        d = i.long() + e
        wt = w if e else 1 - w
        if periodic:
            d = d % n
        else:
            wt = torch.where((d >= 0) & (d < n), wt, torch.zeros_like(wt))
            d = d.clamp(0, n - 1)
        shape = list(f.shape)
        idx = (d[:, :, None] if dim == 1 else d[:, None, :]).expand(shape)
        out = out + f.gather(dim, idx) * (wt[:, :, None] if dim == 1 else wt[:, None, :])
    return out


def _fields(psi, q, mags, pad, shift, pshift):
    """v (K, nd, H, W) of the transmissions psi (K, H, W) and the probe (None: 1)."""
    K, H, W = psi.shape
    y, x = (torch.arange(n, device=DEV, dtype=F64) for n in (H, W))
    out = []
    for j, m in enumerate(mags):
        t = shift[:, j] if shift is not None else torch.zeros((K, 2), device=DEV, dtype=F64)
        phi = 1 + _axis(_axis(psi - 1, 1, H / 2 + m * (y - H / 2) - t[:, :1], False), 2,
                        W / 2 + m * (x - W / 2) - t[:, 1:], False)
        if q is not None:
            Q = _propagate(q, synth.M0 * (m - 1) / (m * (synth.M0 - 1)), pad)
            if pshift is not None:
                sj = pshift[:, j]
                Q = _axis(_axis(Q[None].expand(K, H, W), 1, y - sj[:, :1], True), 2, x - sj[:, 1:], True)
            phi = Q * phi
        out.append(_propagate(phi, (synth.M0 - m) / (m * (synth.M0 - 1)), pad))
    return torch.stack(out, 1)


def _cost(v, a, functional):
    return ((v.abs().square() if functional == "intensity" else v.abs()) - a).square().sum()


def _ray_taps(theta, W):
    """Voxel indices y * W + x and weights (W steps, W bins) of Joseph's sums."""
    c, C, S = W / 2.0, math.cos(theta), math.sin(theta)
    step = torch.arange(W, device=DEV, dtype=F64)[:, None]
    s = torch.arange(W, device=DEV, dtype=F64)[None, :] - c
    ywalk = abs(C) >= abs(S)
    f = c + (s - (step - c) * (S if ywalk else C)) / (C if ywalk else S)
    i = torch.floor(f)
    scale = 1.0 / max(abs(C), abs(S))
    for e in (0, 1):
        d = i.long() + e
        w = ((f - i) if e else 1 - (f - i)) * scale
        ok = (d >= 0) & (d < W)
        w = torch.where(ok, w, torch.zeros_like(w))
        d = d.clamp(0, W - 1)
        yield (step.long() * W + d if ywalk else d * W + step.long()), w


def _slice_matrix(theta, W):
    """Fourier-slice projection of one slice as a (W, W * W) matrix."""
    x = torch.arange(W, device=DEV, dtype=F64) - W // 2
    d = x[:, None] - (x[None, :] * math.cos(theta) + x[:, None] * math.sin(theta)).reshape(1, -1)
    t = torch.tan(math.pi * d / W)
    return torch.where(t.abs() > 1e-14, torch.sin(math.pi * d) / (W * t), torch.ones_like(d))


def _voxels_last(u):
    """(H, W, W) -> (W * W, 2 H) real: a voxel's slices next to each other."""
    H, W, _ = u.shape
    return torch.view_as_real(u.reshape(H, W * W).T.contiguous()).reshape(W * W, 2 * H)


def _project(uv, theta, W, projector):
    """Ray sums (W bins, 2 H) of one angle."""
    if projector == "fourier":
        return _slice_matrix(theta, W) @ uv
    p = 0
    rows = max(1, (1 << 26) // (W * uv.shape[1]))
    for idx, w in _ray_taps(theta, W):
        for r in range(0, W, rows):
            i, ww = idx[r:r + rows], w[r:r + rows]
            p = p + (uv[i.reshape(-1)].reshape(i.shape + (-1,)) * ww[:, :, None]).sum(0)
    return p


def _project_T(g, p, theta, W, projector):
    """g (W * W, 2 H) += the transpose applied to p (W bins, 2 H)."""
    if projector == "fourier":
        g += _slice_matrix(theta, W).T @ p
        return
    rows = max(1, (1 << 26) // (W * p.shape[1]))
    for idx, w in _ray_taps(theta, W):
        for r in range(0, W, rows):
            i, ww = idx[r:r + rows], w[r:r + rows]
            g.index_add_(0, i.reshape(-1), (p[None] * ww[:, :, None]).reshape(-1, p.shape[1]))


class _Model:
    def __init__(self, case, seed, s):
        self.c, self.s = case, s
        self.mags = _mags(case["nd"])
        self.theta = _theta(case["angles"])
        self.q_used = case["functional"] != "conventional"
        as64 = lambda a: None if a is None else torch.from_numpy(a).to(DEV, F64)
        self.shift, self.pshift = (as64(_shifts(case, seed, k)) for k in ("shift", "pshift"))

    def sweep(self, u, q, grad=True, w=None, want_v=False):
        """F, g_u, g_q (or the fields, or J^H w) over the call's angles."""
        c, s = self.c, self.s
        H, W, nd = c["H"], c["W"], c["nd"]
        uv = _voxels_last(u)
        gv = torch.zeros_like(uv) if grad else None
        q = q.detach().requires_grad_(grad)
        F = 0.0
        vs = []
        if w is None and not want_v and self.q_used:
            ref = _cost(_propagate(q, 1.0, c["pad"]), s["amp_ref"].to(F64), c["functional"])
            if grad:
                ref.backward()
            F += ref.item()
        per = max(1, int(4e7 // (nd * H * W * c["pad"] ** 2)))
        for k0 in range(c["k0"], c["k1"], per):
            k1 = min(c["k1"], k0 + per)
            p = torch.stack([_project(uv, t, W, c["projector"]) for t in self.theta[k0:k1]])
            p = torch.view_as_complex(p.reshape(k1 - k0, W, H, 2)).transpose(1, 2)
            psi = torch.exp(1j * synth.KAPPA * p).contiguous().requires_grad_(grad)
            cut = lambda a: None if a is None else a[k0:k1]
            with torch.set_grad_enabled(grad):
                v = _fields(psi, q if self.q_used else None, self.mags, c["pad"], cut(self.shift),
                            cut(self.pshift))
                if want_v:
                    vs.append(v.detach())
                    continue
                if w is None:
                    f = _cost(v, s["amp"][k0:k1].to(F64), c["functional"])
                    F += f.item()
            if not grad:
                continue
            if w is None:
                f.backward()
            else:
                v.backward(w[k0 - c["k0"]:k1 - c["k0"]].to(C128))
            h = -1j * synth.KAPPA * psi.detach().conj() * psi.grad
            h = torch.view_as_real(h.transpose(1, 2).contiguous()).reshape(k1 - k0, W, 2 * H)
            for i, t in enumerate(self.theta[k0:k1]):
                _project_T(gv, h[i], t, W, c["projector"])
        if want_v:
            return torch.cat(vs)
        if not grad:
            return F
        gu = torch.view_as_complex(gv.reshape(W * W, H, 2)).T.reshape(H, W, W)
        return F, gu, q.grad if q.grad is not None else torch.zeros_like(q)

    def solve(self, u, q):
        """Dai-Yuan iterations with the halving line search of holo_cg."""
        dot = lambda a, b: sum(float((x.conj() * y).real.sum()) for x, y in zip(a, b))
        F, *g = self.sweep(u, q)
        x, eta, step, hist, halvings = [u, q], [-a for a in g], _step0(F, *g), [F], []
        for _ in range(self.c["iters"]):
            for h in range(31):
                trial = [a + step * e for a, e in zip(x, eta)]
                Ft = self.sweep(*trial, grad=False)
                if Ft <= F:
                    break
                step *= 0.5
            else:
                return None
            halvings.append(h)
            x = trial
            F, *new = self.sweep(*x)
            hist.append(F)
            gg = dot(new, new)
            den = dot([a - b for a, b in zip(new, g)], eta)
            beta = gg / den if den > 0 else 0.0
            eta = [-a + beta * e for a, e in zip(new, eta)]
            g, step = new, 2.0 * step
        return {"u": x[0], "q": x[1], "F": np.array(hist), "halvings": np.array(halvings, np.int32)}


def _exact_batch(case, seed):
    s = _batch_inputs(case, seed)
    nd, mags, fn = case["nd"], _mags(case["nd"]), case["functional"]
    F, gp, gq, o = [], [], [], 0
    for n in _batch_sizes(case):
        cut = lambda a, k=1: a[k * o:k * (o + n * n)]
        psi = cut(s["psi"]).to(C128).reshape(1, n, n).requires_grad_(True)
        q = cut(s["q"]).to(C128).reshape(n, n).requires_grad_(True)
        f = _cost(_fields(psi, None if fn == "conventional" else q, mags, 1, None, None)[0],
                  cut(s["amp"], nd).to(F64).reshape(nd, n, n), fn)
        if fn != "conventional":
            f = f + _cost(_propagate(q, 1.0), cut(s["amp_ref"]).to(F64).reshape(n, n), fn)
        f.backward()
        F.append(f.item())
        gp.append(psi.grad.reshape(-1))
        gq.append((q.grad if q.grad is not None else torch.zeros_like(q)).reshape(-1))
        o += n * n
    return {"F": torch.tensor(F, dtype=F64), "g_psi": torch.cat(gp), "g_q": torch.cat(gq)}


def exact(case, seed):
    seed = int(seed) % (1 << 27)
    if case["call"] == "batch2d":
        return _exact_batch(case, seed)
    k = case["k1"] - case["k0"]
    lerps = k * case["W"] ** 2 * case["H"] * (4 * case["iters"] + 1)
    # a few seconds to 20 s of 64-bit work at most
    if (lerps * case["W"] > 3.5e13) if case["projector"] == "fourier" else (lerps > 4e10):
        return None
    s = _tomo_inputs(case, seed)
    m = _Model(case, seed, s)
    u, q = s["u"].to(C128), s["q"].to(C128)
    if case["call"] == "fwd":
        return {"v": m.sweep(u, q, grad=False, want_v=True)}
    if case["call"] == "cg":
        return m.solve(u, q)
    F, g_u, g_q = m.sweep(u, q, w=s.get("w"))
    if case["call"] == "adj":
        return {"g_u": g_u, "g_q": g_q}
    return {"F": F if case["call"] == "loss" else torch.tensor([F], dtype=F64), "g_u": g_u, "g_q": g_q}
