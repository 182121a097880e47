"""Performance cases of the library: the calls a reconstruction program makes, through
the Python entry points (``Plan``, ``Batch``, ``ptycho_loss``), at the sizes of the
synthetic workloads and of the paper's call shapes.

``listed()`` holds the named cases, ``draw(rng)`` more of the same ranges. ``prepare``
makes what a program holds before a call (inputs on the GPU, the plan, the output
buffers), ``run`` is one call, ``work`` the bytes and flops the path cannot do without,
``exact`` the same outputs in 64 bits from plain torch. The implementation choice of a
plan is the one the autotuner makes for the shape (``_tune``); near-field, Fourier-shift
and autograd programs use the defaults, which is what the autotuner leaves them with.
"""
import math

import torch

from paper_2510_20929_amd import Batch, Plan, ptycho_loss

PHOTONS = 1.0e4  # per frame
DEV = "cuda"


# ----------------------------------------------------------------------------- cases

def _case(kind, N, M, K, H, W, *, E=1, S=1, loss="amplitude", weights="none", grads="obj+probe+pos",
          scan="raster", lambda_z=0.0, det_lambda_z=0.0, subpixel="bilinear", tuned=True, datasets=""):
    return dict(kind=kind, N=N, M=M, E=E, S=S, K=K, H=H, W=W, loss=loss, weights=weights, grads=grads, scan=scan,
                lambda_z=float(lambda_z), det_lambda_z=float(det_lambda_z), subpixel=subpixel, tuned=tuned,
                datasets=datasets)


def listed():
    return [
        # the smallest training step: a minibatch of 24 frames of 64^2, the loss as a torch
        # operation (forward and backward), an optimiser of object and probe around it
        dict(_case("autograd", 64, 2, 24, 181, 203, grads="obj+probe", scan="random", tuned=False),
             name="autograd 64^2 B24"),
        # a quick single-mode reconstruction of a small raster scan at integer positions
        dict(_case("step", 64, 1, 625, 256, 256, grads="obj+probe", scan="integer"), name="scan 64^2 K625"),
        # the headline workload: 4 modes, 2000 sub-pixel positions, Poisson loss, position refinement
        dict(_case("step", 128, 4, 2000, 1024, 1024, loss="poisson"), name="modes 128^2 M4 K2000"),
        # a mode-heavy dataset (30 modes, 413 x 535 object) in minibatches of 50
        dict(_case("step", 128, 30, 50, 413, 535, scan="random"), name="modes 128^2 M30 B50"),
        # the same dataset in one call: the largest work of a full-batch gradient
        dict(_case("step", 128, 30, 6732, 413, 535), name="modes 128^2 M30 K6732"),
        # orthogonal probe relaxation in minibatches of 16: 15 modes, 3 eigenprobes, no position refinement
        dict(_case("step", 128, 15, 16, 372, 372, E=3, weights="opr", grads="obj+probe+weights", scan="random"),
             name="OPR 128^2 M15 B16"),
        # eight eigenprobes over a large jittered raster of 256^2 frames
        dict(_case("step", 256, 1, 2500, 1129, 1129, E=8, weights="opr", grads="obj+probe+weights"),
             name="OPR 256^2 E8 K2500"),
        # the same relaxation with 512^2 detectors in minibatches of 16
        dict(_case("step", 512, 15, 16, 1476, 1476, E=3, weights="opr", grads="obj+probe+weights", scan="random"),
             name="OPR 512^2 M15 B16"),
        # a thick sample: 8 slices, 2 modes, Fresnel propagation between the slices
        dict(_case("step", 128, 2, 1500, 1200, 1200, S=8, lambda_z=81.92), name="slices 128^2 S8 K1500"),
        # a near-field detector whose distance is refined with the positions
        dict(_case("step", 128, 2, 300, 511, 437, det_lambda_z=60.0, grads="obj+probe+pos+lambda_z", tuned=False),
             name="near field 128^2 K300"),
        # predicted patterns and loss of a validation set: the forward direction alone
        dict(_case("forward", 256, 3, 331, 901, 777, weights="amp"), name="forward 256^2 M3 K331"),
        # independent reconstructions of uneven size together in one batched launch
        dict(_case("batch", 512, 4, 1, 0, 0, weights="amp", grads="obj+probe+pos+weights",
                   datasets="64x1x900 64x3x411 128x2x640 128x4x263 256x1x500 256x2x207 512x1x223 512x3x200"),
             name="batch of 8 datasets"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: every entry point, frame size, loss and option above,
    position counts from a minibatch to a full scan, odd object sizes."""
    what = rng.choice(["autograd", "small", "modes", "modes", "minibatch", "opr", "large", "large", "slices", "near",
                       "fourier", "forward", "batch"])
    loss = rng.choice(["amplitude", "poisson"])

    def extent(N, K, step):  # object of a scan of K positions at about `step` px, odd sizes among them
        side = max(2.0, math.sqrt(K)) * step
        return int(N + 4 + side * rng.uniform(0.7, 1.4)), int(N + 4 + side * rng.uniform(0.7, 1.4))

    if what == "autograd":
        N, M, K = rng.choice([16, 32, 64, 128]), rng.randint(1, 4), _log(rng, 8, 200)
        H, W = extent(N, K, 0.2 * N)
        return _case("autograd", N, M, K, H, W, loss=loss, grads="obj+probe", scan="random", tuned=False)
    if what == "small":
        N, K = rng.choice([32, 64, 64]), _log(rng, 60, 3000)
        H, W = extent(N, K, N / 8)
        return _case("step", N, rng.randint(1, 3), K, H, W, loss=loss, grads="obj+probe", scan="integer")
    if what == "modes":
        M = rng.randint(1, 12)
        K = _log(rng, 300, 3500)
        H, W = extent(128, K, rng.uniform(4, 20))
        return _case("step", 128, M, K, H, W, loss=loss)
    if what == "minibatch":
        N, K = rng.choice([64, 128, 128]), _log(rng, 16, 200)
        return _case("step", N, rng.randint(2, 30), K, N + rng.randint(100, 420), N + rng.randint(100, 420),
                     scan="random")
    if what == "opr":
        K = _log(rng, 12, 960)
        H, W = extent(128, 961, 8)
        return _case("step", 128, rng.randint(2, 15), K, H, W, E=rng.randint(2, 5), weights="opr",
                     grads="obj+probe+weights", scan="random")
    if what == "large":
        N = rng.choice([256, 256, 512])
        M, E = rng.randint(1, 6), rng.choice([1, 3, 8])
        K = _log(rng, 16, 1600 if N == 256 else 260)
        H, W = extent(N, K, 0.1 * N)
        return _case("step", N, M, K, H, W, E=E, loss=loss, weights="opr" if E > 1 else rng.choice(["none", "amp"]),
                     grads="obj+probe" + ("+weights" if E > 1 else "+pos"), scan=rng.choice(["raster", "random"]))
    if what == "slices":
        N, S, K = rng.choice([64, 128, 128]), rng.randint(2, 8), _log(rng, 100, 1500)
        H, W = extent(N, K, 0.15 * N)
        return _case("step", N, rng.randint(1, 3), K, H, W, S=S, loss=loss, lambda_z=(N / 2) ** 2 / 50,
                     grads="obj+probe+pos" + rng.choice(["", "+lambda_z"]))
    if what == "near":
        N, K = rng.choice([64, 128]), _log(rng, 50, 1000)
        H, W = extent(N, K, 0.1 * N)
        return _case("step", N, rng.randint(1, 3), K, H, W, loss=loss, det_lambda_z=rng.uniform(20, 120),
                     grads="obj+probe+pos+lambda_z", tuned=False)
    if what == "fourier":
        N, K = rng.choice([64, 128]), _log(rng, 50, 1000)
        H, W = extent(N, K, 0.1 * N)
        return _case("step", N, rng.randint(1, 3), K, H, W, loss=loss, subpixel="fourier", tuned=False)
    if what == "forward":
        N = rng.choice([64, 128, 256, 512])
        K = _log(rng, 20, 40000 // N)
        H, W = extent(N, K, 0.1 * N)
        return _case("forward", N, rng.randint(1, 4), K, H, W, loss=loss, weights=rng.choice(["none", "amp"]))
    top = {64: 1200, 128: 700, 256: 350, 512: 110}
    sets = " ".join("%dx%dx%d" % (N, rng.randint(1, 4), _log(rng, 40, top[N]))
                    for N in (rng.choice([64, 128, 256, 512]) for _ in range(rng.randint(2, 8))))
    return _case("batch", 512, 4, 1, 0, 0, weights="amp", grads="obj+probe+pos+weights", datasets=sets)


def _tune(c):
    """The autotuner's choice for the shape of a step (its measured winners: the layouts with
    the frame in LDS at 128^2, one workgroup a mode group where a call has few positions)."""
    if not c["tuned"]:
        return None
    N, M, E, S, K = c["N"], c["M"], c["E"], c["S"], c["K"]
    few = S == 1 and M > 1 and K < 256
    if N == 128:
        if few:
            return dict(variant=4 if E > 1 else 5, mode_groups=min(M, -(-512 // K)))
        return dict(variant=5) if S > 1 or E > 1 else dict(variant=6, recompute=1)
    if few:
        return dict(mode_groups=min(M, -(-512 // K)))
    return dict(grid=512) if N == 64 and S == 1 else None


def _parts(c):
    """The datasets of a case: itself, or a batch's (raster at 0.4 N, object to fit)."""
    if c["kind"] != "batch":
        return [c]
    out = []
    for text in c["datasets"].split():
        N, M, K = (int(v) for v in text.split("x"))
        side = int(math.ceil((math.ceil(math.sqrt(K)) - 1) * 0.4 * N)) + N + 3
        out.append(dict(c, N=N, M=M, K=K, H=side, W=side))
    return out


# ----------------------------------------------------------------------------- inputs

def _smooth(shape, sigma, g):
    """White noise with a Gaussian blur of `sigma` px (periodic), zero mean, unit deviation."""
    x = torch.randn(shape, generator=g, device=DEV)
    fy = torch.fft.fftfreq(shape[-2], device=DEV)[:, None]
    fx = torch.fft.rfftfreq(shape[-1], device=DEV)[None]
    x = torch.fft.irfft2(torch.fft.rfft2(x) * torch.exp(-2 * (math.pi * sigma) ** 2 * (fy * fy + fx * fx)), s=shape[-2:])
    return (x - x.mean()) / x.std()


def _modes(N, M, waist, decay, phase_radius):
    """The first M Hermite-Gauss modes with a quadratic phase, orthonormal, powers exp(-j / decay)."""
    t = torch.arange(N, dtype=torch.float64, device=DEV) - (N - 1) / 2
    u = t * (math.sqrt(2) / waist)
    orders = [(a, d - a) for d in range(M + 1) for a in range(d, -1, -1)][:M]
    he = [torch.ones_like(u), 2 * u]
    for n in range(2, max(max(o) for o in orders) + 1):
        he.append(2 * u * he[-1] - 2 * (n - 1) * he[-2])
    env = torch.exp(-(t[:, None] ** 2 + t[None] ** 2) / waist ** 2)
    A = torch.stack([(he[a][:, None] * he[b][None] * env).reshape(-1) for a, b in orders], 1)
    q, _ = torch.linalg.qr(A.cpu())
    power = torch.exp(-torch.arange(M, dtype=torch.float64) / decay)
    q = (q * torch.sqrt(power / power.sum())).T.reshape(M, N, N).to(DEV)
    return q * torch.exp(1j * math.pi * (t[:, None] ** 2 + t[None] ** 2) / phase_radius ** 2)


def _positions(c, g):
    N, K, H, W = c["N"], c["K"], c["H"], c["W"]
    hy, hx = H - N - 2, W - N - 2
    if c["scan"] == "random":
        return torch.rand((K, 2), generator=g, device=DEV, dtype=torch.float64) * torch.tensor([hy, hx], device=DEV)
    ny = min(K, max(1, round(math.sqrt(K * hy / max(hx, 1)))))
    nx = -(-K // ny)
    i = torch.arange(K, device=DEV, dtype=torch.float64)
    y, x = torch.floor(i / nx) * (hy / max(ny - 1, 1)), (i % nx) * (hx / max(nx - 1, 1))
    r = torch.stack([y, x], 1)
    if c["scan"] == "integer":
        return torch.floor(r)
    return r + torch.rand((K, 2), generator=g, device=DEV, dtype=torch.float64)


def _intensity(c, obj, probe, pos, w, lz=None):
    """Intensities of a few positions, in the precision of the inputs (plain torch)."""
    N, S = c["N"], c["S"]
    fl = torch.floor(pos.detach())
    f, y0, x0 = (pos - fl).to(obj.real.dtype), fl[:, 0].long(), fl[:, 1].long()
    fourier = c["subpixel"] == "fourier"
    span = torch.arange(N if fourier else N + 1, device=DEV)
    iy, ix = (y0[:, None] + span).clamp(max=c["H"] - 1), (x0[:, None] + span).clamp(max=c["W"] - 1)
    at = iy[:, :, None] * c["W"] + ix[:, None, :]
    fy, fx = f[:, 0, None, None], f[:, 1, None, None]
    if w is None:
        P = probe[0][None]
    else:
        P = torch.tensordot(w.to(probe.dtype), probe, 1)
    psi = P
    prop = None
    if S > 1 or c["det_lambda_z"]:
        q = torch.fft.fftfreq(N, device=DEV, dtype=torch.float64)
        z = lz if lz is not None else (c["lambda_z"] if S > 1 else c["det_lambda_z"])
        prop = torch.exp(-1j * math.pi * z * (q[:, None] ** 2 + q[None] ** 2)).to(obj.dtype)
    for s in range(S):
        win = torch.index_select(obj[s].reshape(-1), 0, at.reshape(-1)).reshape(at.shape)
        if fourier:
            kap = torch.fft.fftfreq(N, device=DEV, dtype=torch.float64) * N
            ph = (2 * math.pi / N) * (kap[None, :, None] * fy + kap[None, None, :] * fx)
            o = torch.fft.ifft2(torch.fft.fft2(win) * torch.exp(1j * ph).to(win.dtype))
        else:
            o = (1 - fy) * ((1 - fx) * win[:, :-1, :-1] + fx * win[:, :-1, 1:]) \
                + fy * ((1 - fx) * win[:, 1:, :-1] + fx * win[:, 1:, 1:])
        psi = psi * o[:, None]
        if s < S - 1:
            psi = torch.fft.ifft2(prop * torch.fft.fft2(psi))
    if c["det_lambda_z"]:
        psi = torch.fft.ifft2(prop * torch.fft.fft2(psi))
        return psi.real.square().add(psi.imag.square()).sum(1)
    psi = torch.fft.fft2(psi, norm="ortho")
    return torch.fft.fftshift(psi.real.square().add(psi.imag.square()).sum(1), dim=(-2, -1))


def _chunk(c, per=3.0e9):
    return max(1, int(per / (c["N"] ** 2 * 16.0 * (c["M"] * (c["S"] + 2) + 6))))


def _inputs(c, seed):
    """A scan's tensors: photon counts drawn from a truth, and a start point off it."""
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 7919 + 13)
    N, M, E, S, K, H, W = (c[k] for k in ("N", "M", "E", "S", "K", "H", "W"))
    if S > 1:
        obj = torch.exp(0.05j * torch.stack([_smooth((H, W), 2.0, g) for _ in range(S)]))
    else:
        obj = ((0.9 + 0.05 * _smooth((H, W), 2.0, g)) * torch.exp(0.25j * _smooth((H, W), 2.0, g)))[None]
    primary = _modes(N, M, N / 8.0, max(4.0, M / 5.0), N / 4.0)
    eig = [primary] + [primary * (0.5 * torch.complex(_smooth((N, N), N / 16.0, g), _smooth((N, N), N / 16.0, g)))
                       for _ in range(E - 1)]
    probe = torch.stack(eig) * math.sqrt(PHOTONS / float(primary.abs().square().sum() * obj[0].abs().square().mean()))
    obj, probe = obj.to(torch.complex64), probe.to(torch.complex64)
    true = _positions(c, g)
    w = None
    if c["weights"] == "opr":
        w = torch.randn((K, E), generator=g, device=DEV) * torch.tensor([0.1] + [0.05] * (E - 1), device=DEV)
        w[:, 0] += 1.0
    elif c["weights"] == "amp":
        w = 0.85 + 0.3 * torch.rand((K, E), generator=g, device=DEV)
    counts = torch.empty((K, N, N), device=DEV)
    step = _chunk(c)
    for k in range(0, K, step):
        I = _intensity(c, obj, probe, true[k:k + step].float(), None if w is None else w[k:k + step])
        counts[k:k + step] = torch.poisson(I.clamp_min(0).float(), generator=g)
    start_obj = obj * torch.exp(0.1 * torch.complex(_smooth((H, W), 2.0, g), _smooth((H, W), 2.0, g)))
    scale = float(probe.abs().max())
    start_probe = probe + 0.05 * scale * torch.complex(_smooth(probe.shape, 2.0, g), _smooth(probe.shape, 2.0, g))
    if c["scan"] == "integer":
        pos = true
    else:
        pos = true + torch.rand(true.shape, generator=g, device=DEV, dtype=torch.float64) - 0.5
        pos = torch.minimum(pos.clamp_min(0.0), torch.tensor([H - N - 1.001, W - N - 1.001], device=DEV))
    return dict(obj=start_obj.to(torch.complex64).contiguous(), probe=start_probe.to(torch.complex64).contiguous(),
                positions=pos.float().contiguous(), I_meas=counts, weights=w)


class _Shape:
    """What ``Batch`` reads of a dataset."""

    def __init__(self, c):
        self.N, self.M, self.E, self.S, self.H, self.W, self.K = (c[k] for k in ("N", "M", "E", "S", "H", "W", "K"))
        self.loss, self.eps, self.lambda_z = c["loss"], 1e-3, c["lambda_z"]


def _outputs(c):
    """The gradient buffers a program keeps from step to step."""
    z = dict(device=DEV)
    out = {"loss": torch.zeros(1, dtype=torch.float64, **z)}
    grads = c["grads"].split("+")
    if "obj" in grads:
        out["g_obj"] = torch.zeros((c["S"], c["H"], c["W"]), dtype=torch.complex64, **z)
    if "probe" in grads:
        out["g_probe"] = torch.zeros((c["E"], c["M"], c["N"], c["N"]), dtype=torch.complex64, **z)
    if "pos" in grads:
        out["g_pos"] = torch.zeros((c["K"], 2), **z)
    if "weights" in grads:
        out["g_weights"] = torch.zeros((c["K"], c["E"]), **z)
    if "lambda_z" in grads:
        out["g_lambda_z"] = torch.zeros(1, dtype=torch.float64, **z)
    return out


def prepare(case, seed):
    c = dict(case)
    grads = tuple(c["grads"].split("+"))
    if c["kind"] == "batch":
        parts = _parts(c)
        batch = Batch([_Shape(p) for p in parts])
        tensors = [_inputs(p, seed + 101 * i) for i, p in enumerate(parts)]
        outs = [batch.bind(i, t["obj"], t["probe"], t["positions"], t["I_meas"], weights=t["weights"])
                for i, t in enumerate(tensors)]
        return dict(kind="batch", batch=batch, grads=grads, outs=outs, tensors=tensors)
    t = _inputs(c, seed)
    plan = Plan(c["N"], c["M"], c["E"], c["S"], c["H"], c["W"], c["loss"], 1e-3, c["lambda_z"], 0.0, c["K"], _tune(c),
                c["det_lambda_z"] or None, c["subpixel"])
    s = dict(kind=c["kind"], plan=plan, grads=grads, **t)
    if c["kind"] == "forward":
        s["I_pred"] = torch.zeros((c["K"], c["N"], c["N"]), device=DEV)
        s["loss"] = torch.zeros(1, dtype=torch.float64, device=DEV)
    elif c["kind"] == "step":
        s["out"] = _outputs(c)
    else:
        s["obj"].requires_grad_(True)
        s["probe"].requires_grad_(True)
    return s


def _single(x):
    """A loss as a program's history keeps it: the library's sum of single-precision terms is
    held in 64 bits, the history in 32."""
    return x.detach().to(torch.float32)


def run(s):
    if s["kind"] == "batch":
        s["batch"].launch(s["grads"])
        return [dict(o, loss=_single(o["loss"])) for o in s["outs"]]
    if s["kind"] == "forward":
        s["plan"].forward(s["obj"], s["probe"], s["positions"], s["I_meas"], weights=s["weights"], I_pred=s["I_pred"],
                          loss=s["loss"])
        return dict(I_pred=s["I_pred"], loss=_single(s["loss"]))
    if s["kind"] == "autograd":
        loss = ptycho_loss(s["obj"], s["probe"], s["positions"], s["I_meas"], s["plan"], s["weights"])
        g_obj, g_probe = torch.autograd.grad(loss, (s["obj"], s["probe"]))
        return dict(loss=_single(loss).reshape(1), g_obj=g_obj, g_probe=g_probe)
    out = s["plan"].forward_adjoint(s["obj"], s["probe"], s["positions"], s["I_meas"], weights=s["weights"],
                                    grads=s["grads"], out=s["out"])
    out = dict(out, loss=_single(out["loss"]))
    if "g_lambda_z" in out:
        out["g_lambda_z"] = _single(out["g_lambda_z"])
    return out


# ----------------------------------------------------------------------------- work, exact

def work(case):
    total = {"bytes": 0.0, "flops": 0.0}
    for c in _parts(case):
        N, M, E, S, K = (c[k] for k in ("N", "M", "E", "S", "K"))
        NN = float(N * N)
        adj = 1 if c["kind"] == "forward" else 2
        obj = 8.0 * S * c["H"] * c["W"]
        probe = 8.0 * E * M * NN
        per = 4.0 * NN + 8.0 + (4.0 * E if c["weights"] != "none" else 0.0)
        if adj == 1:
            total["bytes"] += obj + probe + K * (per + 4.0 * NN)
        else:
            total["bytes"] += 2 * (obj + probe) + K * (per + 8.0 + (4.0 * E if "weights" in c["grads"] else 0.0))
        ffts = M * (1 + 2 * (S - 1) + (1 if c["det_lambda_z"] else 0)) + (2 if c["subpixel"] == "fourier" else 0)
        fft = 5.0 * NN * math.log2(NN)
        # per pixel: patch taps 14, exit wave 6, probe synthesis 4 E, intensity 3, conjugate products 16
        element = NN * (14.0 + M * (6.0 * S + 3.0 + (4.0 * E if c["weights"] != "none" else 0.0)
                                    + (16.0 * S if adj == 2 else 0.0)))
        total["flops"] += K * (adj * ffts * fft + element)
    return total


def exact(case, seed):
    if case["kind"] == "batch":
        return [_exact(p, seed + 101 * i) for i, p in enumerate(_parts(case))]
    return _exact(case, seed)


def _exact(c, seed):
    t = _inputs(c, seed)
    grads = [] if c["kind"] == "forward" else c["grads"].split("+")
    N, K = c["N"], c["K"]
    obj = t["obj"].to(torch.complex128).requires_grad_("obj" in grads)
    probe = t["probe"].to(torch.complex128).requires_grad_("probe" in grads)
    pos = t["positions"].double().requires_grad_("pos" in grads)
    w = None if t["weights"] is None else t["weights"].double().requires_grad_("weights" in grads)
    # the propagator's products are single-precision parameters of the plan
    lz = torch.tensor(c["lambda_z"] if c["S"] > 1 else c["det_lambda_z"], dtype=torch.float32).double().to(DEV)
    lz.requires_grad_("lambda_z" in grads)
    eps = float(torch.tensor(1e-3, dtype=torch.float32))
    total = torch.zeros(1, dtype=torch.float64, device=DEV)
    pred = torch.empty((K, N, N), dtype=torch.float64, device=DEV) if c["kind"] == "forward" else None
    step = _chunk(c, 6.0e9)
    for k in range(0, K, step):
        I = _intensity(c, obj, probe, pos[k:k + step], None if w is None else w[k:k + step], lz)
        Im = t["I_meas"][k:k + step].double()
        if c["loss"] == "poisson":
            loss = (I - Im * torch.log(I + eps)).sum()
        else:
            loss = (torch.sqrt(I.clamp_min(1e-30)) - torch.sqrt(Im)).square().sum()
        loss = loss / (K * N * N)
        if grads:
            loss.backward()
        else:
            pred[k:k + step] = I
        total += loss.detach()
    if c["kind"] == "forward":
        return dict(I_pred=pred, loss=total)
    out = dict(loss=total)
    for name, x in (("obj", obj), ("probe", probe), ("pos", pos), ("weights", w), ("lambda_z", lz)):
        if name in grads:
            out["g_" + name] = x.grad.reshape(1) if name == "lambda_z" else x.grad
    return out
