"""The on-device transforms are as accurate as radix-4 register DFTs with one separately
rounded twiddle per element: relative error and gain error (the part of the error along the
result itself, which adds up over the transforms of a position) of A and A^H against 64-bit
transforms, bounded by those of an FP32 emulation of that method on the same frames."""
import numpy as np
import pytest

from gpu_util import dev, torch_cuda

SPLIT = {16: (4, 4), 32: (4, 8), 64: (8, 8), 128: (8, 16), 256: (16, 16), 512: (16, 32)}
INNER = {8: (2, 4), 16: (4, 4), 32: (4, 8)}
f32 = np.float32


def _fma(a, b, c):
    return (a.astype(np.float64) * b + c).astype(f32)


def _cmul(a, w):
    """a w with two roundings per component; `a` a pair of FP32 arrays, `w` FP32 parts."""
    wr, wi = f32(w.real), f32(w.imag)
    return _fma(a[0], wr, -(a[1] * wi)), _fma(a[0], wi, a[1] * wr)


def _add(a, b):
    return a[0] + b[0], a[1] + b[1]


def _sub(a, b):
    return a[0] - b[0], a[1] - b[1]


def _w(n, j):
    return np.exp(-2j * np.pi * j / n)


def _dft(v):
    """Register DFT: sizes 2 and 4 by sums, larger ones split with constant twiddles (those of
    quarter turns are exact)."""
    R = len(v)
    if R == 2:
        return [_add(v[0], v[1]), _sub(v[0], v[1])]
    if R == 4:
        s02, d02, s13, d = _add(v[0], v[2]), _sub(v[0], v[2]), _add(v[1], v[3]), _sub(v[1], v[3])
        d13 = (d[1], -d[0])
        return [_add(s02, s13), _add(d02, d13), _sub(s02, s13), _sub(d02, d13)]
    A, B = INNER[R]
    t = []
    for n1 in range(A):
        u = _dft([v[n1 + A * n2] for n2 in range(B)])
        row = []
        for k2 in range(B):
            j = n1 * k2 % R
            if j == 0:
                row.append(u[k2])
            elif 4 * j == R:
                row.append((u[k2][1], -u[k2][0]))
            elif 2 * j == R:
                row.append((-u[k2][0], -u[k2][1]))
            elif 4 * j == 3 * R:
                row.append((-u[k2][1], u[k2][0]))
            else:
                row.append(_cmul(u[k2], _w(R, j)))
        t.append(row)
    out = [None] * R
    for k2 in range(B):
        u = _dft([t[n1][k2] for n1 in range(A)])
        for k1 in range(A):
            out[k2 + B * k1] = u[k1]
    return out


def _lines(re, im, swap=False):
    """FP32 transform of the last axis, its longer register DFTs first (or, `swap`, last)."""
    N = re.shape[-1]
    N1, N2 = SPLIT[N][::-1] if swap else SPLIT[N]
    y = []
    for n1 in range(N1):
        u = _dft([(re[..., n1 + N1 * n2], im[..., n1 + N1 * n2]) for n2 in range(N2)])
        y.append([u[k2] if n1 * k2 == 0 else _cmul(u[k2], _w(N, n1 * k2)) for k2 in range(N2)])
    out = np.empty_like(re), np.empty_like(im)
    for k2 in range(N2):
        u = _dft([y[n1][k2] for n1 in range(N1)])
        for k1 in range(N1):
            out[0][..., k2 + N2 * k1], out[1][..., k2 + N2 * k1] = u[k1]
    return out


def emulated_fft2(x, swap=False):
    """Unitary FP32 transform of complex64 frames."""
    r = _lines(np.ascontiguousarray(x.real), np.ascontiguousarray(x.imag), swap)
    r = _lines(*(np.ascontiguousarray(np.swapaxes(c, -1, -2)) for c in r), swap)
    r = [np.swapaxes(c, -1, -2) / f32(x.shape[-1]) for c in r]
    return r[0] + 1j * r[1]


def _errors(got, ref):
    g, r = np.asarray(got, np.complex128).ravel(), np.asarray(ref, np.complex128).ravel()
    n = np.vdot(r, r).real
    return float(np.sqrt(np.vdot(g - r, g - r).real / n)), float(np.vdot(r, g - r).real / n)


def test_emulation_is_a_transform():
    rng = np.random.default_rng(3)
    for N in SPLIT:
        x = (rng.normal(size=(1, N, N)) + 1j * rng.normal(size=(1, N, N))).astype(np.complex64)
        for swap in (False, True):
            e, _ = _errors(emulated_fft2(x, swap), np.fft.fft2(x.astype(np.complex128), norm="ortho"))
            assert e < 3e-7


# frame, layout (variant), frames per call
CASES = [(32, 0, 64), (64, 0, 32), (64, 1, 32), (128, 0, 16), (128, 1, 16), (128, 6, 16), (256, 0, 4), (256, 1, 4),
         (512, 0, 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("N,variant,frames", CASES)
def test_transform_error(N, variant, frames):
    """The object is 1, so the exit wave is the probe exactly and A's only rounding is the
    transform's; likewise the probe gradient of A^H of one position is the inverse transform
    (the conjugate of the forward one, in either order of its stages) exactly. Frames of other
    random values move the emulation's own figures by 0.2 % (error) and 2 % (gain): 1.5 % and
    5 % are allowed. (Radix-2 butterflies with fused twiddles: 3 to 12 % and up to 50 % above.)"""
    torch_cuda()
    from paper_2510_20929_amd import Plan
    rng = np.random.default_rng(100 + N + variant)
    x = (rng.normal(size=(frames, N, N)) + 1j * rng.normal(size=(frames, N, N))).astype(np.complex64)
    ref = np.fft.fft2(x.astype(np.complex128), norm="ortho")
    em, egain = _errors(emulated_fft2(x), ref)
    es, esgain = _errors(emulated_fft2(x, swap=True), ref)
    obj = dev(np.ones((1, N, N), np.complex64))
    pos = dev(np.zeros((1, 2), np.float32))
    plan = Plan(frame=N, obj_h=N, obj_w=N, n_modes=frames, max_positions=1, tune={"variant": variant})
    psi = plan.apply_A(obj, dev(x[None]), pos).cpu().numpy().reshape(frames, N, N)
    ef, gf = _errors(psi, ref)
    y = dev(x[None])
    _, gp = plan.apply_AH(y, obj, dev(x[None]), pos)
    gp = gp.cpu().numpy().reshape(frames, N, N)
    ei, gi = _errors(gp, np.fft.ifft2(x.astype(np.complex128), norm="ortho"))
    print(f"N={N} variant={variant}: A {ef:.3e} gain {gf:.2e}, A^H {ei:.3e} gain {gi:.2e}, "
          f"emulated {em:.3e} gain {egain:.2e} (other order {es:.3e}, {esgain:.2e})", flush=True)
    assert plan.get_error() == 0
    assert ef <= 1.015 * em and ei <= 1.015 * max(em, es)
    assert abs(gf) <= 1.05 * abs(egain) and abs(gi) <= 1.05 * max(abs(egain), abs(esgain))
