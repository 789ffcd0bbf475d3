"""v_max and the third-order displacement where a thread of the strided passes holds several
butterflies (GPU tests): 384^3 and 768^3 in float32, whose butterflies are shared by 768 threads, and
at 768^3 the y pass that keeps a pair's input in registers.  Against the same fields from torch's
transforms in 64 bits, with the bounds of the smaller sizes (1e-5 relative RMS, 1e-4 of the largest
value: chains of float32 transforms, each ~eps32 log2 N)."""

import math

import pytest

pytestmark = [pytest.mark.gpu, pytest.mark.timeout(300)]


class Reference:
    """Fields of a half spectrum in 64 bits."""

    def __init__(self, dk, box):
        import torch

        self.torch = torch
        self.n = n = dk.shape[0]
        self.dk = dk.to(torch.complex128)
        f = torch.fft.fftfreq(n, 1.0 / n, dtype=torch.float64, device="cuda")
        self.f = (f.view(n, 1, 1), f.view(1, n, 1),
                  torch.arange(n // 2 + 1, dtype=torch.float64, device="cuda").view(1, 1, -1))
        self.f2 = self.f[0] ** 2 + self.f[1] ** 2 + self.f[2] ** 2
        self.inv = 1 / self.f2.clamp_min(1)
        self.inv[0, 0, 0] = 0
        for i in range(3):
            self.inv.select(i, n // 2).zero_()
        self.length = box / (2 * math.pi)

    def real(self, modes):
        return self.torch.fft.irfftn(modes, s=(self.n,) * 3)

    def gradient(self, a, radius):
        """Component a of the Zel'dovich displacement of the field smoothed on `radius` cells."""
        w = self.torch.exp(-0.5 * self.f2 * (2 * math.pi * radius / self.n) ** 2)
        return self.real(self.dk * (1j * self.length * self.f[a] * self.inv * w))

    def tensor(self, source):
        return {(i, j): self.real(self.f[i] * self.f[j] * self.inv * source) for i in range(3) for j in range(i, 3)}

    def lpt3(self):
        rfftn = self.torch.fft.rfftn
        a = self.tensor(self.dk)
        b = self.tensor(rfftn(a[0, 0] * a[1, 1] + a[0, 0] * a[2, 2] + a[1, 1] * a[2, 2]
                              - a[0, 1] ** 2 - a[0, 2] ** 2 - a[1, 2] ** 2))

        def e(t, i, j):
            return t[min(i, j), max(i, j)]

        det = (a[0, 0] * (a[1, 1] * a[2, 2] - a[1, 2] ** 2) - a[0, 1] * (a[0, 1] * a[2, 2] - a[1, 2] * a[0, 2])
               + a[0, 2] * (a[0, 1] * a[1, 2] - a[1, 1] * a[0, 2]))
        mixed = (a[0, 0] + a[1, 1] + a[2, 2]) * (b[0, 0] + b[1, 1] + b[2, 2])
        for i in range(3):
            for j in range(3):
                mixed -= e(a, i, j) * e(b, i, j)
        s = rfftn(det / 3 - 5 / 21 * mixed)
        del det, mixed
        curl = []
        for i in range(3):
            j, k = (i + 1) % 3, (i + 2) % 3
            curl.append(rfftn(sum(e(a, j, m) * e(b, m, k) - e(a, k, m) * e(b, m, j) for m in range(3)) / 7))
        for i in range(3):
            j, k = (i + 1) % 3, (i + 2) % 3
            yield self.real(1j * self.length * self.inv * (-self.f[i] * s + self.f[j] * curl[k] - self.f[k] * curl[j]))


def _close(got, ref, what):
    d = got.double() - ref
    rms = float(d.pow(2).sum().sqrt() / ref.pow(2).sum().sqrt())
    worst = float(d.abs().max() / ref.abs().max())
    print(f"[wide tiles] {what}: relative rms {rms:.3g}, largest {worst:.3g}", flush=True)
    assert rms <= 1e-5 and worst <= 1e-4, what


@pytest.mark.parametrize("n", [384, 768])
def test_wide_tiles_match_torch(lib, n):
    import torch

    box, radii = 2.0 * n, [6.0, 1.5]
    plan = lib.Plan(n, box, radii, prec=lib.PIN_FP32)
    dk = plan.generate_field(500 + n)
    F, R, v = plan.collapse_times_v(dk)
    ref = Reference(dk, box)
    for a in range(3):
        g = [ref.gradient(a, r) for r in radii]
        want = torch.where(R == 0, g[0], torch.where(R == 1, g[1], torch.zeros_like(g[0])))
        _close(v[a], want, f"{n}^3 v_max[{a}]")
        del g, want
    assert int((R == 0).sum()) > 0 and int((R == 1).sum()) > n ** 3 // 4
    assert bool(((R == 255) == (F == 0)).all())
    psi3 = plan.lpt3_displacement(dk)
    for a, want in enumerate(ref.lpt3()):
        _close(psi3[a], want, f"{n}^3 psi3[{a}]")
    plan.close()
    del ref, dk, F, R, v, psi3
    torch.cuda.empty_cache()
