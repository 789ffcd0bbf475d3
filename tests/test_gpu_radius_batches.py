"""The collapse passes over several radii a launch, and whole calls that take the radii from the
last to the first and leave out points that cannot change (GPU tests).

pin_collapse_times must give, bit for bit, what single-radius range calls give in increasing order:
those evaluate every point at every radius and know nothing of batches.  Sizes are the smallest of
each kind (one butterfly a line, results gathered through LDS, tiled and row layouts), with radius
counts on both sides of a batch; spectra of ordinary size, scaled to where squares of the tensor
underflow, all zero (every running maximum stays 0 and ties), and with a NaN mode.
"""

import numpy as np
import pytest

from paper_1305_1505_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n,n_radii", [(8, 2), (12, 17), (24, 16), (48, 33), (64, 1), (96, 9), (128, 5), (192, 2)])
@pytest.mark.parametrize("scale", [1.0, 1e-22, 0.0, float("nan")])
def test_whole_call_equals_single_radii(lib, prec, n, n_radii, scale):
    import torch

    if n > 96 and scale != 1.0:
        pytest.skip("the spectrum's scale is covered at the smaller sizes")
    p = lib.PIN_FP64 if prec == "fp64" else lib.PIN_FP32
    radii = W.radii_cells(n_radii, max(2.0, n / 6), 0.75) if n_radii > 1 else [1.5]
    plan = lib.Plan(n, 2.0 * n, radii, prec=p)
    dk = plan.generate_field(40 + n)
    if np.isnan(scale):
        dk[1, 2, 1] = complex(float("nan"), 0.0)
    else:
        dk *= scale
    F, R = (torch.full((n, n, n), 7, dtype=t, device="cuda") for t in (plan.real, torch.uint8))
    Fv, Rv, v = torch.full_like(F, 7), torch.full_like(R, 7), torch.full((3, n, n, n), 7, dtype=plan.real, device="cuda")
    plan.collapse_times(dk, F, R)
    plan.collapse_times_v(dk, Fv, Rv, v)
    F1, R1, v1 = torch.empty_like(F), torch.empty_like(R), torch.empty_like(v)
    plan.collapse_reset_v(F1, R1, v1)
    for r in range(n_radii):
        plan.collapse_times_range_v(dk, F1, R1, v1, r, r + 1)
    F2, R2 = torch.empty_like(F), torch.empty_like(R)
    plan.collapse_reset(F2, R2)
    half = n_radii // 2
    if half > 0:
        plan.collapse_times_range(dk, F2, R2, 0, half)
    plan.collapse_times_range(dk, F2, R2, half, n_radii)
    torch.cuda.synchronize()
    for name, a, b in (("F", F, F1), ("R", R, R1), ("F of _v", Fv, F1), ("R of _v", Rv, R1), ("v", v, v1),
                       ("F of two ranges", F2, F1), ("R of two ranges", R2, R1)):
        assert torch.equal(a, b), f"{name}: {int((a != b).sum())} of {a.numel()} differ"
    if scale == 1.0:
        assert int((R != 255).sum()) > n ** 3 // 4
    else:
        assert scale != 0.0 or bool((R == 255).all())
    plan.close()


@pytest.mark.parametrize("n", [16, 32, 128, 192])
def test_ties_keep_the_larger_radius(lib, n):
    """Radii so close that their float32 windows are the same numbers tie at every point: the first
    of each such pair is recorded, whichever order and launch the radii are taken in."""
    import torch

    radii = [r * f for r in (4.0, 2.5, 1.0) for f in (1.0, 1.0 - 1e-14)]
    plan = lib.Plan(n, 2.0 * n, radii, prec=lib.PIN_FP32)
    dk = plan.generate_field(3)
    F, R = plan.collapse_times(dk)
    Fv, Rv, _ = plan.collapse_times_v(dk)
    assert bool(((R == 255) | (R % 2 == 0)).all())
    assert torch.equal(F, Fv) and torch.equal(R, Rv)
    # a range call over radii that the state already holds changes nothing
    F2, R2 = F.clone(), R.clone()
    plan.collapse_times_range(dk, F2, R2, 0, len(radii))
    assert torch.equal(F, F2) and torch.equal(R, R2)
    plan.close()


@pytest.mark.parametrize("prec,scale", [("fp32", 1e-12), ("fp32", 3e5), ("fp32", 3e6), ("fp32", 1e9), ("fp64", 1e-62),
                                        ("fp64", 1e39), ("fp64", 1e54)])
@pytest.mark.parametrize("n", [24, 64])
def test_whole_call_equals_single_radii_at_any_scale(lib, prec, scale, n):
    """Tensors so large or small that intermediate powers of the collapse model overflow or
    underflow (in float32 F is then infinite at some points and radii): a point may be left out only
    where the model follows its bound, so whole calls still give what single radii give."""
    import torch

    radii = W.radii_cells(9, n / 6, 0.75)
    plan = lib.Plan(n, 2.0 * n, radii, prec=lib.PIN_FP64 if prec == "fp64" else lib.PIN_FP32)
    dk = plan.generate_field(61) * scale
    F, R, v = plan.collapse_times_v(dk)
    F1, R1, v1 = torch.empty_like(F), torch.empty_like(R), torch.empty_like(v)
    plan.collapse_reset_v(F1, R1, v1)
    for r in range(len(radii)):
        plan.collapse_times_range_v(dk, F1, R1, v1, r, r + 1)
    F2, R2 = plan.collapse_times(dk)
    torch.cuda.synchronize()
    for name, a, b in (("F", F, F1), ("R", R, R1), ("v", v, v1), ("F without v", F2, F1), ("R without v", R2, R1)):
        assert torch.equal(a, b), f"{name}: {int((a != b).sum())} of {a.numel()} differ"
    plan.close()
