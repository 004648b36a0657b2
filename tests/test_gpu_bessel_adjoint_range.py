"""Range of the Bessel-form adjoint's integer sums: the largest plane with an even gradient, whose
pixels all add to few radial samples, and gradients near the end of FP32's range."""
import pytest

pytestmark = pytest.mark.gpu


def test_largest_plane_even_gradient(lib):
    """8192 x 8192 pixels on eight radial samples: the gradient of the whole plane is the sum of its
    quarters' (each quarter's sums are four times smaller).  The gradient's size makes the bound of a
    term all but a power of two: 2^24 pixels reach a sample with 2^39 units each."""
    import torch
    rw = lib
    n = 8192
    plan = rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=n, ny=n, dx=20.0, dy=20.0, z=[150.0],
                   n_theta=16, n_rho=8, model=rw.MODEL_SCALAR)
    k = 2.0 * 3.141592653589793 * 1.518 / 532.0
    E = torch.full((1, 1, 1, n, n), -1j, dtype=torch.complex64, device="cuda")
    g = torch.full((1, 1, n, n), 1.99 / (8.0 * k), device="cuda")
    whole = plan.adjoint_bessel([dict()], E, g)[2].double()
    torch.cuda.synchronize()
    parts = []
    for q in range(4):
        h = torch.zeros_like(g)
        rows = slice(q * n // 4, (q + 1) * n // 4)
        h[:, :, rows] = g[:, :, rows]
        parts.append(plan.adjoint_bessel([dict()], E, h)[2].double())
        torch.cuda.synchronize()
        del h
    plan.close()
    size = sum(p.abs() for p in parts)
    assert size > 0 and torch.isfinite(size)
    # FP32 rounding of eight samples and of the products of their sums
    assert (whole - sum(parts)).abs() < 1e-5 * size


def test_gradient_near_the_end_of_the_range(lib):
    """2 g E of 2^123: the projections fit FP32, their bound does not."""
    import torch
    rw = lib
    plan = rw.Plan(form=rw.FORM_BESSEL, na=1.4, wavelength=532.0, n_i=1.518, nx=9, ny=9, dx=20.0, dy=20.0, z=[0.0],
                   focal_length=1000.0, n_theta=64, n_rho=64)
    E = torch.zeros(1, 1, 3, 9, 9, dtype=torch.complex64, device="cuda")
    E[0, 0, 0, 2, 3] = 1.0
    g = torch.zeros(1, 1, 9, 9, device="cuda")
    g[0, 0, 2, 3] = 1.0
    small = plan.adjoint_bessel([dict(z_offset=70.0)], E, g)
    large = plan.adjoint_bessel([dict(z_offset=70.0)], E, g * 2.0 ** 122)
    torch.cuda.synchronize()
    plan.close()
    assert small[2].abs() > 0
    assert torch.equal(large[2], small[2] * 2.0 ** 122)
