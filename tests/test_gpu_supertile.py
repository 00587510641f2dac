"""Edges of the supertile kernels: odd grids, degrees 2 and 3, bands with and
without BC rows, right-hand sides split over launches, and many partial sums.

References are the forward operator (pinned to the oracle elsewhere), one
right-hand side at a time, and the true residual.  Tolerances: a sum of K
products in another order moves by at most K u times the sum of their sizes;
K is below 2000 and u = 1.1e-16 (FP64 arithmetic for both types), so 1e-12 of
the largest entry for FP64 and two roundings to FP32 (2.4e-7) for FP32.
"""

import pytest

pytestmark = pytest.mark.gpu
BANDS = [("circle", 5, 3), ("circle", 131, 2), ("sphere", 5, 3), ("sphere", 13, 2),
         ("sphere", 33, 3), ("torus", 21, 3)]


def _band(kind, N, p=3, bc=True):
    from paper_2305_04711_amd import cpm
    surface, ibc = {"circle": (cpm.circle, lambda: cpm.point_ibc((1.0, 0.0), (0.0, 1.0))),
                    "sphere": (cpm.sphere, lambda: cpm.latitude_ibc(0.25)),
                    "torus": (lambda: cpm.torus(1.0, 0.4),
                              lambda: cpm.meridian_ibc(1.0, 0.0))}[kind]
    return cpm.Band(surface(), [ibc()] if bc else [], N, p=p)


def _vec(band, nrhs, seed, dtype="float64"):
    import torch
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    u = torch.randn(nrhs, band.n, generator=gen, device="cuda", dtype=torch.float64)
    return u.to(getattr(torch, dtype))


@pytest.mark.parametrize("kind,N,p", BANDS)
@pytest.mark.parametrize("bc", [False, True])
def test_transpose_is_the_adjoint_of_the_forward_operator(kind, N, p, bc):
    import torch
    from paper_2305_04711_amd import cpm
    band = _band(kind, N, p, bc)
    u, w = _vec(band, 3, 1), _vec(band, 3, 2)
    Au = cpm.apply(band, u, 0.5, -1.0)
    Atw = cpm.apply_transpose(band, w, 0.5, -1.0)
    for k in range(3):
        scale = (torch.linalg.norm(w[k]) * torch.linalg.norm(Au[k])).item()
        assert abs(torch.dot(Atw[k], u[k]).item() - torch.dot(w[k], Au[k]).item()) <= 1e-12 * scale


@pytest.mark.parametrize("kind,N,nrhs", [("circle", 64, 5), ("sphere", 24, 20), ("sphere", 32, 70)])
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 2.4e-7)])
def test_transpose_of_many_right_hand_sides_equals_one_at_a_time(kind, N, nrhs, dtype, tol):
    # 20 and 70 columns take one wave per supertile where one column takes
    # two; 70 columns are more than one launch's buffer holds
    import torch
    from paper_2305_04711_amd import cpm
    band = _band(kind, N)
    w = _vec(band, nrhs, 3, dtype)
    z = cpm.apply_transpose(band, w, 0.0, -1.0)
    for k in range(nrhs):
        one = cpm.apply_transpose(band, w[k].contiguous(), 0.0, -1.0)
        assert (z[k] - one).abs().max().item() <= tol * one.abs().max().item()


@pytest.mark.parametrize("kind,N,p", [("circle", 40, 3), ("sphere", 24, 2), ("sphere", 72, 3)])
@pytest.mark.parametrize("nrhs", [2, 7, 40])
@pytest.mark.parametrize("dtype,tol", [("float64", 1e-12), ("float32", 2.4e-7)])
def test_forward_of_many_right_hand_sides_equals_one_at_a_time(kind, N, p, nrhs, dtype, tol):
    # columns apart, several to a workgroup with a shorter last group, in turn
    import torch
    from paper_2305_04711_amd import cpm
    band = _band(kind, N, p)
    u = _vec(band, nrhs, 4, dtype)
    v = cpm.apply(band, u, 0.0, -1.0)
    for k in range(nrhs):
        one = cpm.apply(band, u[k].contiguous(), 0.0, -1.0)
        assert (v[k] - one).abs().max().item() <= tol * one.abs().max().item()


@pytest.mark.parametrize("N", [64, 112, 136])
def test_solve_residual_with_few_and_many_partial_sums(N):
    # 1400, 4000 and 6000 partials of an apply: in one and two passes of a
    # thread's loads, and folded by a kernel of their own first
    import torch
    from paper_2305_04711_amd import cpm
    band = _band("sphere", N)
    b = cpm.rhs(band, torch.ones(band.n_s, device="cuda", dtype=torch.float64),
                torch.zeros(band.n_c, device="cuda", dtype=torch.float64), -1.0)
    x, st = cpm.solve(band, b, 1.0, -1.0, tol=1e-8, mode="f64")
    r = b - cpm.apply(band, x, 1.0, -1.0)
    assert (torch.linalg.norm(r) / torch.linalg.norm(b)).item() <= 1e-8
