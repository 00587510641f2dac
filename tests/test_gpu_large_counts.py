"""More than 2^22 explicit interpolation rows (2^28 stored columns), blocks
whose 64 slots number more than 2^28, and right-hand sides of more than 2^28
entries: the sphere with eight latitude boundaries at h = 1/1224.

The forward operator reads the columns as the apply stores them, the transpose
lists that were sorted from the builder's own, the batch a copy: they have to
agree.  <A u, w> = <u, A^T w> to rounding errors, 1e-12 of the norms with room;
one row whose columns are missing or wrong moves it by about 1/n = 6e-9 of them.
"""

import pytest

pytestmark = pytest.mark.gpu


def test_more_than_four_million_explicit_rows():
    import torch
    from paper_2305_04711_amd import cpm
    band = cpm.Band(cpm.sphere(), [cpm.latitude_ibc(z) for z in
                                   (-0.65, -0.5, -0.3, -0.1, 0.1, 0.3, 0.5, 0.65)], 1224)
    n, n_s, n_c = band.n, band.n_s, band.n_c
    print("DOFs", n, "explicit rows", band.info["n_erows"], band.info["n_lrows"], flush=True)
    assert band.info["n_erows"] > 1 << 22
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    u = torch.randn(n, generator=gen, device="cuda", dtype=torch.float64)
    w = torch.zeros(n, device="cuda", dtype=torch.float64)
    w[n_s:] = torch.randn(n_c, generator=gen, device="cuda", dtype=torch.float64)
    Au = cpm.apply(band, u, 0.5, -1.0)
    for full in (False, True):
        if full:
            w = torch.randn(n, generator=gen, device="cuda", dtype=torch.float64)
        Atw = cpm.apply_transpose(band, w, 0.5, -1.0)
        scale = (w.norm() * Au.norm()).item()
        gap = abs(torch.dot(Atw, u).item() - torch.dot(w, Au).item())
        print("adjoint gap", gap / scale, flush=True)
        assert gap <= 1e-12 * scale
    del Atw, w
    batch = cpm.Batch([band], [0.5], [-1.0])
    v = batch.apply(u.reshape(1, n))[0]
    assert (v - Au).abs().max().item() <= 1e-15 * Au.abs().max().item()
    batch.close()
    del v, Au, u
    f = torch.randn(2, n_s, generator=gen, device="cuda", dtype=torch.float64)
    g = torch.randn(2, n_c, generator=gen, device="cuda", dtype=torch.float64)
    b = cpm.rhs(band, f, g, -1.0)
    assert b.numel() > 1 << 28
    assert torch.equal(b[1], cpm.rhs(band, f[1].contiguous(), g[1].contiguous(), -1.0))
    band.close()
    del f, g, b
    torch.cuda.empty_cache()
