"""The exchange-odd part of G2 in the ladders of the general basis, where it is small.

The ladder products leave the odd part out only below the rounding of the even
part's product.  The error of a right-hand side against the CPU oracle must
therefore be that of an exchange-symmetric state: at most twice the products, and
the largest of as many rounding errors, a factor of three in all.
"""
import numpy as np
import pytest
import torch

from oracle import general as OG
from workloads import factorized_w, gue, random_g2, random_gless, rng

pytestmark = pytest.mark.gpu


def T(x):
    return torch.as_tensor(np.asarray(x), dtype=torch.complex128)


@pytest.mark.parametrize("nb", [3, 8, 17, 45])
@pytest.mark.parametrize("se", ["tpp", "tph", "dsl"])
def test_small_odd_part_costs_no_precision(lib, nb, se):
    from paper_2002_12717_amd import binding as B
    r = rng(701, nb, len(se))
    h, w, gl = gue(nb, r), factorized_w(nb, 2 * nb, r), random_gless(nb, r)
    even = random_g2(nb, r, scale=0.05, exchange=True)
    a = random_g2(nb, r, scale=0.05, exchange=False)
    odd = 0.5 * (a - a.transpose(1, 0, 3, 2))
    odd *= np.abs(even).max() / np.abs(odd).max()
    p = B.Propagator(B.GENERAL, {"tpp": B.TPP, "tph": B.TPH, "dsl": B.DSL}[se], nb, h, gl, w=w)
    err = []
    for size in (0.0, 0.9 * nb * 2.0 ** -54, 0.9 * 2.0 ** -44):
        g2 = even + size * odd
        g1d, g2d = torch.as_tensor(gl, device="cuda"), torch.as_tensor(g2, device="cuda")
        d1, d2 = torch.zeros_like(g1d), torch.zeros_like(g2d)
        p.rhs(0.0, g1d, g2d, d1, d2)
        ref = OG.rhs(T(h), T(w), T(gl), T(g2), se)[1].numpy()
        err.append(float(np.abs(d2.cpu().numpy() - ref).max() / np.abs(ref).max()))
    p.close()
    print(f"[odd part] nb={nb} {se}: errors {err[0]:.2e} {err[1]:.2e} {err[2]:.2e}", flush=True)
    assert err[1] < 3 * err[0] and err[2] < 3 * err[0]


@pytest.mark.parametrize("nb", [2, 9, 12, 43, 44])
@pytest.mark.parametrize("se", ["tpp", "dsl"])
@pytest.mark.parametrize("exchange", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_products_of_both_sectors_at_once(lib, nb, se, exchange, prec):
    """The particle-particle ladder's 32x32 tiles: one tile, tiles that hold pairs of the
    even sector only, and the largest basis of that form beside the first of the
    64x64 one.  The bounds are those of the right-hand side at other sizes."""
    from paper_2002_12717_amd import binding as B
    r = rng(702, nb, len(se))
    h, w, gl = gue(nb, r), factorized_w(nb, 6, r), random_gless(nb, r)
    g2 = random_g2(nb, r, scale=0.05, exchange=exchange)
    p = B.Propagator(B.GENERAL, {"tpp": B.TPP, "dsl": B.DSL}[se], nb, h, gl, w=w,
                     precision=B.FP64 if prec == "fp64" else B.MIXED)
    g1d, g2d = torch.as_tensor(gl, device="cuda"), torch.as_tensor(g2, device="cuda")
    d1, d2 = torch.zeros_like(g1d), torch.zeros_like(g2d)
    p.rhs(0.0, g1d, g2d, d1, d2)
    p.close()
    ref = OG.rhs(T(h), T(w), T(gl), T(g2), se)[1].numpy()
    err = float(np.abs(d2.cpu().numpy() - ref).max() / np.abs(ref).max())
    print(f"[both sectors] nb={nb} {se} exchange={exchange} {prec}: {err:.2e}", flush=True)
    assert err < (1e-12 if prec == "fp64" else 2e-5)
