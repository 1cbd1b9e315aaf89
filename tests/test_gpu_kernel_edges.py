"""Kernel variants at the sizes where their dispatch or their tiles change:
edges of tiles, remainders, the smallest and largest of a range."""
import pytest
import torch

from .helpers import log, make_pair, rand_vec

pytestmark = pytest.mark.gpu


# Block sizes that are not multiples of 8 (ragged tiles) in every precision, and FP64
# operators just above the size from which they take the single-read form (24 MB of
# blocks): n = 48 (largest FP64 tile), 42 (ragged), 32.  The forms add the same terms in
# the same order: equal bit for bit.
@pytest.mark.parametrize("dims,ntv,mu,precs", [
    ((2, 2, 2, 2), 1, 0.1, ("f32", "f16s")), ((4, 2, 2, 4), 5, 0.2, ("f32", "f16s")),
    ((2, 4, 2, 2), 23, 0.0, ("f32", "f16s")), ((4, 2, 2, 2), 31, 0.1, ("f32", "f16s")),
    ((4, 4, 4, 4), 24, 0.1, ("f64",)), ((4, 4, 4, 4), 21, 0.0, ("f64",)),
    ((6, 4, 4, 4), 16, 0.2, ("f64",)), ((16, 2, 8, 4), 9, 0.1, ("f64",))])
def test_single_read_ragged_and_f64(dims, ntv, mu, precs):
    import paper_2205_09104_amd as dc
    gop, oop = make_pair(dims, ntv, 3.0, mu=mu, store=("f64", "f32", "f16s"))
    ne = oop.V // 2
    for prec in precs:
        x = rand_vec(ne, oop.n, 17, 0).cuda()
        x = x if prec == "f64" else x.to(torch.complex64)
        for kw in (dict(), dict(adjoint=True), dict(block_jacobi=True)):
            try:
                dc.set_reduced_kernels(1)
                a = gop.apply_reduced(x, prec=prec, **kw)
                dc.set_reduced_kernels(0)
                gop.profile_apply(1)
                b = gop.apply_reduced(x, prec=prec, **kw)
            finally:
                dc.set_reduced_kernels(0)
            # the single-read form ran: x_e plus eight partial vectors
            assert gop.profile_apply_passes(prec, 1) == 9
            gop.profile_apply(0)
            log(f"  {dims} n {oop.n} {prec} {kw}: max |difference| {float((a - b).abs().max()):.1e}")
            assert torch.equal(a, b) and bool(torch.isfinite(b.abs()).all())
    gop.close()
