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


def _rel(y, ref):
    return float((y - ref).abs().norm() / ref.abs().norm())


# Multi-right-hand-side apply on FP16 pieces: tiles T = 1..8 (full and ragged),
# right-hand sides around the column tiles, extents that leave partial 4 x 4 x 4 bricks.
# The bound is the one of the oracle comparison of these kernels (2e-6 of the same
# storage's result), here against R single applies in the same storage.
@pytest.mark.parametrize("dims,ntv,R", [((5, 3, 6, 2), 1, 1), ((4, 4, 4, 2), 4, 15),
                                        ((6, 5, 1, 3), 7, 16), ((2, 7, 3, 2), 8, 17),
                                        ((4, 1, 5, 2), 12, 33), ((3, 2, 2, 2), 15, 64),
                                        ((2, 3, 2, 2), 20, 65), ((5, 2, 2, 1), 22, 32),
                                        ((2, 2, 3, 2), 28, 31), ((2, 2, 2, 2), 32, 64)])
def test_multi_pieces_tiles(dims, ntv, R):
    import paper_2205_09104_amd as dc
    gop, oop = make_pair(dims, ntv, 3.0, mu=0.2, store=("f64", "f32", "f16s"))
    X = torch.stack([rand_vec(oop.V, oop.n, 23, r) for r in range(R)]).cuda().to(torch.complex64)
    for prec in ("f32", "f16s"):
        for adj in (False, True):
            ref = torch.stack([gop.apply(x, prec=prec, adjoint=adj) for x in X])
            try:
                for tile in (16, 32, 64):
                    dc.set_multi_tile_mode(tile)
                    y = gop.apply_multi(X, prec=prec, adjoint=adj)
                    assert _rel(y, ref) <= 2e-6, (prec, adj, tile)
            finally:
                dc.set_multi_tile_mode(0)
    gop.close()


def test_multi_pieces_range_and_nonfinite():
    """Columns and sites of very different magnitude keep their own relative
    accuracy; a non-finite entry reaches its column's neighbouring sites only."""
    import numpy as np
    gop, oop = make_pair((4, 2, 2, 2), 12, 3.0, mu=0.1, store=("f64", "f32"))
    R = 20
    X = torch.stack([rand_vec(oop.V, oop.n, 29, r) for r in range(R)]).cuda()
    colscale = torch.logspace(-25, 25, R, dtype=torch.float64, device="cuda")
    X = (X * colscale[:, None, None]).to(torch.complex64)
    y = gop.apply_multi(X, prec="f32")
    ref = gop.apply_multi(X.to(torch.complex128))
    for r in range(R):
        assert _rel(y[r].to(torch.complex128), ref[r]) <= 2e-6, r
    nb = gop.neighbours()
    for bad in (float("inf"), float("nan")):
        Z = X.clone()
        Z[7, 3, 5] = bad
        z = gop.apply_multi(Z, prec="f32")
        hit = np.zeros(oop.V, dtype=bool)
        hit[3] = True
        hit[nb[:, 3]] = True
        fin = torch.isfinite(torch.view_as_real(z)).all(-1)
        assert not bool(fin[7][torch.from_numpy(hit).cuda()].any())
        assert bool(fin[7][torch.from_numpy(~hit).cuda()].all())
        keep = [r for r in range(R) if r != 7]
        assert torch.equal(z[keep], y[keep])
    gop.close()


# Self-block inverses in registers: every grid of entries per thread (n <= 16, 32, 48, 64) and
# ragged sizes, on blocks that need their pivoting -- unitary ones with shuffled rows and
# leading zeros, condition number 1, so B^{-1} v is exact to rounding (n eps and growth: 1e-12).
@pytest.mark.parametrize("ntv", [1, 3, 8, 9, 16, 17, 24, 25, 31, 32])
def test_block_inverse_pivoting(ntv):
    import numpy as np
    from paper_2205_09104_amd import CoarseOp
    n, dims, V = 2 * ntv, (2, 2, 1, 2), 8
    rng = np.random.default_rng(ntv)
    A = np.zeros((V, n, n), dtype=np.complex128)
    for x in range(V):
        if x % 2:   # a permutation with phases: every pivot but one per column is zero
            A[x, np.arange(n), rng.permutation(n)] = np.exp(2j * np.pi * rng.random(n))
        else:       # two unitary blocks, rows shuffled
            h = max(1, n // 3)
            A[x, :h, :h] = np.linalg.qr(rng.normal(size=(h, h)) + 1j * rng.normal(size=(h, h)))[0]
            A[x, h:, h:] = np.linalg.qr(rng.normal(size=(n - h, n - h)) +
                                        1j * rng.normal(size=(n - h, n - h)))[0]
            A[x] = A[x][rng.permutation(n)]
    B = torch.zeros((V, 4, n, n), dtype=torch.complex128)
    op = CoarseOp(torch.from_numpy(A).cuda(), B.cuda(), dims, store=("f64",))
    v = rand_vec(V, n, 31, 0)
    import ctypes as C
    from paper_2205_09104_amd._lib import check, load
    out = torch.empty_like(v, device="cuda")
    vg = v.cuda()
    check(load().dc_apply_block_jacobi(op._h, C.c_void_p(vg.data_ptr()),
                                       C.c_void_p(out.data_ptr()), None))
    torch.cuda.synchronize()
    ref = np.linalg.solve(A, v.numpy()[:, :, None])[:, :, 0]
    assert _rel(out.cpu(), torch.from_numpy(ref)) <= 1e-12
    op.close()


def test_block_inverse_singular_is_refused():
    from paper_2205_09104_amd import CoarseOp, DcError
    n, V = 6, 4
    A = torch.eye(n, dtype=torch.complex128).repeat(V, 1, 1)
    A[2, :, 4] = 0
    op = CoarseOp(A.cuda(), torch.zeros((V, 4, n, n), dtype=torch.complex128).cuda(), (2, 2, 1, 1))
    x = torch.ones((V, n), dtype=torch.complex128, device="cuda")
    from paper_2205_09104_amd._lib import check, load
    import ctypes as C
    with pytest.raises(DcError):
        check(load().dc_apply_block_jacobi(op._h, C.c_void_p(x.data_ptr()),
                                           C.c_void_p(torch.empty_like(x).data_ptr()), None))
    op.close()


# Gram-Schmidt steps: bases through 1, 2, 4, 8, 16, 32, 48, 64 and beyond 64 vectors, and
# vectors of less than two tiles (odd length), of one tile per workgroup, and of several
# (partials summed by the next kernel or by a launch of their own).  The bound is the one
# of the other Hessenberg comparison; the oracle's own H moves by less than 1e-12 of its
# largest entry under a start vector perturbed by 1e-13.  Single-sync: that process's
# bound, over the steps where one pass keeps the basis orthogonal.
@pytest.mark.parametrize("dims,ntv,steps,ortho,tol", [
    ((3, 2, 2, 2), 2, 30, 0, 1e-10), ((4, 4, 4, 4), 9, 70, 0, 1e-10),
    ((8, 6, 6, 6), 10, 40, 0, 1e-10), ((3, 2, 2, 2), 2, 12, 1, 1e-9),
    ((4, 4, 4, 4), 9, 12, 1, 1e-9), ((8, 6, 6, 6), 10, 18, 1, 1e-9)])
def test_gram_schmidt_steps(dims, ntv, steps, ortho, tol):
    from oracle import operator as dop
    from oracle.krylov import arnoldi
    from paper_2205_09104_amd import Opts
    gop, oop = make_pair(dims, ntv, 3.0, mu=0.1)
    v = rand_vec(oop.V, oop.n, 80)
    ref = arnoldi(lambda u: dop.apply(oop, u.reshape(oop.V, oop.n)).reshape(-1),
                  v.numpy().reshape(-1), steps, "mgs").Hbar
    for _ in range(2):
        H, s = gop.arnoldi(v.cuda(), steps, Opts(m=steps, ortho=ortho))
        assert s == steps
        err = float(abs(H - ref).max() / abs(ref).max())
        log(f"  gram-schmidt {dims} n {oop.n} steps {steps} ortho {ortho}: {err:.1e}")
        assert err <= tol
    gop.close()


# The same steps on FP32 vectors, with a recycle space before the basis: mixed solves
# whose cycles pass 64 vectors, to the tolerance on the FP64 true residual.
@pytest.mark.parametrize("ortho", [0, 1])
def test_gram_schmidt_fp32_recycled(ortho):
    from paper_2205_09104_amd import Opts
    from .helpers import oracle_relres
    gop, oop = make_pair((4, 4, 4, 4), 5, 3.0, mu=0.1, store=("f64", "f32", "f16s"))
    o = Opts(m=80, k=8, d=4, prec="f32", outer=1, inner_tol=1e-5, seed=1, ortho=ortho)
    for r in range(2):
        b = rand_vec(oop.V, oop.n, 81, r)
        x, st, rc = gop.solve(b.cuda(), 1e-10, o)
        assert rc == 0 and st[0]["rel_res_true"] <= 1e-10, st
        assert oracle_relres(oop, x.cpu().numpy(), b.numpy()) <= 1e-10
    gop.close()


# The full-lattice apply's routes, forward and adjoint, in every precision: one launch up
# to 32 MB of blocks and two beyond (full and ragged tiles just on either side; FP64 tiles
# of n > 40 always two), non-temporal block loads beyond 256 MB, a degenerate extent.
# Bounds: those of the other apply comparisons with the oracle.
@pytest.mark.parametrize("dims,ntv", [((4, 4, 4, 4), 20), ((4, 4, 4, 4), 21),
                                      ((5, 4, 4, 3), 22), ((6, 5, 6, 6), 8), ((8, 7, 5, 6), 9),
                                      ((9, 7, 5, 11), 13), ((1, 7, 8, 8), 16),
                                      ((6, 5, 4, 8), 31)])
@pytest.mark.parametrize("mu", [0.0, 0.21])
def test_apply_routes(dims, ntv, mu):
    from oracle import mixed
    from oracle import operator as dop
    from .helpers import rel
    small = dims[0] * dims[1] * dims[2] * dims[3] * 20 * ntv * ntv * 16 < 64 << 20
    gop, oop = make_pair(dims, ntv, 2.5, mu=mu, store=("f64", "f32", "f16s"))
    x = rand_vec(oop.V, oop.n, 7)
    xg, x = x.cuda(), x.numpy()
    refa = dop.apply_adjoint(oop, x)
    assert rel(gop.apply(xg).cpu().numpy(), dop.apply(oop, x)) <= 1e-13
    assert rel(gop.apply(xg, adjoint=True).cpu().numpy(), refa) <= 1e-13
    x32 = xg.to(torch.complex64)
    for prec in ("f32", "f16s"):
        if small:   # the oracle's rounded blocks of larger operators take minutes
            lo = mixed.lowprec_apply(oop, prec)(x)
            assert rel(gop.apply(x32, prec=prec).cpu().numpy(), lo) <= 2e-6, prec
        assert rel(gop.apply(x32, prec=prec, adjoint=True).cpu().numpy(), refa) <= (
            2e-6 if prec == "f32" else 3e-3), prec
    gop.close()


# Multi-right-hand-side apply in FP64: tiles T = 1..8 (odd ones lack the second unit row of
# their last tile; at T = 1 that is the whole tile but one), full and ragged, uneven step
# counts per wave, both right-hand-side tiles.  The bound is that of the oracle comparison
# of this kernel; a tile changes no bit of the result.
@pytest.mark.parametrize("dims,ntv,R", [((5, 3, 2, 2), 1, 1), ((4, 2, 2, 2), 4, 5),
                                        ((3, 2, 2, 3), 8, 16), ((2, 3, 2, 2), 11, 17),
                                        ((2, 2, 3, 2), 12, 15), ((4, 2, 1, 2), 16, 33),
                                        ((2, 2, 2, 2), 19, 12), ((2, 2, 2, 2), 20, 40),
                                        ((2, 2, 2, 1), 27, 31), ((2, 1, 2, 2), 28, 16),
                                        ((2, 2, 1, 2), 31, 20)])
def test_multi_f64_tiles(dims, ntv, R):
    import paper_2205_09104_amd as dc
    gop, oop = make_pair(dims, ntv, 3.0, mu=0.2)
    X = torch.stack([rand_vec(oop.V, oop.n, 37, r) for r in range(R)]).cuda()
    for adj in (False, True):
        ref = torch.stack([gop.apply(x, adjoint=adj) for x in X])
        out = []
        try:
            for tile in (16, 32):
                dc.set_multi_tile_mode(tile)
                out.append(gop.apply_multi(X, adjoint=adj))
        finally:
            dc.set_multi_tile_mode(0)
        log(f"  multi f64 {dims} n {oop.n} R {R} adjoint {adj}: {_rel(out[0], ref):.1e}")
        assert _rel(out[0], ref) <= 1e-13 and torch.equal(out[0], out[1])
    gop.close()


# Multi-right-hand-side apply of FP32 vectors on operands whose entries are not of one size:
# blocks with graded rows, with graded columns and the vectors graded the other way, block
# diagonal with vectors graded over its parts, near-equal operands whose piece errors add
# up, and magnitudes towards both ends of FP32.  All inputs are stored exactly in every
# precision tested, so the reference is 64-bit arithmetic on the same numbers, and the error
# of every single entry is held against the sum of the magnitudes that enter it: 2e-6 of it,
# the normwise bound of the oracle comparison (each product is held to one FP32 rounding,
# 6e-8, and a few dozen rounded sums follow).
def _graded(kind, prec, V, n, R, rng):
    import numpy as np

    def mantissa(*shape):   # 9 significant bits: an FP16 code, also times 2^-13
        def real():
            return rng.integers(256, 513, shape) / 512.0 * rng.choice([-1.0, 1.0], shape)
        return real() + 1j * real()

    def full(*shape):
        return (rng.normal(size=shape) + 1j * rng.normal(size=shape)).astype(np.complex64).astype(
            np.complex128)

    e = np.arange(n) / (n - 1)
    half = prec == "f16s"
    M = mantissa(V, 5, n, n) if half else full(V, 5, n, n)
    X = full(R, V, n)

    def pow2(t):
        return 2.0 ** np.round(t)

    deep = 13 if half else 40   # FP16 codes hold a block's entries over 2^14
    if kind == "rows":
        M *= pow2(-deep * e)[:, None]   # self blocks only: a hop also acts transposed
        M[:, 1:] = 0
    elif kind == "columns":
        M *= pow2(-deep * e)[None, :]
        X *= pow2(deep * e)
    elif kind == "parts":
        M[..., : n // 2, n // 2:] = 0
        M[..., n // 2:, : n // 2] = 0
        X[..., n // 2:] *= 2.0 ** -40
    elif kind == "near one":
        M[:] = 1 + 2.0 ** -(9 if half else 11)
        X = np.full((R, V, n), 1 + 2.0 ** -11 + 2.0 ** -23 + 0j)
    else:
        block, vec = kind
        M *= 2.0 ** block
        X *= (2.0 ** np.linspace(vec - 8, vec, R).round())[:, None, None]
    if half and not isinstance(kind, tuple) and kind != "near one":
        M[:, :1 if kind == "rows" else 5, 0, 0] = 1 + 0.5j   # the block's scale: a power of two, so codes are exact
    elif half and isinstance(kind, tuple):
        M[..., 0, 0] = 2.0 ** kind[0]
    elif half:
        M[..., 0, 0] = 2.0
    return M, X.astype(np.complex64).astype(np.complex128)


@pytest.mark.parametrize("prec", ["f32", "f16s"])
@pytest.mark.parametrize("kind", ["rows", "columns", "parts", "near one", (-8, 122), (-30, 124),
                                  (70, 40), (110, -110), (-110, 110), (-100, 30), (20, -118)])
@pytest.mark.parametrize("dims,ntv,R", [((3, 2, 2, 2), 3, 5), ((2, 3, 2, 1), 24, 40)])
def test_multi_graded_operands(prec, kind, dims, ntv, R):
    import numpy as np
    import paper_2205_09104_amd as dc
    from paper_2205_09104_amd import CoarseOp
    V, n = dims[0] * dims[1] * dims[2] * dims[3], 2 * ntv
    M, X = _graded(kind, prec, V, n, R, np.random.default_rng(ntv))
    op = CoarseOp(torch.from_numpy(M[:, 0].copy()).cuda(), torch.from_numpy(M[:, 1:].copy()).cuda(),
                  dims, store=("f64", prec))
    nb = op.neighbours()
    g = np.where(np.arange(n) < ntv, 1.0, -1.0)
    for adj in (False, True):   # without a mass term D^H = Gamma5 D Gamma5
        v = X * g if adj else X
        ref = np.einsum("xij,rxj->rxi", M[:, 0], v)
        mag = np.einsum("xij,rxj->rxi", abs(M[:, 0]), abs(v))
        for mu in range(4):
            f, b = nb[mu], nb[4 + mu]
            ref += np.einsum("xij,rxj->rxi", M[:, 1 + mu], v[:, f])
            mag += np.einsum("xij,rxj->rxi", abs(M[:, 1 + mu]), abs(v[:, f]))
            ref += g * np.einsum("xji,rxj->rxi", M[b, 1 + mu].conj(), v[:, b] * g)
            mag += np.einsum("xji,rxj->rxi", abs(M[b, 1 + mu]), abs(v[:, b]))
        if adj:
            ref = ref * g
        # entries whose terms leave FP32's normal range in the sum are not compared
        top, low = np.finfo(np.float32).max / 2, np.finfo(np.float32).tiny * 2.0 ** 24
        use = (mag < top) & (mag > low)
        assert use.any()
        single = torch.stack([op.apply(torch.from_numpy(x.astype(np.complex64)).cuda(), prec=prec,
                                       adjoint=adj) for x in X]).cpu().numpy()
        es = np.max(np.where(use, abs(single - ref) / mag, 0))
        for tile in (16, 32, 64):
            try:
                dc.set_multi_tile_mode(tile)
                y = op.apply_multi(torch.from_numpy(X.astype(np.complex64)).cuda(), prec=prec,
                                   adjoint=adj).cpu().numpy()
            finally:
                dc.set_multi_tile_mode(0)
            err = np.where(use, abs(y - ref) / mag, 0)
            log(f"  graded {kind} {prec} n {n} R {R} adjoint {adj} tile {tile}: "
                f"{np.max(err):.1e} (single applies {es:.1e})")
            assert np.max(err) <= 2e-6
    op.close()


# The multi-apply uses what the layout of the blocks recorded (largest entries, FP16
# scales): after an update to blocks of very different size it must use the new ones.
# Bound of the other comparisons with R single applies in the same storage.
@pytest.mark.parametrize("factor", [1e4, 2.0 ** 80, 2.0 ** -90])
def test_multi_after_update(factor):
    from paper_2205_09104_amd import CoarseOp
    import synth
    dims, ntv, R = (3, 2, 4, 2), 6, 18
    A, B = synth.self_blocks(dims, ntv, 3.0, 0).cuda(), synth.hop_blocks(dims, ntv, 0).cuda()
    op = CoarseOp(A, B, dims, store=("f64", "f32", "f16s"))
    V, n = A.shape[0], 2 * ntv
    X = torch.stack([rand_vec(V, n, 41, r) for r in range(R)]).cuda().to(torch.complex64)
    for _ in range(2):
        for prec in ("f32", "f16s"):
            ref = torch.stack([op.apply(x, prec=prec) for x in X])
            y = op.apply_multi(X, prec=prec)
            rel = float((y - ref).abs().to(torch.float64).div(ref.abs().max()).norm() /
                        ref.abs().to(torch.float64).div(ref.abs().max()).norm())
            assert rel <= 2e-6, (prec, factor, rel)
        op.update(A * factor, B * factor)
    op.close()


# An Arnoldi step into a nearly invariant space: three eigenvalues and hops of size eps, so
# the fourth vector's norm before scaling is rounding-sized against ||A v_j|| while the
# breakdown threshold (1e-14, FP32 1e-6) is not reached; with no hops the space is invariant
# and the process ends at three steps.  h_{43} against Arnoldi in extended precision; bound:
# 50 units of rounding of ||A|| (64 entries, two passes over three vectors) over h.
@pytest.mark.parametrize("prec,eps", [("f64", 1e-5), ("f64", 1e-9), ("f64", 1e-11),
                                      ("f32", 1e-2), ("f32", 1e-3)])
def test_arnoldi_nearly_invariant(prec, eps):
    import numpy as np
    from oracle import operator as dop
    from paper_2205_09104_amd import CoarseOp, Opts
    import synth
    dims, ntv = (2, 2, 2, 2), 2
    n, V = 4, 16
    A = torch.zeros((V, n, n), dtype=torch.complex128)
    for x in range(V):
        for i in range(n):
            A[x, i, i] = (1.0, 2.0, 4.0)[(x + i) % 3]
    B = (synth.hop_blocks(dims, ntv, 0) * eps).to(torch.complex64).to(torch.complex128)
    v = rand_vec(V, n, 43, 0).to(torch.complex64).to(torch.complex128)
    for hops in (B, torch.zeros_like(B)):
        op = CoarseOp(A.cuda(), hops.cuda(), dims, store=("f64", "f32"))
        H, s = op.arnoldi(v.cuda(), 6, Opts(m=6, prec=prec))
        op.close()
        if hops is not B:
            assert s == 3
            continue
        oop = dop.build(dims, A.numpy(), B.numpy(), 0.0)
        D = np.stack([dop.apply(oop, e.reshape(V, n)).reshape(-1)
                      for e in np.eye(V * n, dtype=np.complex128)], axis=1).astype(np.clongdouble)
        q = [v.numpy().reshape(-1).astype(np.clongdouble)]
        q[0] = q[0] / np.sqrt((abs(q[0]) ** 2).sum())
        for j in range(3):
            w = D @ q[j]
            for _ in range(3):
                for u in q:
                    w = w - u * (u.conj() * w).sum()
            h = np.sqrt((abs(w) ** 2).sum())
            q.append(w / h)
        unit = 2.0 ** (-52 if prec == "f64" else -23)
        err = abs(float(H[3, 2].real) / float(h) - 1)
        log(f"  nearly invariant {prec} eps {eps}: h {float(h):.3e}, relative error {err:.1e}")
        assert s >= 4 and err <= 50 * unit * 4 / float(h)


# The profile's kernel 0: a small operator's apply is one launch, which reads the input
# and writes the output; a larger one's block kernel reads the input.
def test_profile_passes_of_the_full_apply():
    for dims, ntv, passes in (((4, 4, 4, 4), 8, 2), ((4, 4, 4, 4), 24, 1)):
        gop, oop = make_pair(dims, ntv, 3.0)
        x = rand_vec(oop.V, oop.n, 3, 0).cuda()
        gop.profile_apply(1)
        for adj in (False, True):
            gop.apply(x, adjoint=adj)
        assert gop.profile_apply_read("f64")[0] == 2
        assert gop.profile_apply_passes("f64") == 2 * passes
        gop.close()


# Single-read form around the size from which its tiles are loaded non-temporally (288 MB
# of blocks), full and ragged tiles: bit for bit the two-kernel form, forward, adjoint and
# with block Jacobi.
@pytest.mark.parametrize("dims,ntv,prec", [((4, 8, 6, 6), 24, "f64"), ((8, 8, 6, 6), 24, "f64"),
                                           ((8, 8, 6, 6), 21, "f64"), ((8, 8, 6, 6), 24, "f32"),
                                           ((8, 8, 8, 8), 24, "f32"), ((8, 8, 8, 8), 21, "f32")])
def test_single_read_around_the_cache_size(dims, ntv, prec):
    import paper_2205_09104_amd as dc
    from paper_2205_09104_amd import CoarseOp
    V, n = dims[0] * dims[1] * dims[2] * dims[3], 2 * ntv
    g = torch.Generator(device="cuda").manual_seed(5)

    def rand(*shape):
        return torch.randn(*shape, dtype=torch.complex128, device="cuda", generator=g)

    A = rand(V, n, n) * 0.3 / n ** 0.5 + 4.0 * torch.eye(n, dtype=torch.complex128, device="cuda")
    op = CoarseOp(A, rand(V, 4, n, n) / n ** 0.5, dims, mu=0.1, store=("f64", prec))
    del A
    x = rand(V // 2, n).to(torch.complex128 if prec == "f64" else torch.complex64)
    for kw in (dict(), dict(adjoint=True), dict(block_jacobi=True)):
        try:
            dc.set_reduced_kernels(1)
            a = op.apply_reduced(x, prec=prec, **kw)
        finally:
            dc.set_reduced_kernels(0)
        op.profile_apply(1)
        b = op.apply_reduced(x, prec=prec, **kw)
        assert op.profile_apply_passes(prec, 1) == 9
        op.profile_apply(0)
        assert torch.equal(a, b) and bool(torch.isfinite(b.abs()).all())
    op.close()


# Which operators' full apply is one launch (two vector passes in the profile, one with
# two launches): up to 4,096 sites, beyond which its workgroups cost more than the second
# launch, and up to 32 MB of blocks as they are stored, padded to whole tiles.
@pytest.mark.parametrize("dims,ntv,prec,passes", [
    ((8, 8, 8, 8), 3, "f64", 2), ((8, 8, 13, 5), 3, "f64", 1), ((8, 8, 13, 5), 3, "f16s", 1),
    ((9, 7, 5, 13), 3, "f32", 2), ((16, 8, 8, 8), 1, "f32", 1), ((8, 8, 8, 4), 5, "f64", 1),
    ((8, 8, 8, 3), 5, "f64", 2), ((8, 8, 8, 4), 8, "f32", 2), ((8, 8, 8, 7), 8, "f32", 1)])
def test_one_launch_apply_range(dims, ntv, prec, passes):
    from paper_2205_09104_amd import CoarseOp
    V, n = dims[0] * dims[1] * dims[2] * dims[3], 2 * ntv
    g = torch.Generator(device="cuda").manual_seed(5)
    A = torch.randn(V, n, n, dtype=torch.complex128, device="cuda", generator=g)
    B = torch.randn(V, 4, n, n, dtype=torch.complex128, device="cuda", generator=g)
    op = CoarseOp(A, B, dims, store=("f64", prec))
    x = torch.randn(V, n, dtype=torch.complex128, device="cuda", generator=g)
    y = op.apply(x)
    op.profile_apply(1)
    z = op.apply(x if prec == "f64" else x.to(torch.complex64), prec=prec)
    assert op.profile_apply_read(prec)[0] == 1 and op.profile_apply_passes(prec) == passes
    assert _rel(z.to(torch.complex128), y) <= {"f64": 0.0, "f32": 2e-6, "f16s": 3e-3}[prec]
    op.close()


# The hop gradient's thread mapping: one row and many rows per pass, threads past the rows
# (n < 16), rows that do not divide n, the largest n, extents of one site.  Two or four
# products per entry: rounding only, 1e-14 of the largest.
@pytest.mark.parametrize("dims,ntv", [((3, 2, 1, 2), 1), ((2, 3, 2, 2), 3), ((2, 2, 2, 2), 7),
                                      ((2, 1, 3, 2), 8), ((2, 2, 2, 1), 9), ((1, 2, 2, 2), 16),
                                      ((2, 2, 1, 2), 21), ((2, 2, 2, 1), 32)])
def test_grad_hops_thread_mapping(dims, ntv):
    gop, oop = make_pair(dims, ntv, 3.0)
    V, n = oop.V, oop.n
    lam, x = rand_vec(V, n, 61, 0).cuda(), rand_vec(V, n, 61, 1).cuda()
    nb = torch.from_numpy(gop.neighbours()).long().cuda()
    g5 = torch.where(torch.arange(n, device="cuda") < ntv, 1.0, -1.0).to(torch.complex128)
    for tied in (True, False):
        out = gop.grad_hops(lam, x, tied=tied)
        for d in range(4 if tied else 8):
            y = nb[d]
            ref = -lam[:, :, None] * x[y].conj()[:, None, :]
            if tied:
                ref = ref - (g5 * x)[:, :, None] * (lam[y].conj() * g5)[:, None, :]
            assert float((out[:, d] - ref).abs().max()) <= 1e-14 * float(ref.abs().max())
    gop.close()


# Blocks with entries beyond FP32, infinite or NaN in reduced storage: the multi-apply is
# finite where the single apply is, and nowhere else.
@pytest.mark.parametrize("prec", ["f32", "f16s"])
@pytest.mark.parametrize("bad", [1e39, float("inf"), float("nan")])
def test_multi_nonfinite_blocks(prec, bad):
    from paper_2205_09104_amd import CoarseOp
    import synth
    dims, ntv, R = (4, 3, 2, 2), 5, 9
    A, B = synth.self_blocks(dims, ntv, 3.0, 0), synth.hop_blocks(dims, ntv, 0)
    A[7, 3, 2] = bad
    B[20, 1, 4, 4] = bad
    op = CoarseOp(A.cuda(), B.cuda(), dims, store=("f64", prec))
    V, n = A.shape[0], 2 * ntv
    X = torch.stack([rand_vec(V, n, 47, r) for r in range(R)]).cuda().to(torch.complex64)
    ref = torch.stack([op.apply(x, prec=prec) for x in X])
    y = op.apply_multi(X, prec=prec)
    want = torch.isfinite(torch.view_as_real(ref)).all(-1)
    have = torch.isfinite(torch.view_as_real(y)).all(-1)
    assert not bool(want[:, 7, 3].any())                 # the row of the bad entry
    assert torch.equal(want.all(-1), have.all(-1))       # the same sites
    assert not bool((have & ~want).any())                # no entry turned finite
    keep = want.all(-1)
    assert float((y[keep] - ref[keep]).abs().max()) <= 2e-6 * float(ref[keep].abs().max())
    op.close()
