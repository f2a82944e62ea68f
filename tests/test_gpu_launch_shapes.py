"""The launch shapes that a rule on sizes chooses: on both sides of each rule's
line the results match the oracle and do not depend on the grouping of the
right-hand sides (byte for byte).  (GPU)"""
import numpy as np
import pytest
import torch

import oracle
from oracle import evenodd, sap as osap
from paper_2407_00041_amd import DiracOp, clover_term, synth, tune_get, tune_set

from util import TOL, need_gpu, rel_l2

pytestmark = pytest.mark.gpu


# 16^4: one right-hand side per lane up to 4, pairs and a lone last one at 5; 24 x 16^2 x 24 is past 2^17 sites
# (the FP64 column walk, chunks of four slices) and a pair there past 2^18 site-right-hand-sides; 10 x 32^2 x 14
# ends in a half chunk of the column walk
@pytest.mark.parametrize("dims,n", [((16, 16, 16, 16), 3), ((16, 16, 16, 16), 5), ((24, 16, 16, 24), 3),
                                    ((10, 32, 32, 14), 2)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("compress,ap", [(True, False), (False, True)])
def test_reduced_operator_shapes(dims, n, prec, compress, ap):
    need_gpu()
    U = synth.smooth_links(dims, 71, device="cuda").cpu().numpy()
    op = DiracOp(dims, U, -0.3, 1.0, antiperiodic_t=ap, even_odd=True, compress_links=compress,
                 compress_clover=compress)
    psi = synth.gaussian_spinor(dims, 72, nrhs=n, device="cuda")
    e, o = op.split(op.pack(psi, prec), prec, n)
    out, tmp = op.empty_parity(prec, n), op.empty_parity(prec, n)
    rb = op.parity_field_bytes(prec, 1)
    for dagger in (False, True):
        op.apply_schur_native(out, e, tmp, n, prec, dagger)
        for r in range(n):
            o1, t1 = op.empty_parity(prec, 1), op.empty_parity(prec, 1)
            op.apply_schur_native(o1, e[r * rb:(r + 1) * rb], t1, 1, prec, dagger)
            assert torch.equal(o1, out[r * rb:(r + 1) * rb]), (dagger, r)
    op.apply_schur_native(out, e, tmp, n, prec)
    even_sites = evenodd.sites_of(dims, 0)
    pick = np.sort(np.random.default_rng(73).choice(len(even_sites), 48, replace=False))
    o.zero_()
    got = op.unpack(op.merge(out, o, prec, n), prec, n)[:, torch.from_numpy(even_sites[pick]).cuda()].cpu().numpy()
    for r in range(n):
        want = evenodd.schur_sites(dims, U, psi[r].cpu().numpy()[even_sites], even_sites[pick], -0.3, 1.0,
                                   antiperiodic_t=ap)
        assert rel_l2(got[r], want) < TOL[prec], r


# slices of less than 256 half-lattice sites, dealt in slabs of several: a shorter last slab (34 x 4^3 in slabs of 12,
# 22 x 4 x 6 x 8 of 5), one slab for all, and 6 x 8^3 (256), dealt by slices
@pytest.mark.parametrize("dims,n", [((34, 4, 4, 4), 3), ((22, 4, 6, 8), 2), ((70, 2, 2, 2), 1), ((6, 8, 8, 8), 1)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("compress,ap", [(True, False), (False, True)])
def test_reduced_operator_slabs(dims, n, prec, compress, ap):
    test_reduced_operator_shapes(dims, n, prec, compress, ap)


# odd counts in pairs: the last right-hand side in the pairs' launch, and after a full launch of sixteen
@pytest.mark.parametrize("dims,n", [((16, 16, 16, 16), 17), ((16, 16, 16, 34), 3)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("compress,ap", [(True, False), (False, True)])
def test_reduced_operator_odd_counts(dims, n, prec, compress, ap):
    test_reduced_operator_shapes(dims, n, prec, compress, ap)


# FP64 below 2^17 sites: columns where the pairs' waves fill whole rounds (16^4 of eight, 16 x 12 x 24^2 of three), the
# same bits as the site kernel of a single right-hand side
@pytest.mark.parametrize("dims,n", [((16, 16, 16, 16), 8), ((16, 12, 24, 24), 3)])
@pytest.mark.parametrize("compress,ap", [(True, False), (False, True)])
def test_reduced_operator_rounds(dims, n, compress, ap):
    test_reduced_operator_shapes(dims, n, "f64", compress, ap)


# applies neither tuned nor set. The small-lattice kernel (V n up to 2^14 at FP64, 2^15 else): ragged tiles at
# 3 x 5 x 7 x 9, extents of two, 8^4 with 4 and 8 on the two lines and 5 and 9 past them. 12^4: one right-hand side
# per lane up to 6, pairs at 7 (past 2^17 site-right-hand-sides). 16^4: pairs, at FP32 with two-row links
# link-stationary from 6. 24 x 16^2 x 24: FP64 columns. 32 x 16^2 x 32: FP32 columns too, in pairs with a lone last
# one. Odd extents.
@pytest.mark.parametrize("dims,n", [((3, 5, 7, 9), 2), ((2, 2, 2, 2), 1), ((8, 8, 8, 8), 4), ((8, 8, 8, 8), 5),
                                    ((8, 8, 8, 8), 8), ((8, 8, 8, 8), 9), ((12, 12, 12, 12), 6),
                                    ((12, 12, 12, 12), 7), ((16, 16, 16, 16), 3), ((16, 16, 16, 16), 6),
                                    ((24, 16, 16, 24), 2), ((32, 16, 16, 32), 3), ((17, 19, 21, 23), 1)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("compress,ap,dagger", [(True, False, False), (False, True, True)])
def test_untuned_apply_shapes(dims, n, prec, compress, ap, dagger):
    need_gpu()
    U = synth.smooth_links(dims, 81, device="cuda").cpu().numpy()
    op = DiracOp(dims, U, -0.3, 1.0, antiperiodic_t=ap, compress_links=compress, compress_clover=compress)
    psi = synth.gaussian_spinor(dims, 82, nrhs=n, device="cuda")
    x = op.pack(psi, prec)
    out, one = op.empty(prec, n).zero_(), op.empty(prec, 1).zero_()  # a field's padding bytes stay as they are
    op.apply_native(out, x, n, prec, dagger)
    rb = op.field_bytes(prec, 1)
    for r in range(n):
        op.apply_native(one, x[r * rb:(r + 1) * rb], 1, prec, dagger)
        assert torch.equal(one, out[r * rb:(r + 1) * rb]), r
    sites = synth.random_sites(dims, 64, 83)
    got = op.unpack(out, prec, n)[:, torch.from_numpy(sites).cuda()].cpu().numpy()
    for r in range(n):
        want = oracle.dirac_apply_sites(dims, U, psi[r].cpu().numpy(), sites, -0.3, 1.0, antiperiodic_t=ap,
                                        dagger=dagger)
        assert rel_l2(got[r], want) < TOL[prec], r


# thin lattices: T-slices dealt in slabs (130 x 4^3 in slabs of eight, the last one shorter; 600 x 2^3; 90 x 5 x 6 x 7 by
# slices of 210 in slabs of two), z-planes too few for the link-stationary kernel (64 x 4 x 16^2, FP32 of six), slices
# too small for pairs of FP64 columns (512 x 8^3 of eight)
@pytest.mark.parametrize("dims,n", [((130, 4, 4, 4), 5), ((600, 2, 2, 2), 8), ((90, 5, 6, 7), 3), ((64, 4, 16, 16), 6),
                                    ((512, 8, 8, 8), 8)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("compress,ap,dagger", [(True, False, False), (False, True, True)])
def test_untuned_apply_thin(dims, n, prec, compress, ap, dagger):
    need_gpu()
    U = synth.smooth_links(dims, 86, device="cuda").cpu().numpy()
    op = DiracOp(dims, U, -0.3, 1.0, antiperiodic_t=ap, compress_links=compress, compress_clover=compress)
    psi = synth.gaussian_spinor(dims, 87, nrhs=n, device="cuda")
    x = op.pack(psi, prec)
    out, one = op.empty(prec, n).zero_(), op.empty(prec, 1).zero_()
    op.apply_native(out, x, n, prec, dagger)
    op.apply_native(one, x[-op.field_bytes(prec, 1):], 1, prec, dagger)
    assert torch.equal(one, out[-op.field_bytes(prec, 1):])
    sites = synth.random_sites(dims, 64, 88)
    got = op.unpack(out, prec, n)[:, torch.from_numpy(sites).cuda()].cpu().numpy()
    for r in range(n):
        want = oracle.dirac_apply_sites(dims, U, psi[r].cpu().numpy(), sites, -0.3, 1.0, antiperiodic_t=ap,
                                        dagger=dagger)
        assert rel_l2(got[r], want) < TOL[prec], r


# counts that the register block does not divide, knobs set: the rest in the whole blocks' launch (9 in pairs; 5, 6, 7 in
# fours), alone (3 in fours) and after a full table of 24 blocks (49 in pairs, 99 in fours); and more right-hand sides
# than a table of the small-lattice kernel (26, neither tuned nor set)
@pytest.mark.parametrize("order,nr,n", [(2, 2, 9), (3, 2, 9), (2, 2, 49), (3, 2, 49), (2, 4, 3), (2, 4, 5), (2, 4, 6),
                                        (2, 4, 7), (6, 4, 7), (2, 4, 99), (None, 1, 26)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16s"])
@pytest.mark.parametrize("compress", [True, False])
def test_register_block_rests(order, nr, n, prec, compress):
    need_gpu()
    dims = (4, 6, 2, 6)
    U = synth.smooth_links(dims, 84).numpy()
    op = DiracOp(dims, U, -0.3, 1.0, antiperiodic_t=True, compress_links=compress, compress_clover=compress)
    psi = synth.gaussian_spinor(dims, 85, nrhs=n)
    x = op.pack(torch.from_numpy(psi).cuda(), prec)
    out, one = op.empty(prec, n).zero_(), op.empty(prec, 1).zero_()
    saved = {k: tune_get(k) for k in ("order", "nr_" + prec, "explicit")}
    try:
        if order is not None:
            tune_set("order", order)
            tune_set("nr_" + prec, nr)
        op.apply_native(out, x, n, prec)
        rb = op.field_bytes(prec, 1)
        for r in range(n):
            op.apply_native(one, x[r * rb:(r + 1) * rb], 1, prec)
            assert torch.equal(one, out[r * rb:(r + 1) * rb]), r
    finally:
        for k, v in saved.items():
            tune_set(k, v)
    got = op.unpack(out, prec, n).cpu().numpy()
    want = oracle.dirac_apply(dims, U, psi, -0.3, 1.0, antiperiodic_t=True)
    for r in range(n):
        assert rel_l2(got[r], want[r]) < TOL[prec], r


# 64-site tiles over eighths of a T-slice: ragged eighths, a slice below one tile, extents of two, whole tiles
@pytest.mark.parametrize("dims", [(5, 7, 9, 11), (3, 2, 5, 2), (2, 2, 2, 2), (4, 8, 8, 16), (2, 16, 16, 16)])
def test_clover_term_tiles(dims):
    need_gpu()
    U = synth.smooth_links(dims, 91, device="cuda")
    got = clover_term(dims, U).cpu().numpy()
    want = oracle.clover_term(dims, U.cpu().numpy())
    assert rel_l2(got, want) < TOL["f64"]


# slices below 512 sites, dealt in slabs of several: a shorter last slab (17 x 4^3 in one slab, 130 x 4^3 in three of
# 44, 600 x 2^3 in two), slices that are no multiple of a tile, and 8^3 (512 sites), dealt by slices
@pytest.mark.parametrize("dims", [(17, 4, 4, 4), (130, 4, 4, 4), (600, 2, 2, 2), (11, 5, 7, 9), (14, 7, 9, 8),
                                  (9, 8, 8, 8)])
def test_clover_term_slabs(dims):
    need_gpu()
    U = synth.smooth_links(dims, 92, device="cuda")
    got = clover_term(dims, U).cpu().numpy()
    want = oracle.clover_term(dims, U.cpu().numpy())
    assert rel_l2(got, want) < TOL["f64"]


# Schwarz blocks whose residual takes its own sites from LDS and the rest from faces: extents of one (a site leaves
# the block both ways; with T also across the antiperiodic boundary), three-site blocks, block counts that are no
# multiple of eight, a block that spans directions, 256 sites
@pytest.mark.parametrize("dims,block,additive", [
    ((4, 4, 6, 8), (1, 2, 3, 2), False), ((6, 6, 2, 4), (1, 1, 2, 4), False), ((6, 6, 2, 4), (1, 3, 1, 2), True),
    ((2, 2, 2, 4), (1, 1, 1, 1), False), ((8, 4, 8, 8), (4, 4, 4, 4), True), ((4, 10, 2, 6), (4, 5, 1, 3), False)])
@pytest.mark.parametrize("compress,ap", [(True, True), (False, False)])
def test_schwarz_faces(dims, block, additive, compress, ap):
    need_gpu()
    U = synth.smooth_links(dims, 101).numpy()
    b = synth.gaussian_spinor(dims, 102)
    op = DiracOp(dims, U, -0.3, 1.0, antiperiodic_t=ap, precisions=("f64", "f32"), compress_links=compress,
                 compress_clover=compress)
    cycles, mr = 2, 2
    want = osap.Schwarz(dims, U, -0.3, 1.0, block, antiperiodic_t=ap).apply(b, cycles, mr, additive=additive)
    bn = op.pack(torch.from_numpy(b).cuda(), "f64")
    kw = dict(block=block, cycles=cycles, mr_iters=mr, additive=additive)
    for prec in ("f64", "f32"):
        got = op.unpack(op.sap(bn, prec=prec, **kw), "f64").cpu().numpy()[0]
        # one apply's bound for each application that a site's result has passed through
        assert rel_l2(got, want) < TOL[prec] * cycles * 2 * (mr + 1), prec
