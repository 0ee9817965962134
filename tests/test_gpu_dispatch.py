"""Kernels and dispatch branches at the sizes where they can go wrong, against
the oracle (same tolerances as test_gpu_parity.py)."""
from dataclasses import replace

import numpy as np
import pytest
import torch

import synth
from gpu_util import OracleCase, gpu_problem, rel, seeded_state
from test_gpu_parity import _coarse_case, _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny,nz,coarse_dof", [(2, 2, 2, 72), (6, 6, 6, 576), (4, 4, 36, 1539)])
def test_coarse_block_elimination_sizes(nx, ny, nz, coarse_dof):
    """The blocked inversion at a size of one full and one partial 64-unknown
    block, of whole blocks only, and just above the 24 blocks up to which a
    step is one launch: coarse operator, V-cycle and FGMRES solve vs the
    oracle."""
    h = 1.0 / max(nx, ny, nz)
    p = synth.Problem(nx, ny, nz, lx=nx * h, ly=ny * h, lz=nz * h, n_levels=2, patch=2, depth_increment=0.01)
    _coarse_case(p, 2, coarse_dof, f"{nx}x{ny}x{nz} L2")


def test_coarse_inverse_of_an_indefinite_operator():
    """An austenite with c11 < c12 (negative tetragonal shear modulus) makes
    the operators indefinite (about a quarter of the coarsest level's
    eigenvalues are negative), and the elimination with pivoting inside 64 x 64
    blocks loses digits: its check sends the matrix to the elimination with
    pivoting over all rows.  The V-cycle, which contains that inverse, agrees
    with the oracle's LU; condition 1.4e6."""
    nx, ny, nz = 6, 8, 10
    h = 1.0 / nz
    p = synth.Problem(nx, ny, nz, lx=nx * h, ly=ny * h, lz=nz * h, n_levels=2, patch=4, depth_increment=0.01)
    p = replace(p, material=replace(p.material, cubic=(60.0, 126.0, 96.0)))
    U, En = seeded_state(p, 5e-4)
    oc = OracleCase(p, U, En, p.depth_increment, direct=False)
    v = np.random.default_rng(7).standard_normal(oc.sys.b.shape[0])
    gp = gpu_problem(p, U, En, "fp64")
    gp.newton_system(p.depth_increment)
    z = gp.precondition(_dev(v)).cpu().numpy()
    zo = oc.mg.precondition(v)
    assert rel(z, zo) < 1e-10, rel(z, zo)
    gp.close()


@pytest.mark.parametrize("nx,ny,nz,kind", [(4, 4, 4, "patch"), (20, 12, 8, "patch"), (34, 6, 6, "cap"),
                                           (16, 16, 8, "sphere")])
def test_galerkin_level1_from_gauss_points(nx, ny, nz, kind):
    """Level 1 of the Galerkin hierarchy summed straight from the Gauss-point
    tangents (parents per row below, above and at multiples of a workgroup's
    8; the constrained bottom plane; the top layer through the element
    matrices, with contact) is the coarsened assembled finest level.  Entries
    of ~1000 terms summed in another order."""
    h = 1.0 / nx
    p = synth.Problem(nx, ny, nz, lx=1.0, ly=ny * h, lz=nz * h, n_levels=2, kind=kind, patch=2, radius=0.2,
                      depth_increment=0.01)
    U, En = seeded_state(p, 1e-3)
    gp = gpu_problem(p, U, En, "fp64", coarse="galerkin")
    gp.newton_system(p.depth_increment)
    n1 = (nx // 2 + 1) * (ny // 2 + 1) * (nz // 2 + 1)
    x = _dev(np.random.default_rng(3).standard_normal(9 * n1))
    y = gp.jacobian_apply(1, x)
    ya = gp.jacobian_apply(1, x.abs())
    gp.set_tuning("matrix_free", 0, 0)
    gp.newton_system(p.depth_increment)
    z = gp.jacobian_apply(1, x)
    assert torch.isfinite(y).all()
    err = (y - z).reshape(-1, 9)
    scale = z.reshape(-1, 9).abs().amax(0) + ya.reshape(-1, 9).abs().amax(0)
    assert float((err.abs().amax(0) / scale).max()) < 1e-12, (err.abs().amax(0) / scale)
    gp.close()


@pytest.mark.parametrize("precision,tol,ptol", [("fp64", 1e-12, 3e-14), ("mixed", 1e-4, 2e-5)])
@pytest.mark.parametrize("nx,ny,nz,levels", [(4, 4, 4, 2), (6, 10, 2, 2), (16, 4, 12, 3), (24, 24, 24, 3), (28, 24, 24, 3)])
def test_vcycle_of_both_level_kernel_families(nx, ny, nz, levels, precision, tol, ptol):
    """A V-cycle with the small-grid row kernel on every level (row counts that
    leave a remainder of its 8 rows and of a tile, 125 to 18125 rows), and with
    the two-pass kernels: the same 27 x 9 products per entry, summed in another
    order, over 9 sweeps whose factors are below 3 (FP64 243 * 1.1e-16 * 9 * 3;
    FP32 the square root of the terms).  The matrix-free finest level is on
    either side of the node gather's limit of 256 tiles.  The assembled
    product by itself, relative to |A x| + |A |x||: 243 roundings per entry."""
    h = 1.0 / max(nx, ny, nz)
    p = synth.Problem(nx, ny, nz, lx=nx * h, ly=ny * h, lz=nz * h, n_levels=levels, patch=2, depth_increment=0.01)
    U, En = seeded_state(p, 1e-3)
    gp = gpu_problem(p, U, En, precision)
    x = _dev(np.random.default_rng(5).standard_normal(9 * (nx + 1) * (ny + 1) * (nz + 1)))
    for mf in (1, 0):
        gp.set_tuning("matrix_free", 0, mf)
        gp.newton_system(p.depth_increment)
        gp.set_tuning("small_grid_nodes", 0, 40000)
        z = gp.precondition(x)
        gp.set_tuning("small_grid_nodes", 0, 0)
        z2 = gp.precondition(x)
        assert torch.isfinite(z).all()
        err = float((z - z2).norm() / z2.norm())
        assert err < tol, (mf, err)
    kind = 0 if precision == "fp64" else 1
    y2, ya = gp.jacobian_apply(0, x, kind), gp.jacobian_apply(0, x.abs(), kind)
    gp.set_tuning("small_grid_nodes", 0, 40000)
    y = gp.jacobian_apply(0, x, kind)
    assert float((y - y2).norm() / (y2.norm() + ya.norm())) < ptol
    gp.close()


def test_batch_of_both_coarse_elimination_kinds():
    """Coarsest levels of 576 unknowns (a step in one launch) and of 1539 (25
    blocks: panels in a launch of their own) in one batch: every V-cycle is
    bitwise the one of the problem by itself."""
    from paper_2011_08802_amd import mvpf
    probs = []
    for i, (nx, ny, nz) in enumerate([(6, 6, 6), (4, 4, 36), (4, 4, 4)]):
        h = 1.0 / nz
        probs.append(synth.Problem(nx, ny, nz, lx=nx * h, ly=ny * h, lz=1.0, n_levels=2, patch=2, depth_increment=0.01,
                                   seed=synth.BASE_SEED + 40 + i))
    B = mvpf.Batch(probs, "fp64")
    states = [seeded_state(p, 1e-3) for p in probs]
    for i, (U, En) in enumerate(states):
        B.problem(i).set_state(U[:, :3], U[:, 3:], En, 0.0)
    B.newton_system([p.depth_increment for p in probs])
    for i, (p, (U, En)) in enumerate(zip(probs, states)):
        v = _dev(np.random.default_rng(11 + i).standard_normal(9 * (p.nx + 1) * (p.ny + 1) * (p.nz + 1)))
        gp = gpu_problem(p, U, En, "fp64")
        gp.newton_system(p.depth_increment)
        z = gp.precondition(v)
        assert torch.isfinite(z).all()
        assert torch.equal(B.problem(i).precondition(v), z), i
        gp.close()
    B.close()


def _indefinite(p):
    """c11 < c12: about a quarter of the coarsest operator's eigenvalues are negative."""
    return replace(p, material=replace(p.material, cubic=(60.0, 126.0, 96.0)))


def _two_level(nx, ny, nz, seed=synth.BASE_SEED):
    h = 1.0 / max(nx, ny, nz)
    return synth.Problem(nx, ny, nz, lx=nx * h, ly=ny * h, lz=nz * h, n_levels=2, patch=2, depth_increment=0.01, seed=seed)


@pytest.mark.parametrize("overlap", [1, 0])
def test_rejected_coarse_inverse_is_reported_and_replaced(overlap):
    """A definite coarsest operator (1080 unknowns) keeps the block
    elimination's inverse, an indefinite one is rejected by its check and
    inverted with pivoting over all rows, on the side stream or in order: the
    V-cycle is bitwise that of an inversion by pivoting alone, also in the
    next system of the same problem."""
    for p, rejected in ((_two_level(6, 8, 10), 0), (_indefinite(_two_level(6, 8, 10)), 1)):
        U, En = seeded_state(p, 5e-4)
        v = _dev(np.random.default_rng(7).standard_normal(9 * p.n_nodes))
        gp = gpu_problem(p, U, En, "fp64")
        gp.set_tuning("coarse_overlap", 0, overlap)
        out = []
        for force in (0, 1, 0):
            gp.set_tuning("coarse_pivoting", 0, force)
            gp.newton_system(p.depth_increment)
            assert gp.get_tuning("coarse_pivoted") == (1 if force else rejected)
            out.append(gp.precondition(v))
        gp.close()
        assert torch.equal(out[0], out[2])
        if rejected:
            assert torch.equal(out[0], out[1])
        else:
            assert float((out[0] - out[1]).norm() / out[1].norm()) < 1e-10


def test_batch_with_rejected_coarse_inverses():
    """Indefinite and definite coarsest operators of several panel variants
    (576, 1080 and 1296 unknowns rejected, 576 and 72 kept) in one batch: the
    rejected ones are inverted again together, and every V-cycle is bitwise
    the one of the problem by itself."""
    from paper_2011_08802_amd import mvpf
    shapes = [(6, 6, 6, 1), (6, 6, 6, 0), (6, 8, 10, 1), (2, 2, 2, 0), (6, 10, 10, 1)]
    probs = []
    for i, (nx, ny, nz, bad) in enumerate(shapes):
        p = _two_level(nx, ny, nz, synth.BASE_SEED + 60 + i)
        probs.append(_indefinite(p) if bad else p)
    states = [seeded_state(p, 5e-4) for p in probs]
    B = mvpf.Batch(probs, "fp64")
    for i, (U, En) in enumerate(states):
        B.problem(i).set_state(U[:, :3], U[:, 3:], En, 0.0)
    for _ in range(2):
        B.newton_system([p.depth_increment for p in probs])
        for i, (p, (U, En)) in enumerate(zip(probs, states)):
            assert B.problem(i).get_tuning("coarse_pivoted") == shapes[i][3], i
            v = _dev(np.random.default_rng(11 + i).standard_normal(9 * p.n_nodes))
            gp = gpu_problem(p, U, En, "fp64")
            gp.newton_system(p.depth_increment)
            z = gp.precondition(v)
            assert torch.isfinite(z).all()
            assert torch.equal(B.problem(i).precondition(v), z), i
            gp.close()
    B.close()


@pytest.mark.parametrize("nx,ny,nz,coarse_dof", [
    (2, 2, 2, 72),      # one row per thread, one narrow sub-panel
    (6, 6, 6, 576),     # two rows per thread, five outer panels
    (6, 8, 10, 1080),   # five rows per thread of a half-size workgroup
    (6, 10, 10, 1296),  # three rows per thread
    (4, 4, 36, 1539),   # four rows per thread
    (12, 12, 12, 3087), # tournament pivoting, seven blocks of rows, the last one short
])
def test_pivoting_over_all_rows(nx, ny, nz, coarse_dof):
    """The inversion with pivoting over all rows by itself, in each of its
    panel variants: the V-cycle against the oracle's LU (as the tests of the
    block elimination), on the side stream and in order bitwise the same."""
    p = _two_level(nx, ny, nz)
    U, En = seeded_state(p, 5e-4)
    oc = OracleCase(p, U, En, p.depth_increment, direct=False)
    assert oc.mg.levels[-1].A.shape[0] == coarse_dof
    v = np.random.default_rng(7).standard_normal(oc.sys.b.shape[0])
    gp = gpu_problem(p, U, En, "fp64")
    gp.set_tuning("coarse_pivoting", 0, 1)
    out = []
    for overlap in (1, 0):
        gp.set_tuning("coarse_overlap", 0, overlap)
        gp.newton_system(p.depth_increment)
        assert gp.get_tuning("coarse_pivoted") == 1
        out.append(gp.precondition(_dev(v)))
    gp.close()
    assert torch.equal(out[0], out[1])
    err = rel(out[0].cpu().numpy(), oc.mg.precondition(v))
    assert err < 1e-10, err


@pytest.mark.parametrize("nx,ny,nz", [(2, 2, 2), (6, 6, 6), (6, 10, 10), (12, 12, 12), (16, 16, 16), (16, 18, 18)])
def test_definite_coarse_operators_keep_the_block_elimination(nx, ny, nz):
    """The check does not reject the definite operators of the workloads, up
    to 6561 unknowns (128^3's coarsest level) and 8100."""
    p = _two_level(nx, ny, nz)
    U, En = seeded_state(p, 5e-4)
    gp = gpu_problem(p, U, En, "mixed")
    gp.newton_system(p.depth_increment)
    assert gp.get_tuning("coarse_pivoted") == 0
    gp.close()


@pytest.mark.parametrize("kind,coarse,matrix_free,n_var", [
    ("patch", "rediscretise", 1, 6), ("sphere", "galerkin", 1, 6), ("sphere", "rediscretise", 0, 6),
    ("patch", "galerkin", 0, 6), ("patch", "rediscretise", 0, 12)])
def test_slabs_of_every_assembly_path(kind, coarse, matrix_free, n_var):
    """Slabs of one, two and four node layers on 8 x 6 x 12 elements (slabs
    that begin inside a workgroup's 32 elements and inside a tile of 64
    nodes): the diagonal blocks of a matrix-free finest level, the stored
    blocks of an assembled one and its Galerkin products are bitwise those of
    the whole level; seen in the right-hand side, every level's product and
    the V-cycle."""
    from paper_2011_08802_amd import mvpf
    nx, ny, nz = 8, 6, 12
    h = 1.0 / nz
    m = synth.config_material() if n_var == 6 else synth.twelve_variant_material(rho=10.0)
    p = synth.Problem(nx, ny, nz, lx=nx * h, ly=ny * h, lz=nz * h, n_levels=2, kind=kind, patch=2, radius=0.4,
                      depth_increment=0.01, material=m)
    U, En = seeded_state(p, 1e-3)
    nd = 3 + n_var
    rng = np.random.default_rng(8)
    xs = [_dev(rng.standard_normal(nd * (nx // s + 1) * (ny // s + 1) * (nz // s + 1))) for s in (1, 2)]
    nxy = nx * ny
    outs = []
    gp = gpu_problem(p, U, En, "mixed", coarse=coarse)
    if n_var == 6:
        gp.set_tuning("matrix_free", 0, matrix_free)
    # a slab of L node layers holds L + 1 element layers, rounded up to 64
    for slab in (0, *((L + 1) * nxy + 64 for L in (1, 2, 4))):
        gp.set_tuning("assembly_slab_elements", 0, slab)
        gp.newton_system(p.depth_increment)
        outs.append([gp.get_rhs(), gp.jacobian_apply(0, xs[0], mvpf.FP64), gp.jacobian_apply(0, xs[0], mvpf.MIXED),
                     gp.jacobian_apply(1, xs[1], mvpf.FP64), gp.precondition(xs[0])])
    gp.close()
    for o in outs[1:]:
        for k, (a, b) in enumerate(zip(o, outs[0])):
            assert torch.isfinite(a).all() and torch.equal(a, b), k


@pytest.mark.parametrize("precision,tol,ptol", [("fp64", 1e-12, 3e-14), ("mixed", 1e-4, 2e-5)])
@pytest.mark.parametrize("kind,nx,ny,nz", [("patch", 24, 24, 24), ("patch", 28, 24, 24), ("sphere", 2, 2, 2),
                                           ("sphere", 16, 28, 32), ("sphere", 28, 24, 24), ("patch", 12, 16, 16),
                                           ("sphere", 16, 16, 16)])
def test_finest_level_gathers_against_the_assembled_level(kind, nx, ny, nz, precision, tol, ptol):
    """The node gathers by tiles (up to 256 tiles of 64 nodes: 25^3 nodes, 245
    tiles, and 17 x 29 x 33, 255; the FP32 sweep 64: 13 x 17 x 17, 59, and 17^3,
    77) and by nodes (29 x 25 x 25), product, defect and sweep with contact
    faces and without, against the assembled finest level: the product
    relative to |A x| + |A |x|| and the V-cycle, tolerances as for the two
    kernel families of the assembled levels."""
    from paper_2011_08802_amd import mvpf
    h = 1.0 / nx
    p = synth.Problem(nx, ny, nz, lx=1.0, ly=ny * h, lz=nz * h, n_levels=2 if nx == 2 else 3, kind=kind,
                      patch=2, radius=0.4, depth_increment=0.01)
    U, En = seeded_state(p, 1e-3)
    x = _dev(np.random.default_rng(5).standard_normal(9 * p.n_nodes))
    k = mvpf.FP64 if precision == "fp64" else mvpf.MIXED
    gp = gpu_problem(p, U, En, precision)
    out = []
    for mf in (1, 0):
        gp.set_tuning("matrix_free", 0, mf)
        gp.newton_system(p.depth_increment)
        out.append((gp.jacobian_apply(0, x, k), gp.jacobian_apply(0, x.abs(), k), gp.precondition(x)))
    gp.close()
    (y, ya, z), (y0, ya0, z0) = out
    assert torch.isfinite(y).all() and torch.isfinite(z).all()
    assert float((y - y0).norm() / (y0.norm() + ya0.norm())) < ptol
    assert float((z - z0).norm() / z0.norm()) < tol


def test_batch_assembled_in_slabs_with_a_rejected_coarse_inverse():
    """A batch of which one problem assembles in slabs takes a stream per
    problem: its coarsest operators are still inverted together, the rejected
    one again beside the others' assembly, and every V-cycle and right-hand side is
    bitwise the one of the problem by itself."""
    from paper_2011_08802_amd import mvpf
    probs = [_two_level(6, 6, 6, synth.BASE_SEED + 80), _indefinite(_two_level(6, 8, 10, synth.BASE_SEED + 81)),
             _two_level(8, 6, 12, synth.BASE_SEED + 82)]
    states = [seeded_state(p, 5e-4) for p in probs]
    B = mvpf.Batch(probs, "mixed")
    B.problem(2).set_tuning("assembly_slab_elements", 0, 2 * 48 + 64)
    for i, (U, En) in enumerate(states):
        B.problem(i).set_state(U[:, :3], U[:, 3:], En, 0.0)
    for _ in range(2):
        B.newton_system([p.depth_increment for p in probs])
        for i, (p, (U, En)) in enumerate(zip(probs, states)):
            assert B.problem(i).get_tuning("coarse_pivoted") == (i == 1)
            v = _dev(np.random.default_rng(11 + i).standard_normal(9 * p.n_nodes))
            gp = gpu_problem(p, U, En, "mixed")
            gp.newton_system(p.depth_increment)
            z = gp.precondition(v)
            assert torch.isfinite(z).all()
            assert torch.equal(B.problem(i).precondition(v), z), i
            assert torch.equal(B.problem(i).get_rhs(), gp.get_rhs()), i
            gp.close()
    B.close()
