"""GPU parity of coarse_dslash (Eq. 3) against the oracle: FP64 to 1e-12 and
FP32 to 1e-5 relative (max norm), over the configuration-1 Galerkin operator,
the shapes of the 3-level hierarchy, every launch shape on small grids,
ragged sizes and the edge cases of the interface."""
import numpy as np
import pytest
import torch

import synth
from oracle import coarse, lattice, transfer, wilson
from gpu_util import dev, divisors, host, rel_err

pytestmark = pytest.mark.gpu

TOL = {'c128': 1e-12, 'c64': 1e-5}
CDT = {'c128': torch.complex128, 'c64': torch.complex64}


@pytest.fixture(scope='module')
def galerkin_8x8x8x8_op():
    """Fine 8^4, eps 0.4, seed 0, c_sw 1, m0 -0.2; Gaussian Nvec 24; block 4^4 -> 2^4, N 48."""
    dims, block = (8, 8, 8, 8), (4, 4, 4, 4)
    V = lattice.volume(dims)
    U = synth.gauge_field(dims, 0.4, 0)
    A = wilson.clover_field(U, dims, 1.0)
    Vb = transfer.block_orthonormalize(synth.gaussian((24, V, 12), 0, 1), dims, block)
    return coarse.galerkin(coarse.FineParent(U, A, -0.2, dims), Vb, block)


def random_op(cdims, N, seed):
    Vc = lattice.volume(cdims)
    return coarse.CoarseOp(cdims, synth.gaussian((Vc, N, N), seed, 2), synth.gaussian((8, Vc, N, N), seed + 1, 2))


def gpu_apply(op, u, prec, launch=None):
    from paper_1612_07873_amd import CoarseOp
    g = CoarseOp(op.dims, dev(op.X), dev(op.Y), prec)
    if launch is not None:
        g.set_launch(*launch)
    y = g.apply(dev(u, CDT[prec]))
    return host(y), g


@pytest.mark.parametrize('prec', ['c128', 'c64'])
def test_galerkin_operator_8x8x8x8(galerkin_8x8x8x8_op, prec):
    u = synth.gaussian((16, 48), 0, 2)
    ref = galerkin_8x8x8x8_op.apply(u)
    y, _ = gpu_apply(galerkin_8x8x8x8_op, u, prec)
    err = rel_err(y, ref)
    print('8^4 Galerkin 2^4 N48 %s rel err %.3e' % (prec, err))
    assert err <= TOL[prec]


@pytest.mark.parametrize('cdims,N', [((4, 4, 4, 8), 48), ((2, 2, 2, 4), 64), ((2, 2, 2, 2), 48),
                                     ((8, 8, 8, 16), 48)])
@pytest.mark.parametrize('prec', ['c128', 'c64'])
def test_hierarchy_shapes(cdims, N, prec):
    op = random_op(cdims, N, 10)
    u = synth.gaussian((lattice.volume(cdims), N), 3, 2)
    ref = op.apply(u)
    y, g = gpu_apply(op, u, prec)
    err = rel_err(y, ref)
    print('%s N%d %s launch %s rel err %.3e' % (cdims, N, prec, g.launch(), err))
    assert err <= TOL[prec]


@pytest.mark.parametrize('prec', ['c128', 'c64'])
@pytest.mark.parametrize('cdims,N', [((2, 2, 2, 2), 48), ((2, 2, 2, 4), 64)])
def test_every_launch_shape_agrees(cdims, N, prec):
    op = random_op(cdims, N, 20)
    u = synth.gaussian((lattice.volume(cdims), N), 4, 2)
    ref = op.apply(u)
    from paper_1612_07873_amd import CoarseOp
    g = CoarseOp(op.dims, dev(op.X), dev(op.Y), prec)
    ud = dev(u, CDT[prec])
    J = g.chunks_per_row
    n = 0
    for rows in divisors(N):
        for split in divisors(J):
            if rows * split > 1024:
                continue
            g.set_launch(rows, split)
            err = rel_err(host(g.apply(ud)), ref)
            assert err <= TOL[prec], (rows, split, err)
            n += 1
    assert n > 50


@pytest.mark.parametrize('cdims,N', [((3, 2, 5, 2), 2), ((2, 3, 2, 2), 128), ((5, 2, 2, 3), 30)])
def test_ragged_and_extreme_sizes(cdims, N):
    op = random_op(cdims, N, 30)
    u = synth.gaussian((lattice.volume(cdims), N), 5, 2)
    ref = op.apply(u)
    for prec in ('c128', 'c64'):
        y, _ = gpu_apply(op, u, prec)
        assert rel_err(y, ref) <= TOL[prec]


def test_export_round_trip_and_repeatability(galerkin_8x8x8x8_op):
    from paper_1612_07873_amd import CoarseOp
    g = CoarseOp(galerkin_8x8x8x8_op.dims, dev(galerkin_8x8x8x8_op.X), dev(galerkin_8x8x8x8_op.Y), 'c128')
    X, Y = g.export()
    assert np.array_equal(host(X), galerkin_8x8x8x8_op.X) and np.array_equal(host(Y), galerkin_8x8x8x8_op.Y)
    g32 = CoarseOp(galerkin_8x8x8x8_op.dims, dev(galerkin_8x8x8x8_op.X), dev(galerkin_8x8x8x8_op.Y), 'c64')
    X32, _ = g32.export()
    assert np.array_equal(host(X32), galerkin_8x8x8x8_op.X.astype(np.complex64).astype(np.complex128))
    u = dev(synth.gaussian((16, 48), 1, 2))
    a = host(g.apply(u))
    for _ in range(3):
        assert np.array_equal(host(g.apply(u)), a)     # no atomics: bitwise repeatable


def test_interface_errors(galerkin_8x8x8x8_op):
    from paper_1612_07873_amd import CoarseOp, QmgError
    g = CoarseOp(galerkin_8x8x8x8_op.dims, dev(galerkin_8x8x8x8_op.X), dev(galerkin_8x8x8x8_op.Y), 'c128')
    u = dev(synth.gaussian((16, 48), 1, 2))
    with pytest.raises(TypeError):
        g.apply(u.to(torch.complex64))
    with pytest.raises(QmgError):
        g.set_launch(5, 1)          # 5 does not divide N = 48
    with pytest.raises(QmgError):
        g.set_launch(48, 432)       # more than 1024 threads
    g.set_launch(0, 0)
    assert g.launch()[0] > 0


@pytest.mark.parametrize('storage', ['c128', 'c64', 'h16'])
@pytest.mark.parametrize('cdims,N,nrhs,launches', [
    # (rows, split): two rows per thread or one (odd row tiles), 1 to 3 chunks
    # left after the groups of four, fewer chunks than a group
    ((5, 2, 4, 5), 12, 2, [(12, 1), (3, 9), (6, 3), (12, 27)]),
    ((4, 4, 4, 4), 20, 7, [(20, 1), (5, 5), (10, 9), (20, 45)]),
    ((2, 4, 6, 4), 48, 9, [(48, 1), (16, 9), (48, 12), (24, 36), (3, 108)]),
])
def test_batched_stencil_equals_the_single_one(cdims, N, nrhs, launches, storage):
    """The batched stencil sums in the single one's order whatever the launch
    shape: every member bitwise equal to its single call, whole lattice and (all
    extents even) red-black, and the single call against the oracle."""
    from paper_1612_07873_amd import CoarseOp
    op = random_op(cdims, N, 40)
    V = lattice.volume(cdims)
    U = np.stack([synth.gaussian((V, N), 70 + k, 2) for k in range(nrhs)])
    dt = torch.complex128 if storage == 'c128' else torch.complex64
    g = CoarseOp(op.dims, dev(op.X), dev(op.Y), storage)
    ud = dev(U, dt)
    ref = op.apply(U[0])
    n = 0
    for rows, split in launches:
        if g.chunks_per_row // (2 if storage == 'h16' else 1) % split:
            continue
        g.set_launch(rows, split)
        y = g.apply(ud)
        one = [g.apply(ud[k].contiguous()) for k in range(nrhs)]
        assert all(torch.equal(y[k], one[k]) for k in range(nrhs)), (rows, split)
        assert rel_err(host(one[0]), ref) <= {'c128': 1e-12, 'c64': 1e-5, 'h16': 5e-3}[storage]
        n += 1
    assert n >= 2
    if all(d % 2 == 0 for d in cdims):
        g.prepare_schur()
        ue = ud[:, :V // 2].contiguous()
        y = g.schur(ue)
        assert all(torch.equal(y[k], g.schur(ue[k].contiguous())) for k in range(nrhs))


@pytest.mark.parametrize('N', [16, 32, 48, 64])
@pytest.mark.parametrize('nrhs,storage', [(8, 'h16'), (16, 'b16'), (64, 'h16')])
def test_batch_rounded_in_place_equals_rows_rounded_one_by_one(N, nrhs, storage):
    """The complex64 batch's own rounding to 16 bits against the row-by-row
    quantiser: the same codes and scales, so the same outputs to the bit.  135
    sites: the last work-group of 8 members is half empty.  One row is zero."""
    from paper_1612_07873_amd import CoarseOp, quantize_sites
    cdims = (3, 3, 3, 5)
    V = lattice.volume(cdims)
    op = CoarseOp(cdims, dev(synth.gaussian((V, N, N), 1, 2)), dev(synth.gaussian((8, V, N, N), 2, 2)), storage)
    u = dev(synth.gaussian((nrhs, V, N), 3, 2), torch.complex64)
    u[nrhs - 1, V - 1] = 0
    q, sc = quantize_sites(u.permute(1, 0, 2).contiguous().reshape(V * nrhs, N), storage)
    ref = op.apply_mrhs(q.reshape(V, nrhs, N), sc.reshape(V, nrhs)).permute(1, 0, 2)
    assert torch.equal(torch.view_as_real(op.apply_mrhs_c64(u)), torch.view_as_real(ref.contiguous()))
