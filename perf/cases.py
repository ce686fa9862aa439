"""Timed cases of the multigrid framework: its operators, transfers, setup
product, learned smoother and whole solves through the package's public classes.

A case names a `kind` and its sizes.  Twelve right-hand sides are one
propagator (a source for each spin and colour), the batch lattice QCD programs
solve together; 8, 16, 32 and 64 are the batches of the matrix-core stencil.
Links are U = exp(i eps H) with H a random traceless Hermitian matrix; vectors
are complex Gaussian.  Coarse operators carry a diagonally dominant local
block, as Galerkin products do.
"""
import json
import math
import os

import numpy as np
import torch

from paper_1612_07873_amd import PTC, BiCGStab, CoarseOp, FineOp, Multigrid, Transfer, build_coarse_op

EPS = 0.3
C128 = torch.complex128
ITEM = {'c128': 16, 'c64': 8, 'h16': 4, 'b16': 4}   # bytes of a stored complex number
with open(os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), 'tests', 'golden',
                       'm0_16x16x16x32.json')) as _f:
    M0 = float(json.load(_f)['m0'])


# ------------------------------------------------------------------- the cases
def listed():
    return [
        # the smallest coarsest grid in full precision: one launch, all latency
        dict(name='coarse 2x2x2x2 N48 c128', kind='coarse', form='apply', dims='2x2x2x2', N=48, storage='c128',
             nrhs=1),
        # level 1 of a 16^3x32 hierarchy, the stencil of a single FP32 solve
        dict(name='coarse 4x4x4x8 N48 c64', kind='coarse', form='apply', dims='4x4x4x8', N=48, storage='c64', nrhs=1),
        # the red-black coarse operator on a propagator's twelve right-hand sides, FP32
        dict(name='coarse schur 4x4x4x8 N64 x12', kind='coarse', form='schur', dims='4x4x4x8', N=64, storage='c64',
             nrhs=12),
        # level 1 of a 32^3x64 hierarchy, 16-bit links, a batch on the matrix cores
        dict(name='coarse mrhs 8x8x8x16 N48 x16', kind='coarse', form='mrhs', dims='8x8x8x16', N=48, storage='h16',
             nrhs=16),
        # the fine operator of a single FP32 solve
        dict(name='fine 16x16x16x32 c64', kind='fine', form='apply', dims='16x16x16x32', storage='c64', reals=18,
             nrhs=1),
        # the fine operator of the outer FP64 solve on a lattice with odd extents
        dict(name='fine 7x10x9x14 c128', kind='fine', form='apply', dims='7x10x9x14', storage='c128', reals=18,
             nrhs=1),
        # the red-black fine operator with 16-bit links on a propagator, no power-of-two extents
        dict(name='fine schur 12x12x12x24 h16 x12', kind='fine', form='schur', dims='12x12x12x24', storage='h16',
             reals=18, nrhs=12),
        # restriction and prolongation of a propagator between the two finest levels
        dict(name='transfer 16x16x16x32 c64 x12', kind='transfer', dims='16x16x16x32', dof=12, block='4x4x4x4',
             nvec=24, storage='c64', nrhs=12),
        # the Galerkin product of the setup, fine operator to level 1
        dict(name='galerkin 16x16x16x32 nvec24', kind='galerkin', dims='16x16x16x32', dof=12, block='4x4x4x4',
             nvec=24),
        # training of the learned smoother: gradients of a mini-batch of two
        dict(name='ptc train 8x8x8x16', kind='ptc', form='train', dims='8x8x8x16', hidden=8, batch=2),
        # time to solution of one right-hand side, red-black on every level
        dict(name='solve 16x16x16x32 c64', kind='solve', dims='16x16x16x32', block='4x4x4x4', nvec=24, nvec2=32,
             storage='c64', evenodd=True, nrhs=1),
        # time to solution of a propagator
        dict(name='solve 16x16x16x32 c64 x12', kind='solve', dims='16x16x16x32', block='4x4x4x4', nvec=24, nvec2=32,
             storage='c64', evenodd=True, nrhs=12),
    ]


def _extents(rng, lo, hi, most, even):
    """Four lattice extents in [lo, hi], the time extent not the smallest, at most `most` sites."""
    while True:
        d = [int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))))) for _ in range(4)]
        if even:
            d = [max(2, 2 * ((x + 1) // 2)) for x in d]
        d[3] = max(d)
        if math.prod(d) <= most:
            return d


def _x(d):
    return 'x'.join(str(v) for v in d)


def draw(rng):
    kind = rng.choice(['coarse', 'coarse', 'coarse', 'fine', 'fine', 'fine', 'transfer', 'transfer', 'galerkin', 'ptc',
                       'solve', 'bicgstab'])
    if kind == 'coarse':
        form = rng.choice(['apply', 'apply', 'schur', 'mrhs'])
        if form == 'mrhs':
            return dict(kind=kind, form=form, dims=_x(_extents(rng, 2, 10, 4096, False)),
                        N=rng.choice([16, 32, 48, 64]), storage=rng.choice(['h16', 'b16']),
                        nrhs=rng.choice([8, 16, 32, 64]))
        storage = rng.choice(['c128', 'c64', 'c64', 'h16'])
        return dict(kind=kind, form=form, dims=_x(_extents(rng, 2, 8, 1024, form == 'schur')),
                    N=4 * rng.randint(4, 16) if storage == 'h16' else 2 * rng.randint(8, 32), storage=storage,
                    nrhs=rng.choice([1, rng.randint(2, 16), 12]))
    if kind == 'fine':
        form = rng.choice(['apply', 'schur'])
        storage = rng.choice(['c128', 'c64', 'h16', 'b16'])
        nrhs = rng.choice([1, 1, rng.randint(2, 12)])
        return dict(kind=kind, form=form, dims=_x(_extents(rng, 4, 24, 131072 // nrhs, form == 'schur')),
                    storage=storage, reals=18 if storage == 'c128' else rng.choice([18, 18, 12]), nrhs=nrhs)
    if kind in ('transfer', 'galerkin'):
        block = [rng.choice([2, 3, 4]) for _ in range(4)]
        fine = rng.random() < 0.7
        while True:
            dims = [b * rng.randint(2, 5) for b in block]
            if math.prod(dims) <= (65536 if fine else 2048):
                break
        nvec = rng.randint(8, 32) if fine else rng.randint(8, 24)
        while nvec > math.prod(block) * 6:
            nvec -= 1
        case = dict(kind=kind, dims=_x(dims), dof=12 if fine else 2 * rng.randint(8, 24), block=_x(block), nvec=nvec)
        if kind == 'transfer':
            case.update(storage=rng.choice(['c64', 'c64', 'h16', 'c128']), nrhs=rng.choice([1, rng.randint(2, 16)]))
        return case
    if kind == 'ptc':
        return dict(kind=kind, form=rng.choice(['train', 'forward']), dims=_x(_extents(rng, 4, 16, 16384, False)),
                    hidden=8, batch=rng.randint(1, 3))
    if kind == 'bicgstab':
        return dict(kind=kind, dims=_x(_extents(rng, 6, 12, 16384, True)), storage=rng.choice(['c64', 'h16']))
    dims = [4 * rng.randint(2, 4) for _ in range(3)] + [4 * rng.randint(2, 6)]
    return dict(kind='solve', dims=_x(dims), block='4x4x4x4', nvec=4 * rng.randint(3, 6), nvec2=0,
                storage=rng.choice(['c64', 'h16']), evenodd=rng.choice([True, False]), nrhs=rng.choice([1, 4, 8, 12]))


# ------------------------------------------------------------------ the inputs
def _dims(text):
    return tuple(int(v) for v in text.split('x'))


def _dev():
    return torch.device('cuda' if torch.cuda.is_available() else 'cpu')


def _gen(seed, salt):
    g = torch.Generator(device=_dev())
    g.manual_seed(1000003 * int(seed) + salt)
    return g


def _gaussian(shape, g, dtype=C128):
    """Complex Gaussian (N(0,1) + i N(0,1)) / sqrt(2), drawn in 64 bits."""
    return torch.randn(shape, dtype=C128, device=_dev(), generator=g).to(dtype)


def _gauge(dims, g):
    """U = exp(i eps H), H = sum_a h_a lambda_a / 2 with Gaussian h_a: [4][V][3][3] complex128."""
    V = math.prod(dims)
    h = torch.randn((4 * V, 8), dtype=torch.float64, device=_dev(), generator=g) * (0.5 * EPS)
    A = torch.zeros((4 * V, 3, 3), dtype=C128, device=_dev())
    r3 = 1 / math.sqrt(3.0)
    A[:, 0, 0], A[:, 1, 1], A[:, 2, 2] = h[:, 2] + r3 * h[:, 7] + 0j, -h[:, 2] + r3 * h[:, 7] + 0j, -2 * r3 * h[:, 7] + 0j
    for (r, c), (a, b) in (((0, 1), (0, 1)), ((0, 2), (3, 4)), ((1, 2), (5, 6))):
        A[:, r, c] = torch.complex(h[:, a], -h[:, b])
        A[:, c, r] = torch.complex(h[:, a], h[:, b])
    A = 1j * A / 16
    U = torch.eye(3, dtype=C128, device=_dev()).expand(4 * V, 3, 3).clone()
    for k in range(14, 0, -1):     # Taylor series of exp(A), Horner form
        U = _mm3(A, U) / k
        for i in range(3):
            U[:, i, i] += 1
    for _ in range(4):             # exp(16 A)
        U = _mm3(U, U)
    return U.reshape(4, V, 3, 3).contiguous()


def _mm3(a, b):
    """Products of 3x3 matrices over the leading index, written out (thin batched products are slow as library calls)."""
    return sum(a[..., :, k, None] * b[..., None, k, :] for k in range(3))


def _coarse_blocks(V, N, g):
    """X [V][N][N] and Y [8][V][N][N] complex128: X near a multiple of the unit matrix, hops of order one in norm."""
    X = _gaussian((V, N, N), g) * (0.5 / math.sqrt(N))
    X += 4.0 * torch.eye(N, dtype=C128, device=_dev())
    Y = _gaussian((8, V, N, N), g) * (0.5 / math.sqrt(N))
    return X, Y


def _vec(storage):
    return C128 if storage == 'c128' else torch.complex64


def _lead(nrhs, *shape):
    return (nrhs,) + shape if nrhs > 1 else shape


def _inputs(case, seed):
    """The random inputs of a case on the GPU, from the seed alone."""
    kind = case['kind']
    g = _gen(seed, 1)
    dims = _dims(case['dims'])
    V = math.prod(dims)
    if kind == 'coarse':
        X, Y = _coarse_blocks(V, case['N'], g)
        rows = V // 2 if case['form'] == 'schur' else V
        lead = (case['nrhs'],) if case['form'] == 'mrhs' else _lead(case['nrhs'])
        return dict(X=X, Y=Y, u=_gaussian(lead + (rows, case['N']), g, _vec(case['storage'])))
    if kind == 'fine':
        rows = V // 2 if case['form'] == 'schur' else V
        return dict(U=_gauge(dims, g), psi=_gaussian(_lead(case['nrhs'], rows, 4, 3), g, _vec(case['storage'])))
    if kind == 'transfer':
        Vc = V // math.prod(_dims(case['block']))
        dt = _vec(case['storage'])
        return dict(null=_gaussian((case['nvec'], V, case['dof']), g),
                    f=_gaussian(_lead(case['nrhs'], V, case['dof']), g, dt),
                    c=_gaussian(_lead(case['nrhs'], Vc, 2 * case['nvec']), g, dt))
    if kind == 'galerkin':
        out = dict(null=_gaussian((case['nvec'], V, case['dof']), g))
        if case['dof'] == 12:
            out['U'] = _gauge(dims, g)
        else:
            out['X'], out['Y'] = _coarse_blocks(V, case['dof'], g)
        return out
    if kind == 'ptc':
        C = case['hidden']
        W1 = _gaussian((9, C, 1, 4, 4), g) * 0.05
        W2 = _gaussian((9, 1, C, 4, 4), g) * 0.05
        W1[0, 0, 0] += torch.eye(4, device=_dev())
        W2[0, 0, 0] += torch.eye(4, device=_dev()) / (4.0 + M0)
        return dict(U=_gauge(dims, g), W1=W1.to(torch.complex64), W2=W2.to(torch.complex64),
                    r=_gaussian((case['batch'], V, 4, 3), g, torch.complex64))
    out = dict(U=_gauge(dims, g), x=_gaussian((case.get('nrhs', 1), V, 4, 3), g))
    if kind == 'solve':
        Vc = V // math.prod(_dims(case['block']))
        out['starts'] = [_gaussian((case['nvec'], V, 12), g)]
        if case['nvec2']:
            out['starts'].append(_gaussian((case['nvec2'], Vc, 2 * case['nvec']), g))
    return out


def prepare(case, seed):
    kind = case['kind']
    t = _inputs(case, seed)
    dims = _dims(case['dims'])
    state = dict(kind=kind, form=case.get('form'))
    if kind == 'coarse':
        op = CoarseOp(dims, t['X'], t['Y'], case['storage'])
        u = t['u']
        state.update(op=op, u=u, out=torch.empty_like(u))
        if case['form'] == 'apply':       # launch shapes are tuned once per lattice, N and storage
            one = u if u.dim() == 2 else u[0]
            op.tune(one.contiguous(), torch.empty_like(one), cold=op.V >= 64)
        elif case['form'] == 'schur':
            op.prepare_schur()
    elif kind == 'fine':
        op = FineOp(dims, t['U'], M0, 1.0, True, case['storage'], link_reals=case['reals'])
        state.update(op=op, psi=t['psi'], out=torch.empty_like(t['psi']))
    elif kind == 'transfer':
        T = Transfer(dims, case['dof'], _dims(case['block']), t['null'], case['storage'])
        state.update(T=T, f=t['f'], c=t['c'], cout=torch.empty_like(t['c']), fout=torch.empty_like(t['f']))
    elif kind == 'galerkin':
        state['T'] = Transfer(dims, case['dof'], _dims(case['block']), t['null'], 'c128')
        state['fine'] = FineOp(dims, t['U'], M0, 1.0, True, 'c128') if case['dof'] == 12 else None
        state['parent'] = CoarseOp(dims, t['X'], t['Y'], 'c128') if case['dof'] != 12 else None
    elif kind == 'ptc':
        net = PTC(FineOp(dims, t['U'], M0, 1.0, True, 'c64'), case['hidden'])
        net.set_weights(t['W1'], t['W2'])
        state.update(net=net, r=[r.contiguous() for r in t['r']])
    else:
        hi = FineOp(dims, t['U'], M0, 1.0, True, 'c128')
        b = hi.apply(t['x'])
        state['x'] = torch.empty_like(t['x'])
        if kind == 'bicgstab':
            lo = FineOp(dims, t['U'], M0, 1.0, True, case['storage'])
            state.update(solver=BiCGStab(hi, lo, True), b=b[0].contiguous(), x=state['x'][0].contiguous())
        else:
            h16 = 'h16' if case['storage'] == 'h16' else None
            level = dict(block=_dims(case['block']), nvec=case['nvec'], setup_iters=100, smoother_steps=4,
                         coarse_tol=0.25, coarse_maxit=10 if case['nvec2'] else 100, coarse_storage=h16)
            levels = [level]
            if case['nvec2']:
                levels.append(dict(level, block=(2, 2, 2, 2), nvec=case['nvec2'], coarse_maxit=100))
            mg = Multigrid(dims, t['U'], M0, 1.0, levels, t['starts'], fine_storage=h16)
            mg.set_evenodd(case['evenodd'])
            state.update(mg=mg, b=b, single=case['nrhs'] == 1)
            if state['single']:
                state.update(b=b[0].contiguous(), x=state['x'][0].contiguous())
    return state


def run(s):
    kind, form = s['kind'], s['form']
    if kind == 'coarse':
        if form == 'apply':
            return s['op'].apply(s['u'], s['out'])
        if form == 'schur':
            return s['op'].schur(s['u'], s['out'])
        return s['op'].apply_mrhs_c64(s['u'], s['out'])
    if kind == 'fine':
        return s['op'].apply(s['psi'], s['out']) if form == 'apply' else s['op'].schur(s['psi'], s['out'])
    if kind == 'transfer':
        return {'restrict': s['T'].restrict(s['f'], s['cout']), 'prolong': s['T'].prolong(s['c'], s['fout'])}
    if kind == 'galerkin':
        X, Y = build_coarse_op(s['T'], fine=s['fine'], parent=s['parent'], storage='c128').export()
        return {'X': X, 'Y': Y}
    if kind == 'ptc':
        net = s['net']
        if form == 'forward':
            return [net.forward(r) for r in s['r']]
        net.zero_grad()
        for r in s['r']:
            net.accumulate_residual(r)
        G1, G2, loss = net.grad()
        return {'G1': G1, 'G2': G2, 'loss': loss}
    # a propagator is kept to 1e-12 so that it is right to nine digits
    if kind == 'bicgstab':
        return s['solver'].solve(s['b'], s['x'], tol=1e-12)[0]
    if s['single']:
        return s['mg'].solve(s['b'], s['x'], tol=1e-12)[0]
    return s['mg'].solve_multi(s['b'], s['x'], tol=1e-12)[0]


# ------------------------------------------------------- what a pass has to do
def work(case):
    kind = case['kind']
    dims = _dims(case['dims'])
    V, m = math.prod(dims), case.get('nrhs', 1)
    if kind == 'coarse':
        N, cb = case['N'], ITEM[case['storage']]
        vb = 16 if case['storage'] == 'c128' else 8
        if case['form'] == 'schur':
            # X_ee, X_oo^-1 and the 16 hop blocks of a pair of sites
            return {'bytes': V // 2 * (18 * N * N * cb + 2 * N * m * vb), 'flops': V // 2 * 18 * 8 * N * N * m}
        return {'bytes': V * (9 * N * N * cb + 2 * N * m * vb), 'flops': V * 72 * N * N * m}
    if kind == 'fine':
        cb = ITEM[case['storage']]
        vb = 16 if case['storage'] == 'c128' else 8
        links = 4 * case['reals'] * cb // 2
        local = 36 * cb                       # the clover term, two packed 6x6 Hermitian blocks
        if case['form'] == 'schur':
            # every link once, C on the even and C^-1 on the odd sites
            return {'bytes': V * links + V * local + V // 2 * 24 * vb * m, 'flops': V * 1824 * m}
        return {'bytes': V * (links + local + 24 * vb * m), 'flops': V * 1824 * m}
    if kind in ('transfer', 'galerkin'):
        dof, nvec, cb = case['dof'], case['nvec'], ITEM[case.get('storage', 'c128')]
        Vc, N = V // math.prod(_dims(case['block'])), 2 * case['nvec']
        if kind == 'transfer':
            vb = 16 if case['storage'] == 'c128' else 8
            # each direction reads the basis once
            return {'bytes': 2 * (V * dof * nvec * cb + m * (V * dof + Vc * N) * vb), 'flops': 16 * V * dof * nvec * m}
        half = dof // 2
        parent = (72 + 72) * 16 // 2 if dof == 12 else 9 * dof * dof * 16
        # per site and term: H P (two chirality halves), then P^+ (H P)
        flops = 9 * 8 * (dof * half * 2 * nvec + 2 * nvec * half * N)
        if dof == 12:
            flops = 9 * 8 * (6 * 6 * nvec * 2 + 2 * nvec * half * N)
        return {'bytes': V * (dof * nvec * 16 + parent) + Vc * 9 * N * N * 16, 'flops': V * flops}
    if kind == 'ptc':
        C, B = case['hidden'], case['batch']
        transports = 9 * 4 * 66 * 2
        mix = 9 * 4 * 4 * 3 * 8 * C
        if case['form'] == 'forward':
            return {'bytes': B * V * (288 + 192), 'flops': B * V * (2 * transports + 9 * 9 * 4 * 4 * 3 * 8)}
        # forward, backward through the data and the weights, M and M^+ of the residual loss
        return {'bytes': B * V * (288 + 288 + 96 + 2 * C * 96), 'flops': B * V * (6 * transports + 5 * mix + 2 * 1824)}
    # about ten applications of M for each of twenty preconditioned outer steps
    cb = ITEM[case['storage']]
    applies = 200
    return {'bytes': applies * V * (72 * cb + 192 * m), 'flops': applies * V * 1824 * m}


# ------------------------------------------------- the same values in 64 bits
def _neighbours(dims, mu, step, dev):
    x = torch.arange(math.prod(dims), device=dev).reshape(tuple(reversed(dims)))
    return torch.roll(x, -step, dims=3 - mu).reshape(-1)


def _coords(dims, dev):
    i = torch.arange(math.prod(dims), device=dev)
    out = []
    for d in dims:
        out.append(i % d)
        i = i // d
    return out


def _parity_sites(dims, p, dev):
    return torch.nonzero(sum(_coords(dims, dev)) % 2 == p).reshape(-1)


def _gammas():
    s = [np.array([[0, 1], [1, 0]], complex), np.array([[0, -1j], [1j, 0]]), np.array([[1, 0], [0, -1]], complex)]
    z = np.zeros((2, 2), complex)
    g = [np.block([[z, -1j * k], [1j * k, z]]) for k in s]
    return g + [np.block([[z, np.eye(2)], [np.eye(2), z]])]


class _Dirac:
    """The Wilson-clover operator on [nrhs][V][4][3] fields in complex128."""

    def __init__(self, U, dims, m0, csw=1.0):
        self.U, self.dims, self.V, self.m0 = U, dims, math.prod(dims), m0
        dev = U.device
        self.dev = dev
        self.nb = {(mu, s): _neighbours(dims, mu, s, dev) for mu in range(4) for s in (1, -1)}
        t = _coords(dims, dev)[3]
        one = torch.ones(self.V, dtype=torch.float64, device=dev)
        self.eta = {(mu, s): one for mu in range(4) for s in (1, -1)}
        self.eta[(3, 1)] = torch.where(t == dims[3] - 1, -one, one)
        self.eta[(3, -1)] = torch.where(t == 0, -one, one)
        g = _gammas()
        self.g = [torch.tensor(x, dtype=C128, device=dev) for x in g]
        # clover term, [V][2][6][6]: its two chirality blocks
        A = torch.zeros((self.V, 4, 3, 4, 3), dtype=C128, device=dev)
        for mu in range(4):
            for nu in range(mu + 1, 4):
                Q = self._leaves(mu, nu)
                F = (Q - Q.mH) / 8
                sg = torch.tensor(0.5j * (g[mu] @ g[nu] - g[nu] @ g[mu]), dtype=C128, device=dev)
                A += (0.5j * csw) * sg[None, :, None, :, None] * F[:, None, :, None, :]
        A = A.reshape(self.V, 2, 6, 2, 6)
        self.C = torch.stack([A[:, 0, :, 0], A[:, 1, :, 1]], dim=1)
        self.C = self.C + (4.0 + m0) * torch.eye(6, dtype=C128, device=dev)

    def _leaves(self, mu, nu):
        Um, Un = self.U[mu], self.U[nu]
        pm, pn, mm, mn = self.nb[mu, 1], self.nb[nu, 1], self.nb[mu, -1], self.nb[nu, -1]

        def chain(*m):
            out = m[0]
            for x in m[1:]:
                out = _mm3(out, x)
            return out
        q = chain(Um, Un[pm], Um[pn].mH, Un.mH)
        q = q + chain(Un, Um[pn[mm]].mH, Un[mm].mH, Um[mm])
        q = q + chain(Um[mm].mH, Un[mn[mm]].mH, Um[mn[mm]], Un[mn])
        return q + chain(Un[mn].mH, Um[mn], Un[mn[pm]], Um.mH)

    def transport(self, psi, mu, s):
        """eta U_mu(x) psi(x + mu), or eta U_mu(x - mu)^+ psi(x - mu); psi [..][V][spin][3]."""
        n = self.nb[mu, s]
        W = self.U[mu] if s > 0 else self.U[mu][n].mH
        p = psi[..., n, :, :]
        t = sum(W[:, None, :, k] * p[..., :, k, None] for k in range(3))
        return self.eta[mu, s][:, None, None] * t

    def hops(self, psi):
        out = torch.zeros_like(psi)
        for mu in range(4):
            for s in (1, -1):
                t = self.transport(psi, mu, s)
                out -= 0.5 * (t - s * self.spin(self.g[mu], t))
        return out

    def spin(self, W, t):
        return sum(W[..., :, b, None] * t[..., :, b, None, :] for b in range(4))

    def local(self, psi, C=None):
        C = self.C if C is None else C
        p = psi.reshape(psi.shape[:-2] + (2, 6))
        return sum(C[..., k] * p[..., k, None] for k in range(6)).reshape(psi.shape)

    def apply(self, psi):
        return self.local(psi) + self.hops(psi)


def _inverse(C):
    """Inverses of 6x6 blocks near a multiple of the unit matrix (Gauss-Jordan, no pivoting)."""
    n = C.shape[-1]
    a = torch.cat([C, torch.eye(n, dtype=C.dtype, device=C.device).expand(C.shape)], dim=-1)
    for k in range(n):
        row = a[..., k, :] / a[..., k, k, None]
        a = a - a[..., :, k, None] * row[..., None, :]
        a[..., k, :] = row
    return a[..., n:]


def _coarse_sum(X, Y, u, nbrs, sites):
    """sum over the given blocks at `sites`: X u + sum_d Y_d u(neighbour); u [m][V][N], X or Y may be None."""
    out = 0
    if X is not None:
        out = torch.matmul(X[sites], u[:, sites].permute(1, 2, 0).contiguous())
    if Y is not None:
        for d in range(8):
            out = out + torch.matmul(Y[d][sites], u[:, nbrs[d][sites]].permute(1, 2, 0).contiguous())
    return out.permute(2, 0, 1).contiguous()


def _basis(null, dims, dof, block):
    """Block-orthonormal basis [Vc][2][B*dof/2][nvec] (QR of each aggregate and chirality, positive
    diagonal), the sites of each aggregate [Vc][B] and the aggregate of each site."""
    dev = null.device
    x = _coords(dims, dev)
    cd = [d // b for d, b in zip(dims, block)]
    owner, f = torch.zeros_like(x[0]), 1
    for m in range(4):
        owner += f * (x[m] // block[m])
        f *= cd[m]
    sites = torch.argsort(owner, stable=True).reshape(f, -1)
    B, nvec, half = sites.shape[1], null.shape[0], dof // 2
    W = null[:, sites].reshape(nvec, f, B, 2, half).permute(1, 3, 2, 4, 0).reshape(f, 2, B * half, nvec).contiguous()
    for _ in range(2):                  # Cholesky QR, twice
        G = torch.matmul(W.mH.contiguous(), W).cpu()
        L = torch.linalg.cholesky(G)
        Ri = torch.linalg.solve_triangular(L.mH, torch.eye(nvec, dtype=C128).expand(G.shape), upper=True)
        W = torch.matmul(W, Ri.contiguous().to(dev))
    return W, sites, owner


def exact(case, seed):
    kind = case['kind']
    t = _inputs(case, seed)
    dims = _dims(case['dims'])
    V = math.prod(dims)
    dev = _dev()
    if kind == 'coarse':
        u = t['u'].to(C128)
        u = u if u.dim() == 3 else u[None]
        nbrs = [_neighbours(dims, d // 2, 1 - 2 * (d % 2), dev) for d in range(8)]
        if case['form'] == 'schur':
            even, odd = _parity_sites(dims, 0, dev), _parity_sites(dims, 1, dev)
            full = torch.zeros((u.shape[0], V, case['N']), dtype=C128, device=dev)
            full[:, even] = u
            Xi = torch.from_numpy(np.linalg.inv(t['X'][odd].cpu().numpy())).to(dev)
            h = torch.matmul(Xi, _coarse_sum(None, t['Y'], full, nbrs, odd).permute(1, 2, 0).contiguous())
            mid = torch.zeros_like(full)
            mid[:, odd] = h.permute(2, 0, 1)
            y = _coarse_sum(t['X'], None, full, nbrs, even) - _coarse_sum(None, t['Y'], mid, nbrs, even)
        else:
            y = _coarse_sum(t['X'], t['Y'], u, nbrs, torch.arange(V, device=dev))
        return y if case['form'] == 'mrhs' or case['nrhs'] > 1 else y[0]
    if kind == 'fine':
        D = _Dirac(t['U'], dims, M0)
        psi = t['psi'].to(C128)
        if case['form'] == 'apply':
            return D.apply(psi)
        even, odd = _parity_sites(dims, 0, dev), _parity_sites(dims, 1, dev)
        full = torch.zeros(psi.shape[:-3] + (V, 4, 3), dtype=C128, device=dev)
        full[..., even, :, :] = psi
        h = D.hops(full)
        mid = torch.zeros_like(full)
        mid[..., odd, :, :] = D.local(h[..., odd, :, :].contiguous(), _inverse(D.C[odd]))
        out = D.local(full) - D.hops(mid)
        return out[..., even, :, :].contiguous()
    if kind in ('transfer', 'galerkin'):
        dof, nvec, half = case['dof'], case['nvec'], case['dof'] // 2
        W, sites, owner = _basis(t['null'], dims, dof, _dims(case['block']))
        Vc, B = sites.shape
        if kind == 'transfer':
            f, c = t['f'].to(C128), t['c'].to(C128)
            m = case['nrhs']
            f, c = f.reshape(m, V, dof), c.reshape(m, Vc, 2, nvec)
            fb = f[:, sites].reshape(m, Vc, B, 2, half).permute(1, 3, 2, 4, 0).reshape(Vc, 2, B * half, m).contiguous()
            r = torch.matmul(W.mH.contiguous(), fb).permute(3, 0, 1, 2).reshape(t['c'].shape)
            p = torch.matmul(W, c.permute(1, 2, 3, 0).contiguous())
            out = torch.empty((m, V, dof), dtype=C128, device=dev)
            out[:, sites.reshape(-1)] = p.reshape(Vc, 2, B, half, m).permute(4, 0, 2, 1, 3).reshape(m, V, dof)
            return {'restrict': r.contiguous(), 'prolong': out.reshape(t['f'].shape)}
        return _galerkin(t, dims, dof, nvec, W, sites, owner)
    if kind == 'ptc':
        return _ptc(case, t, dims)
    return t['x'] if case.get('nrhs', 1) > 1 else t['x'][0]


def _galerkin(t, dims, dof, nvec, W, sites, owner):
    dev, half, N = W.device, dof // 2, 2 * nvec
    Vc, B = sites.shape
    V = Vc * B
    P = torch.zeros((V, dof, N), dtype=C128, device=dev)     # the slice of the prolongator at each site
    Wb = W.reshape(Vc, 2, B, half, nvec).permute(0, 2, 1, 3, 4).reshape(V, 2, half, nvec)
    at = sites.reshape(-1)
    P[at, :half, :nvec], P[at, half:, nvec:] = Wb[:, 0], Wb[:, 1]
    X = torch.zeros((Vc, N, N), dtype=C128, device=dev)
    Y = torch.zeros((8, Vc, N, N), dtype=C128, device=dev)
    if dof == 12:
        D = _Dirac(t['U'], dims, M0)
        spin = [(torch.eye(4, dtype=C128, device=dev) - (1 - 2 * (d % 2)) * D.g[d // 2]) for d in range(8)]
    step = max(1, 16384 // B)
    for c0 in range(0, Vc, step):
        s = sites[c0:c0 + step]
        n = s.shape[0]
        xs = s.reshape(-1)
        PH = P[xs].mH.contiguous()

        def block_sum(T, mask=None):
            T = T.reshape(n, B, N, N)
            return T.sum(1) if mask is None else (T * mask.reshape(n, B, 1, 1)).sum(1)
        if dof == 12:
            L = torch.zeros((xs.numel(), 12, 12), dtype=C128, device=dev)
            L[:, :6, :6], L[:, 6:, 6:] = D.C[xs, 0], D.C[xs, 1]
        else:
            L = t['X'][xs]
        X[c0:c0 + n] += block_sum(torch.matmul(PH, torch.matmul(L, P[xs])))
        for d in range(8):
            nb = _neighbours(dims, d // 2, 1 - 2 * (d % 2), dev)
            xn = nb[xs]
            if dof == 12:
                mu, sgn = d // 2, 1 - 2 * (d % 2)
                G = D.U[mu][xs] if sgn > 0 else D.U[mu][xn].mH
                G = -0.5 * D.eta[mu, sgn][xs][:, None, None] * G
                H = (spin[d][None, :, None, :, None] * G[:, None, :, None, :]).reshape(-1, 12, 12)
            else:
                H = t['Y'][d][xs]
            T = torch.matmul(PH, torch.matmul(H, P[xn]))
            inside = (owner[xn] == owner[xs]).to(C128)
            X[c0:c0 + n] += block_sum(T, inside)
            Y[d, c0:c0 + n] += block_sum(T, 1 - inside)
    return {'X': X, 'Y': Y}


def _ptc(case, t, dims):
    D = _Dirac(t['U'], dims, M0)
    W1, W2 = (t[k].to(C128).requires_grad_(case['form'] == 'train') for k in ('W1', 'W2'))

    def layer(W, h):                    # W [9][out][in][4][4], h [in][V][4][3]
        out = 0
        for p in range(9):
            T = h if p == 0 else D.transport(h, (p - 1) // 2, 1 - 2 * ((p - 1) % 2))
            out = out + sum(D.spin(W[p, :, b, None], T[b]) for b in range(h.shape[0]))
        return out
    loss, ys = 0, []
    for r in t['r'].to(C128):
        y = layer(W2, layer(W1, r[None]))[0]
        if case['form'] == 'forward':
            ys.append(y)
            continue
        e = r - D.apply(y)
        loss = loss + (e.abs() ** 2).sum() / (r.abs() ** 2).sum()
    if case['form'] == 'forward':
        return ys
    loss.backward()
    return {'G1': W1.grad, 'G2': W2.grad, 'loss': loss.item()}
