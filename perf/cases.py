"""Performance cases: what a program that uses this library has it do, through paper_2608_14123_amd.binding.

Each case is one call (or the few calls that belong together) on a mesh, with the solver handle made
beforehand as a program keeps it.  The kinds:

  residual   r = g - A u on the finest level: the matrix-free operator by itself
  schwarz    z = B r on the finest level: the preconditioner inside another program's Krylov solver
  smooth     a few WAS or SCG smoothing steps from a given iterate
  transfers  projection, restriction and prolongation between the two finest levels
  vcycle     one FAS V-cycle from zero: the preconditioner call, and one step of a solve
  solve      a whole solve to a relative residual of 1e-10 from zero
  mlp        loss and gradient of the learned correction's network over one mini-batch

on box meshes (curved, Cartesian or stretched; odd and unequal extents; Dirichlet, Neumann or
periodic), the hp front with degrees 2..8, the unstructured diamond mesh and the locally refined
cube.  `exact` evaluates the same quantities in plain torch FP64 on the box meshes.
"""
import functools
import math

import numpy as np
import torch

from paper_2608_14123_amd import binding as B
from paper_2608_14123_amd import workloads as W

DEV = 'cuda'
F64 = torch.float64

# Options of a box case that are not written out.  A default is what most calls take.
BOX = dict(mesh='box', amp=0.0, lz=1.0, perturb=0.0, bc='dirichlet', kappa=0.0, nu='one', mu_star=5.0, overlap=1,
           delta=0.0, smoother='scg', ns1=3, ns2=2, root_rtol=0.1, root_max_iter=500, precision='fp64', n_rhs=1,
           graph=False, order='natural', h_levels=0, steps=1)


def listed():
    return [
        # The smallest whole solve: 4^3 unit cubes at p = 4, where every kernel is far below one wave
        # of the chip and launches, synchronisations and the root solve's iterations count.
        dict(name='solve_cart_p4_4', kind='solve', nx=4, ny=4, nz=4, p=4, smoother='was', ns1=2, ns2=2, mu_star=2.0,
             root_rtol=1e-12),
        # The operator by itself at the size of the curved benchmark (16.8M DOF): HBM bound at best.
        dict(name='residual_curved_p7_32', kind='residual', nx=32, ny=32, nz=32, p=7, amp=0.1),
        # The Schwarz preconditioner by itself at that size: FP64 contractions, gather and scatter.
        dict(name='schwarz_curved_p7_32', kind='schwarz', nx=32, ny=32, nz=32, p=7, amp=0.1),
        # The benchmark's step: one FP64 V-cycle with SCG(3,2) on levels p = 7, 3, 1.
        dict(name='vcycle_curved_p7_32', kind='vcycle', nx=32, ny=32, nz=32, p=7, amp=0.1),
        # Anisotropic elements need the wide overlap (three layers at p = 8, two at p = 4); several
        # right-hand sides share the geometry.  Odd extents.
        dict(name='smooth_stretched_p8_rhs4', kind='smooth', nx=15, ny=13, nz=17, p=8, lz=100.0, perturb=0.2,
             overlap=-1, delta=0.24, n_rhs=4, steps=4),
        # Time to solution in the fastest form measured: h-levels before the p-levels, FP32 smoothing.
        dict(name='solve_curved_p7_32_fp32', kind='solve', nx=32, ny=32, nz=32, p=7, amp=0.1, h_levels=2,
             precision='fp32'),
        # A middle-sized solve on the matrix cores, each cycle replayed as one HIP graph: the form for
        # a program that solves over and over.
        dict(name='solve_curved_p7_16_bf16', kind='solve', nx=16, ny=16, nz=16, p=7, amp=0.05, precision='bf16',
             graph=True, root_rtol=0.0, root_max_iter=16),
        # The hp-adaptive front (degrees 2..8, 3.2M DOF), autotuned launches and graph legs.
        dict(name='solve_front_27', kind='solve', mesh='front', nx=27),
        # The irregular periodic mesh (oriented faces, merged edges and vertices) at p = 4.
        dict(name='vcycle_diamond_p4_16', kind='vcycle', mesh='diamond', nx=16, nz=24, p=4, ns1=8, ns2=4),
        # Local refinement with full multigrid start: many small levels, composite residual.
        dict(name='solve_local_p7_16', kind='solve', mesh='local', nx=16, p=7),
        # Transfers of a p = 8 mesh to p = 4 and back.
        dict(name='transfers_curved_p8_24', kind='transfers', nx=24, ny=24, nz=24, p=8, amp=0.05),
        # One training step's gradient of the correction network at its p = 8 size.
        dict(name='mlp_gradient_p8_4096', kind='mlp', n_in=1340, n_hidden=256, n_out=1331, rows=4096),
    ]


def draw(rng):
    """One more case of the listed ranges: every degree, extents from 2 to about 40 elements a side (odd and
    unequal ones), the boundary conditions, precisions, batches and orders that programs choose between."""
    kind = rng.choice(['residual', 'residual', 'schwarz', 'schwarz', 'smooth', 'vcycle', 'vcycle', 'solve', 'solve',
                       'transfers', 'mlp'])
    if kind == 'mlp':
        p = rng.choice([5, 6, 7, 8])
        ns3 = (p + 3) ** 3
        return dict(kind='mlp', n_in=ns3 + 9, n_hidden=rng.choice([64, 128, 192, 256]), n_out=ns3,
                    rows=int(round(math.exp(rng.uniform(math.log(64), math.log(4096))))))
    if kind in ('vcycle', 'solve') and rng.random() < 0.2:
        if kind == 'solve':
            return dict(kind='solve', mesh='front', nx=rng.randint(7, 27))
        return dict(kind='vcycle', mesh='diamond', nx=rng.randint(3, 12), nz=rng.randint(4, 16), p=rng.randint(2, 6),
                    ns1=rng.randint(3, 8), ns2=rng.randint(2, 4))
    p = rng.randint(2 if kind in ('transfers', 'vcycle', 'solve') else 1, 8)
    top = {'residual': 1.6e7, 'schwarz': 1.6e7, 'transfers': 1e7, 'smooth': 6e6, 'vcycle': 6e6, 'solve': 2.5e6}[kind]
    dof = math.exp(rng.uniform(math.log(5e3), math.log(top)))
    side = (dof / (p + 1) ** 3) ** (1.0 / 3.0)
    ext = [max(2, min(40, int(round(side * rng.uniform(0.7, 1.4))))) for _ in range(3)]
    c = dict(kind=kind, nx=ext[0], ny=ext[1], nz=ext[2], p=p, amp=rng.choice([0.0, 0.01, 0.02, 0.03]))
    c['bc'] = rng.choice(['dirichlet', 'dirichlet', 'neumann', 'periodic'])
    if c['bc'] == 'periodic':
        c.update(nx=max(3, c['nx']), ny=max(3, c['ny']), nz=max(3, c['nz']))
    c['kappa'] = 0.0 if c['bc'] == 'dirichlet' and rng.random() < 0.6 else round(rng.uniform(0.2, 2.0), 3)
    if kind in ('residual', 'schwarz') and rng.random() < 0.3:
        c['nu'] = 'smooth'
    if kind != 'solve':
        c['order'] = rng.choice(['natural', 'natural', 'morton'])
        if rng.random() < 0.3 and dof < top / 4:
            c['n_rhs'] = rng.randint(2, 4)
    if p in (4, 8) and rng.random() < 0.3:
        c.update(overlap=-1, delta=0.24)
    if kind == 'smooth':
        c['steps'] = rng.randint(1, 4)
        c['smoother'] = rng.choice(['was', 'scg', 'scg'])
    if kind == 'solve':
        c['precision'] = rng.choice(['fp64', 'fp32', 'bf16', 'fp32_mfma'])
        if rng.random() < 0.5:
            c.update(graph=True, root_rtol=0.0, root_max_iter=rng.randint(16, 24))
    return c


def full(case):
    return {**BOX, **case}


# ---- what a program has before the call -----------------------------------------------------------

def generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def uniform(n, g):
    return torch.rand(n, generator=g, device=DEV, dtype=F64) * 2.0 - 1.0


def box_coords(c, xi):
    """(E, 3, n, n, n) coordinates at the tensor points xi: a trilinear box grid on [0,1]^2 x [0,lz] with
    interior vertices displaced by up to `perturb` times the shortest edge, then the sine bump of `amp`."""
    xi = torch.as_tensor(np.asarray(xi), device=DEV, dtype=F64)
    ext = (c['nx'], c['ny'], c['nz'])
    length = (1.0, 1.0, c['lz'])
    ax = [torch.arange(m + 1, device=DEV, dtype=F64) / m * l for m, l in zip(ext, length)]
    V = torch.stack(torch.broadcast_tensors(ax[0][None, None, :], ax[1][None, :, None], ax[2][:, None, None]), -1).clone()
    if c['perturb']:
        h = min(l / m for m, l in zip(ext, length))
        d = torch.from_numpy(np.random.default_rng(4).uniform(-1, 1, size=tuple(V.shape))).to(DEV) * (c['perturb'] * h)
        V[1:-1, 1:-1, 1:-1] += d[1:-1, 1:-1, 1:-1]
    lo, hi = 0.5 * (1 - xi), 0.5 * (1 + xi)
    for dim in (2, 1, 0):                  # x, y, z: (.., m+1, ..) -> (.., m, .., n)
        a, b = V.narrow(dim, 0, V.shape[dim] - 1), V.narrow(dim, 1, V.shape[dim] - 1)
        V = a.unsqueeze(-1) * lo + b.unsqueeze(-1) * hi
    X = V.permute(0, 1, 2, 3, 6, 5, 4)     # (ez, ey, ex, coord, k, j, i)
    X = X.reshape((-1, 3) + (len(xi),) * 3)
    if c['amp']:
        s = torch.sin(2 * math.pi * X[:, 0]) * torch.sin(2 * math.pi * X[:, 1]) * torch.sin(2 * math.pi * X[:, 2])
        X = X + c['amp'] * s[:, None]
    return X.contiguous()


def box_nu(c, X):
    """Nodal diffusivity between 1/2 and 3/2, or None."""
    if c['nu'] == 'one':
        return None
    return 1.0 + 0.5 * torch.cos(math.pi * X[:, 0]) * torch.cos(math.pi * X[:, 1]) * torch.cos(math.pi * X[:, 2])


def stream():
    return torch.cuda.current_stream().cuda_stream


def box_solver(c):
    X = box_coords(c, B.gll(c['p'])[0])
    nbr, bc = W.box_topology(c['nx'], c['ny'], c['nz'], periodic=(c['bc'] == 'periodic',) * 3,
                             bc_code=W.NEUMANN if c['bc'] == 'neumann' else W.DIRICHLET)
    nu = box_nu(c, X)
    o = B.default_options(kappa=c['kappa'], mu_star=c['mu_star'], overlap=c['overlap'], delta=c['delta'],
                          smoother=B.SCG if c['smoother'] == 'scg' else B.WAS, ns1=c['ns1'], ns2=c['ns2'],
                          root_rtol=c['root_rtol'], root_max_iter=c['root_max_iter'], n_rhs=c['n_rhs'],
                          precision={'fp64': B.FP64, 'fp32': B.FP32, 'bf16': B.BF16, 'fp32_mfma': B.FP32_MFMA}[c['precision']],
                          graph=int(c['graph']), order=B.ORDER_MORTON if c['order'] == 'morton' else B.ORDER_NATURAL,
                          h_levels=c['h_levels'])
    return B.Solver(np.full(len(X), c['p'], np.int32), X.cpu().numpy(), nbr, bc, o, stream=stream(),
                    box=(c['nx'], c['ny'], c['nz']) if c['h_levels'] else None,
                    nu=None if nu is None else nu.cpu().numpy())


@functools.lru_cache(maxsize=1)
def front_mesh(ne):
    """The hp front's mesh: degrees and, per element, coordinates at its own degree's nodes."""
    deg = W.front_degrees(ne)
    nbr, bc = W.box_topology(ne, ne, ne)
    V = W.box_vertices(ne, ne, ne)
    off = np.concatenate(([0], np.cumsum((deg.astype(np.int64) + 1) ** 3)))
    X = np.empty(3 * off[-1])
    P = np.empty((3, off[-1]))              # the same coordinates in the order of a solution vector
    for p in np.unique(deg):
        sel = np.nonzero(deg == p)[0]
        n3 = int(p + 1) ** 3
        C = W.element_coords(V, B.gll(int(p))[0])[sel].reshape(len(sel), 3, n3)
        at = off[sel][:, None] + np.arange(n3)
        for a in range(3):
            P[a, at] = C[:, a]
            X[3 * off[sel][:, None] + a * n3 + np.arange(n3)] = C[:, a]
    return deg, X, nbr, bc, P


@functools.lru_cache(maxsize=1)
def diamond_mesh(nc, layers, p):
    X = W.diamond_coords(nc, layers, B.gll(p)[0], length=2 * np.pi, height=2 * np.pi, shift_seed=1, rot_seed=2)
    return (X,) + W.face_connectivity(X, period=2 * np.pi)


@functools.lru_cache(maxsize=1)
def local_zones(ne):
    return W.local_refine_lists(ne, [((0.5, 0.5, 0.5), 0.3), ((0.5, 0.5, 0.5), 0.15)])


def front_state(c, seed):
    deg, X, nbr, bc, P = front_mesh(c['nx'])
    s = B.Solver(deg, X, nbr, bc, B.default_options(smoother=B.SCG, ns1=3, ns2=2, root_rtol=0.1, batch=B.BATCH_TUNED,
                                                    graph=1), stream=stream())
    s.autotune(None, reps=5)
    # the front has moved a little since the degrees were chosen
    x = torch.from_numpy(P).to(DEV)
    r0 = 0.7 + (torch.rand(1, generator=generator(seed), device=DEV, dtype=F64) - 0.5) * 0.25 / c['nx']
    rho = torch.sqrt((x * x).sum(0)).clamp_min(1e-6)
    t = 50.0 * (rho - r0)
    f = 2.0 * 50.0 ** 3 * (rho - r0) / (1 + t * t) ** 2 - 2.0 * 50.0 / (1 + t * t) / rho
    b = torch.empty_like(f)
    s.rhs(f, b, uD=torch.atan(t))
    return dict(solver=s, f=b, u=torch.zeros_like(b))


def diamond_state(c, seed):
    X, nbr, nf, no, bc = diamond_mesh(c['nx'], c['nz'], c['p'])
    s = B.Solver(np.full(len(X), c['p'], np.int32), X, nbr, bc,
                 B.default_options(kappa=0.0, null_space=1, mu_star=5.0, root_rtol=0.1, smoother=B.SCG, ns1=c['ns1'],
                                   ns2=c['ns2']), stream=stream(), nbr_face=nf, nbr_orient=no)
    f = uniform(s.level_info(s.n_levels)[1], generator(seed))
    f -= f.mean()
    return dict(solver=s, f=f, u=torch.zeros_like(f))


def local_state(c, seed):
    ne, p = c['nx'], c['p']
    refine = local_zones(ne)
    X = box_coords(full(dict(nx=ne, ny=ne, nz=ne, amp=0.1)), B.gll(p)[0])
    nbr, bc = W.box_topology(ne, ne, ne)
    s = B.Solver(np.full(ne ** 3, p, np.int32), X.cpu().numpy(), nbr, bc,
                 B.default_options(local_steps=len(refine), mu_star=5.0, root_rtol=0.1, smoother=B.SCG, ns1=3, ns2=2,
                                   start=B.START_FMG), stream=stream(), refine=refine)
    centre = 0.5 + 0.1 * uniform(3, generator(seed))        # a localised source inside the zones
    for l in range(1, s.n_levels + 1):
        x = torch.from_numpy(s.level_coords(l)).to(DEV)
        f = torch.exp(-50.0 * ((x - centre[None, :, None, None, None]) ** 2).sum(1)).reshape(-1).contiguous()
        b = torch.empty_like(f)
        s.level_rhs(l, f, b)
        if l < s.n_levels:
            s.set_level_rhs(l, b)
    return dict(solver=s, f=b, u=torch.zeros_like(b))


def mlp_inputs(c, seed):
    """Unit subdomain residuals with the element's nine metric entries, and small corrections of them;
    He-normal weights as a program loads them."""
    g = generator(seed)
    i, h, o, rows = c['n_in'], c['n_hidden'], c['n_out'], c['rows']
    X = torch.randn(rows, i, generator=g, device=DEV)
    X[:, :-9] /= X[:, :-9].norm(dim=1, keepdim=True)
    T = torch.randn(rows, o, generator=g, device=DEV) * (0.07 / math.sqrt(o))
    ws = []
    for a, b in ((i, h), (h, h), (h, o)):
        ws += [torch.randn(a * b, generator=g, device=DEV) * math.sqrt(2.0 / a),
               torch.randn(b, generator=g, device=DEV) * 0.01]
    return X, T, torch.cat(ws)


def box_vectors(c, n, seed):
    """Nodal data U[-1, 1], as the benchmark's right-hand side."""
    g = generator(seed)
    return uniform(n, g), uniform(n, g)


def prepare(case, seed):
    c = full(case)
    if c['kind'] == 'mlp':
        X, T, theta = mlp_inputs(c, seed)
        net = B.Mlp(c['n_in'], c['n_hidden'], c['n_out'], seed=5, stream=stream())
        net.set_params(theta.cpu().numpy())
        return dict(kind='mlp', net=net, X=X, T=T, grad=torch.empty(net.n_params, device=DEV))
    if c['mesh'] != 'box':
        s = {'front': front_state, 'diamond': diamond_state, 'local': local_state}[c['mesh']](c, seed)
        return dict(s, kind=c['kind'], exact_hist=True)
    s = box_solver(c)
    L = s.n_levels
    n = c['n_rhs'] * s.level_info(L)[1]
    a, b = box_vectors(c, n, seed)
    st = dict(kind=c['kind'], solver=s, exact_hist=c['precision'] == 'fp64')
    if c['kind'] == 'residual':
        st.update(u=a, g=b, r=torch.empty_like(a))
    elif c['kind'] == 'schwarz':
        st.update(r=a, z=torch.empty_like(a))
    elif c['kind'] == 'smooth':
        st.update(u0=a, g=b, u=torch.empty_like(a), steps=c['steps'])
    elif c['kind'] == 'transfers':
        nc = c['n_rhs'] * s.level_info(L - 1)[1]
        st.update(u0=a, r=b, u=torch.empty_like(a), uc=torch.empty(nc, device=DEV, dtype=F64),
                  rc=torch.empty(nc, device=DEV, dtype=F64))
    else:
        f = torch.empty_like(a)
        s.rhs(a, f)
        st.update(f=f, u=torch.zeros_like(f))
    return st


def run(state):
    kind = state['kind']
    if kind == 'mlp':
        loss = state['net'].gradient(state['X'], state['T'], state['grad'])
        return dict(loss=loss, grad=state['grad'])
    s = state['solver']
    L = s.n_levels
    if kind == 'residual':
        s.residual(L, state['u'], state['g'], state['r'])
        return state['r']
    if kind == 'schwarz':
        s.schwarz(L, state['r'], state['z'])
        return state['z']
    u = state['u']
    if kind == 'smooth':
        u.copy_(state['u0'])
        s.smooth(L, u, state['g'], state['steps'])
        return u
    if kind == 'transfers':
        u.copy_(state['u0'])
        s.project(L, u, state['uc'])
        s.restrict(L, state['r'], state['rc'])
        s.prolong_add(L, state['rc'], u, ubar=state['uc'])
        return dict(uc=state['uc'], rc=state['rc'], u=u)
    u.zero_()
    if kind == 'vcycle':
        s.vcycle(u, state['f'])
        return u
    hist, ok = s.solve(u, state['f'], max_cycles=60, rtol=1e-10)
    # with a reduced-precision smoother the history's last digits are that precision's
    return dict(u=u, hist=hist) if state['exact_hist'] else u


# ---- the work a pass cannot do without -------------------------------------------------------------

# cycles to 1e-10 that the configurations take; draws of other sizes take about ten
CYCLES = {'solve_cart_p4_4': 7, 'solve_curved_p7_32_fp32': 16, 'solve_front_27': 12, 'solve_local_p7_16': 20}


def work(case):
    """Operator: u, g, r and the coordinates once (48 bytes a DOF in FP64) and the 1D contractions; Schwarz:
    r and z once and the subdomain contractions; a smoothing step is both with the update (72 bytes, half of
    it in FP32); a cycle is its steps and two residuals on every level (the levels below hold about an
    eighth of the DOF); a solve its cycles."""
    c = full(case)
    if c['kind'] == 'mlp':
        i, h, o, rows = c['n_in'], c['n_hidden'], c['n_out'], c['rows']
        flops = 2.0 * rows * (2 * i * h + 3 * h * h + 3 * h * o)
        return dict(bytes=4.0 * (rows * (i + o) + 2 * (i * h + h * h + h * o)), flops=flops)
    if c['mesh'] == 'front':
        deg = W.front_degrees(c['nx']).astype(np.int64)
        dof, p = float(((deg + 1) ** 3).sum()), 8
    elif c['mesh'] == 'diamond':
        p = c['p']
        dof = 5.0 * c['nx'] ** 2 * c['nz'] * (p + 1) ** 3
    elif c['mesh'] == 'local':
        p = c['p']
        dof = 2.45 * c['nx'] ** 3 * (p + 1) ** 3           # base and the two zones' active elements
    else:
        p = c['p']
        dof = float(c['n_rhs'] * c['nx'] * c['ny'] * c['nz'] * (p + 1) ** 3)
    n = p + 1
    ns = n + 2
    op = 12.0 * n + 40
    sz = (12.0 * ns + 1) * (ns / n) ** 3
    if c['kind'] == 'residual':
        return dict(bytes=48 * dof, flops=op * dof)
    if c['kind'] == 'schwarz':
        return dict(bytes=16 * dof, flops=sz * dof)
    step = 36.0 if c['precision'] != 'fp64' else 72.0
    if c['kind'] == 'smooth':
        return dict(bytes=c['steps'] * step * dof, flops=c['steps'] * (op + sz) * dof)
    if c['kind'] == 'transfers':
        m = max(1, p // 2) + 1
        return dict(bytes=8 * dof * (4 + 2 * (m / n) ** 3), flops=12.0 * m * dof)
    sweeps = c['ns1'] + c['ns2']
    cycles = 1 if c['kind'] == 'vcycle' else CYCLES.get(c.get('name'), 10)
    return dict(bytes=cycles * 1.14 * dof * (sweeps * step + 96), flops=cycles * 1.14 * dof * sweeps * (op + sz))


# ---- the same in plain FP64 on the box meshes ------------------------------------------------------

def gll(p):
    """Gauss-Lobatto-Legendre nodes and weights."""
    c = np.zeros(p + 1)
    c[p] = 1.0
    d = np.polynomial.legendre.legder(c)
    x = np.concatenate(([-1.0], np.sort(np.polynomial.legendre.legroots(d).real) if p > 1 else [], [1.0]))
    for _ in range(3):                       # Newton on P_p' inside, P_p'' from Legendre's equation
        P, dP = (np.polynomial.legendre.legval(x[1:-1], v) for v in (c, d))
        x[1:-1] -= dP / ((2 * x[1:-1] * dP - p * (p + 1) * P) / (1 - x[1:-1] ** 2))
    return x, 2.0 / (p * (p + 1) * np.polynomial.legendre.legval(x, c) ** 2)


def lagrange(x, y):
    L = np.ones((len(y), len(x)))
    for j in range(len(x)):
        for m in range(len(x)):
            if m != j:
                L[:, j] *= (y - x[m]) / (x[j] - x[m])
    return L


def diff_matrix(p):
    x, _ = gll(p)
    P = np.polynomial.legendre.legval(x, np.eye(p + 1)[p])
    with np.errstate(divide='ignore', invalid='ignore'):
        D = P[:, None] / (P[None, :] * (x[:, None] - x[None, :]))
    D[np.arange(p + 1), np.arange(p + 1)] = 0.0
    D[0, 0], D[p, p] = -p * (p + 1) / 4.0, p * (p + 1) / 4.0
    return D


def along(M, u, d):
    """M applied along direction d (0: last axis) of u[..., k, j, i]."""
    return torch.movedim(torch.movedim(u, -1 - d, -1) @ M.T, -1, -1 - d)


def tensor3(M, u):
    return along(M, along(M, along(M, u, 0), 1), 2)


def sipg_1d(p, mu_star, left, right, elements):
    """1D SIPG mass and stiffness on `elements` elements of length 2; ends 'd' Dirichlet or 'n' natural."""
    n, D = p + 1, diff_matrix(p)
    _, w = gll(p)
    N = elements * n
    L, M = np.zeros((N, N)), np.tile(w, elements)
    mu = mu_star * p * (p + 1) / 4.0
    for e in range(elements):
        L[e * n:(e + 1) * n, e * n:(e + 1) * n] += D.T @ np.diag(w) @ D
    for e in range(elements - 1):
        J, A = np.zeros(N), np.zeros(N)
        J[e * n + p], J[(e + 1) * n] = 1.0, -1.0
        A[e * n:(e + 1) * n] = 0.5 * D[p]
        A[(e + 1) * n:(e + 2) * n] = 0.5 * D[0]
        L += mu * np.outer(J, J) - np.outer(A, J) - np.outer(J, A)
    for end, at, row, s in ((left, 0, slice(0, n), -1.0), (right, N - 1, slice(N - n, N), 1.0)):
        if end == 'd':
            v, g = np.zeros(N), np.zeros(N)
            v[at], g[row] = 1.0, s * D[p if s > 0 else 0]
            L += 2 * mu * np.outer(v, v) - np.outer(v, g) - np.outer(g, v)
    return M, L


def subdomain_1d(p, m, mu_star, left, right):
    """Offsets of the subdomain's nodes from the element's first, eigenvectors, eigenvalues and weights."""
    n = p + 1
    lo, hi = left == 'i', right == 'i'
    M, L = sipg_1d(p, mu_star, 'd' if left == 'd' else 'n', 'd' if right == 'd' else 'n', 1 + lo + hi)
    off = np.arange(-m if lo else 0, n + (m if hi else 0))
    at = off + (n if lo else 0)
    s = 1.0 / np.sqrt(M[at])
    lam, Q = np.linalg.eigh(s[:, None] * L[np.ix_(at, at)] * s[None, :])
    x, _ = gll(p)
    Wt = np.ones(len(off))
    if m > 0:
        a = 0.5 * (1 + x[m])
        where = np.floor_divide(off, n) + 0.5 * (1 + x[off % n])       # in elements, 0 and 1 the faces
        for on, d in ((lo, where), (hi, 1.0 - where)):
            if on:
                t = np.clip((d + a) / (2 * a), 0, 1)
                Wt *= np.where(np.abs(d) < 1.0, 10 * t ** 3 - 15 * t ** 4 + 6 * t ** 5, 1.0)
    as_t = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to(DEV)  # noqa: E731
    return as_t(off), as_t(s[:, None] * Q), as_t(lam), as_t(Wt)


class Level:
    """One level of a box mesh: the operator A and the Schwarz method S on arrays (nz, ny, nx, n, n, n)."""

    def __init__(self, c, p, X, nu):
        self.c, self.p, self.n = c, p, p + 1
        self.grid = (c['nz'], c['ny'], c['nx'])
        n, g = self.n, self.grid
        x, w = gll(p)
        self.x, self.X, self.nu = x, X, nu
        self.D = torch.from_numpy(diff_matrix(p)).to(DEV)
        self.w_end = float(w[0])
        wt = torch.from_numpy(w).to(DEV)
        w3 = wt[:, None, None] * wt[None, :, None] * wt[None, None, :]
        J = [[along(self.D, X[:, a], b).reshape(g + (n,) * 3) for b in range(3)] for a in range(3)]
        cof = [[J[(a + 1) % 3][(b + 1) % 3] * J[(a + 2) % 3][(b + 2) % 3]
                - J[(a + 1) % 3][(b + 2) % 3] * J[(a + 2) % 3][(b + 1) % 3] for b in range(3)] for a in range(3)]
        det = sum(J[0][b] * cof[0][b] for b in range(3))
        nun = torch.ones_like(det) if nu is None else nu.reshape(det.shape)
        self.wj = w3 * det
        self.G = [[w3 * nun / det * sum(cof[a][b] * cof[a][d] for a in range(3)) for d in range(3)] for b in range(3)]
        vol = self.wj.sum((3, 4, 5))
        periodic = c['bc'] == 'periodic'
        self.side = ('i', 'i') if periodic else (('n', 'n') if c['bc'] == 'neumann' else ('d', 'd'))
        ws, own = {}, {}
        for ax in range(3):
            for s in (0, 1):
                t = [self.layer(torch.sqrt(sum(cof[a][ax] ** 2 for a in range(3))), ax, s)]
                o = wt[:, None] * wt[None, :]
                ws[ax, s] = t[0] * o
                own[ax, s] = p * (p + 1) / 2.0 * ws[ax, s].sum((3, 4)) / vol
        self.pen, self.inner = {}, {}
        for ax in range(3):
            for s in (0, 1):
                inner = torch.ones(g, device=DEV, dtype=torch.bool)
                if not periodic:
                    inner.select(2 - ax, -1 if s else 0).fill_(False)
                self.inner[ax, s] = inner[..., None, None]
                oth = own[ax, 1 - s].roll(-1 if s else 1, 2 - ax)
                nuo = self.layer(nun, ax, s)
                nub = torch.maximum(nuo, self.layer(nun, ax, 1 - s).roll(-1 if s else 1, 2 - ax))
                mu = c['mu_star']
                self.pen[ax, s] = torch.where(self.inner[ax, s], (mu * 0.5 * (own[ax, s] + oth))[..., None, None] * nub,
                                              2 * mu * own[ax, s][..., None, None] * nuo) * ws[ax, s]
        # surrogate cuboid: linear Legendre coefficients of the map, scaled to the element's volume
        ell = []
        for b in range(3):
            shape = [1, 1, 1]
            shape[2 - b] = n
            if p == 1:
                v = torch.from_numpy(np.array([-0.5, 0.5])).to(DEV).reshape(shape) * 0.25
            else:
                v = 0.375 * w3 * torch.from_numpy(x).to(DEV).reshape(shape)
            ell.append(2 * torch.sqrt(sum((X[:, a] * v).sum((1, 2, 3)) ** 2 for a in range(3))).reshape(g))
        sc = (vol / (ell[0] * ell[1] * ell[2])) ** (1.0 / 3.0)
        d = [e * sc for e in ell]
        nue = (self.wj * nun).sum((3, 4, 5)) / vol
        self.g = [c['kappa'] * d[0] * d[1] * d[2] / 8] + [nue * d[(b + 1) % 3] * d[(b + 2) % 3] / (2 * d[b]) for b in range(3)]
        if c['overlap'] >= 0:
            self.m = min(c['overlap'], p)
        else:
            self.m = min(p, int(np.sum(0.5 * (1 + x) <= c['delta'] + 1e-14)))
        self.sub = {}

    def layer(self, V, ax, s):
        return V.select(-1 - ax, self.n - 1 if s else 0)

    def A(self, u):
        u = u.reshape(self.grid + (self.n,) * 3)
        d = [along(self.D, u, b) for b in range(3)]
        F = [sum(self.G[b][a] * d[a] for a in range(3)) for b in range(3)]
        del d
        lift = [f.clone() for f in F]
        out = self.c['kappa'] * self.wj * u
        for ax in range(3):
            for s in (0, 1):
                sg = 1.0 if s else -1.0
                to = -1 if s else 1
                uo = self.layer(u, ax, s)
                qo = sg / self.w_end * self.layer(F[ax], ax, s)
                un = self.layer(u, ax, 1 - s).roll(to, 2 - ax)
                qn = sg / self.w_end * self.layer(F[ax], ax, 1 - s).roll(to, 2 - ax)
                inner, pen = self.inner[ax, s], self.pen[ax, s]
                edge_row, edge_sig = (pen * uo - qo, -uo) if self.side[s] == 'd' else (0 * uo, 0 * uo)
                row = torch.where(inner, pen * (uo - un) - 0.5 * (qo + qn), edge_row)
                sig = torch.where(inner, -0.5 * (uo - un), edge_sig)
                self.layer(out, ax, s).add_(row)
                for a in range(3):
                    self.layer(lift[a], ax, s).add_(sig * sg / self.w_end * self.layer(self.G[ax][a], ax, s))
        for a in range(3):
            out += along(self.D.T, lift[a], a)
        return out.reshape(-1)

    def groups(self, ax):
        """Elements along an axis that share a 1D subdomain: (first, last + 1, left, right)."""
        e = self.grid[2 - ax]
        l, r = self.side
        if l == 'i':
            return [(0, e, 'i', 'i')]
        if e == 1:
            return [(0, 1, l, r)]
        return [(0, 1, l, 'i'), (1, e - 1, 'i', 'i'), (e - 1, e, 'i', r)]

    def S(self, r):
        n, g = self.n, self.grid
        R = r.reshape(g + (n,) * 3).permute(0, 3, 1, 4, 2, 5).reshape(g[0] * n, g[1] * n, g[2] * n)
        Z = torch.zeros_like(R)
        for gz in self.groups(2):
            for gy in self.groups(1):
                for gx in self.groups(0):
                    if min(q[1] - q[0] for q in (gx, gy, gz)) <= 0:
                        continue
                    for z0 in range(gz[0], gz[1], 8):       # in slabs, for memory
                        self.solve_group(R, Z, gx, gy, (z0, min(gz[1], z0 + 8)) + gz[2:])
        return Z.reshape(g[0], n, g[1], n, g[2], n).permute(0, 2, 4, 1, 3, 5).reshape(-1)

    def solve_group(self, R, Z, gx, gy, gz):
        n = self.n
        one, idx = [], []
        for ax, q in enumerate((gx, gy, gz)):
            if q[2:] not in self.sub:
                self.sub[q[2:]] = subdomain_1d(self.p, self.m, self.c['mu_star'], q[2], q[3])
            one.append(self.sub[q[2:]])
            e = torch.arange(q[0], q[1], device=DEV)
            idx.append((e[:, None] * n + one[-1][0][None, :]) % R.shape[2 - ax])
        ix, iy, iz = idx
        t = R[iz[:, None, None, :, None, None], iy[None, :, None, None, :, None], ix[None, None, :, None, None, :]]
        for d in range(3):
            t = along(one[d][1].T, t, d)
        co = [v[gz[0]:gz[1], gy[0]:gy[1], gx[0]:gx[1], None, None, None] for v in self.g]
        t = t / (co[0] + co[1] * one[0][2] + co[2] * one[1][2][:, None] + co[3] * one[2][2][:, None, None])
        for d in range(3):
            t = along(one[d][1], t, d)
        t = t * one[0][3] * one[1][3][:, None] * one[2][3][:, None, None]
        # overlapping sums, one direction at a time
        a, b, cc, sz, sy, sx = t.shape
        t = torch.zeros((a, b, sz, sy, R.shape[2]), device=DEV, dtype=F64).index_add_(
            4, ix.reshape(-1), t.permute(0, 1, 3, 4, 2, 5).reshape(a, b, sz, sy, cc * sx))
        t = torch.zeros((a, sz, R.shape[1], R.shape[2]), device=DEV, dtype=F64).index_add_(
            2, iy.reshape(-1), t.permute(0, 2, 1, 3, 4).reshape(a, sz, b * sy, R.shape[2]))
        Z.index_add_(0, iz.reshape(-1), t.reshape(a * sz, R.shape[1], R.shape[2]))

    def smooth(self, u, f, steps, smoother):
        if smoother == 'was':
            for _ in range(steps):
                u = u + self.S(f - self.A(u))
            return u
        return self.scg(u, f, steps)

    def scg(self, u, f, steps, stop=0.0):
        """Schwarz-preconditioned CG with the flexible beta, from u, to |r| <= stop."""
        r = f - self.A(u)
        for i in range(steps):
            z = self.S(r)
            if i == 0:
                p = z
            else:
                p = z + (z @ (r - r0)) / gamma * p
            gamma = z @ r
            q = self.A(p)
            alpha = gamma / (p @ q)
            u = u + alpha * p
            r0, r = r, r - alpha * q
            if stop and float(r.norm()) <= stop:
                break
        return u


def box_levels(c):
    """Levels of a box case, the finest first."""
    p = c['p']
    X = box_coords(c, gll(p)[0])
    nu = box_nu(c, X)
    out = [Level(c, p, X, nu)]
    while p > 1:
        q = max(1, p // 2)
        T = torch.from_numpy(lagrange(gll(p)[0], gll(q)[0])).to(DEV)
        X, nu = tensor3(T, X), None if nu is None else tensor3(T, nu)
        out.append(Level(c, q, X, nu))
        out[-2].P = T
        out[-2].I = torch.from_numpy(lagrange(gll(q)[0], gll(p)[0])).to(DEV)
        p = q
    return out


def transfer(M, u, n):
    return tensor3(M, u.reshape((-1,) + (n,) * 3)).reshape(-1)


def cycle(c, lv, k, u, f):
    L = lv[k]
    if k == len(lv) - 1:
        r = float((f - L.A(u)).norm())
        return L.scg(u, f, c['root_max_iter'], c['root_rtol'] * r) if c['root_rtol'] else L.scg(u, f, c['root_max_iter'])
    u = L.smooth(u, f, c['ns1'], c['smoother'])
    ub = transfer(L.P, u, L.n)
    g = lv[k + 1].A(ub) + transfer(L.I.T, f - L.A(u), L.n)
    v = cycle(c, lv, k + 1, ub, g)
    u = u + transfer(L.I, v - ub, lv[k + 1].n)
    return L.smooth(u, f, c['ns2'], c['smoother'])


def exact(case, seed):
    c = full(case)
    if c['kind'] == 'mlp':
        X, T, th = (v.double() for v in mlp_inputs(c, seed))
        i, h, o = c['n_in'], c['n_hidden'], c['n_out']
        th = th.requires_grad_(True)
        W1, b1, W2, b2, W3, b3 = torch.split(th, [i * h, h, h * h, h, h * o, o])
        y = torch.relu(torch.relu(X @ W1.view(i, h) + b1) @ W2.view(h, h) + b2) @ W3.view(h, o) + b3
        loss = ((y - T) ** 2).mean()
        loss.backward()
        return dict(loss=float(loss.detach()), grad=th.grad)
    if c['mesh'] != 'box':
        return None
    ndof = c['nx'] * c['ny'] * c['nz'] * (c['p'] + 1) ** 3
    # a solve's answer is the solution itself: iterated to rounding where that is quick
    if c['kind'] == 'solve' and ndof > 60000:
        return None
    n = c['n_rhs'] * ndof
    a, b = box_vectors(c, n, seed)
    if c['kind'] in ('residual', 'schwarz', 'smooth', 'transfers'):
        lv = box_levels(c)[:2] if c['kind'] == 'transfers' else [Level(c, c['p'], *(lambda X: (X, box_nu(c, X)))(
            box_coords(c, gll(c['p'])[0])))]
    else:
        lv = box_levels(c)
    L, outs = lv[0], []
    for k in range(c['n_rhs']):
        x, y = a[k * ndof:(k + 1) * ndof], b[k * ndof:(k + 1) * ndof]
        if c['kind'] == 'residual':
            outs.append(y - L.A(x))
        elif c['kind'] == 'schwarz':
            outs.append(L.S(x))
        elif c['kind'] == 'smooth':
            outs.append(L.smooth(x, y, c['steps'], c['smoother']))
        elif c['kind'] == 'transfers':
            uc, rc = transfer(L.P, x, L.n), transfer(L.I.T, y, L.n)
            outs.append((uc, rc, x + transfer(L.I, rc - uc, lv[1].n)))
        else:
            f = L.wj.reshape(-1) * x
            if c['kind'] == 'vcycle':
                outs.append(cycle(c, lv, 0, torch.zeros_like(f), f))
            else:
                u = torch.zeros_like(f)
                for _ in range(60):
                    u = cycle(dict(c, smoother='scg', ns1=3, ns2=2, root_rtol=1e-6, root_max_iter=500), lv, 0, u, f)
                    if float((f - L.A(u)).norm()) <= 1e-13 * float(f.norm()):
                        break
                outs.append(u)
    if c['kind'] == 'transfers':
        uc, rc, u = (torch.cat(v) for v in zip(*outs))
        return dict(uc=uc, rc=rc, u=u)
    u = torch.cat(outs)
    return dict(u=u, hist=None) if c['kind'] == 'solve' and c['precision'] == 'fp64' else u
