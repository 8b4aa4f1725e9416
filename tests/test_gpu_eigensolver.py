"""GPU eigensolver (RMM-DIIS step, filter, block stop) against the oracle's
step, and converged eigenvalues against the exact discrete spectra."""
import numpy as np
import pytest

import synthetic
from oracle import hamiltonian, linalg, rmmdiis

torch = pytest.importorskip("torch")
import paper_1306_2953_amd as rsd  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"


def _setup(w, N, B, dtype=np.float64, **kw):
    og, atoms, H = hamiltonian.build_system(w)
    g = rsd.Grid.for_workload(w)
    nl = None
    if atoms is not None:
        nl = rsd.NonLocal(g, atoms.pos, atoms.D, w.rc, w.sigma, max_states=-(-N // B) * B)
    v = torch.from_numpy(H.vloc.astype(dtype)).to(DEV)
    solver = rsd.Eigensolver(g, nl, v, N, B, **kw)
    psi = synthetic.draw_states(synthetic.rng_after_atoms(w), N, og.np)
    psi, _, _ = linalg.orthonormalize(psi, og.dv)
    return og, H, g, solver, psi


@pytest.mark.parametrize("m", [1, 2, 3])
def test_one_step_matches_oracle(m):
    """The same step on the same orthonormal input: eigenvalues, residual norms
    and the updated states agree with the oracle's implementation."""
    w = synthetic.make_workload("sphere_r12_h0.2", radius=2.4, nat=3, atom_radius=1.2)
    N, B = 16, 8
    og, H, g, solver, psi = _setup(w, N, B, m=m, tol=1e-12)
    # a few oracle steps first so the states are not random noise
    opts = rmmdiis.Options(m=m, block=B, tol=1e-12)
    for _ in range(3):
        psi = rmmdiis.rmmdiis_step(H, psi, opts)["psi"]
    want = rmmdiis.rmmdiis_step(H, psi, opts)
    t = torch.from_numpy(rsd.to_blocks(psi, B)).to(DEV)
    eig, res, nconv = solver.step(t)
    got = rsd.from_blocks(t.cpu().numpy())
    assert np.max(np.abs(eig - want["eig"])) < 1e-12 * np.max(np.abs(want["eig"]))
    assert np.max(np.abs(res - want["resnorm"])) < 1e-10 * np.max(want["resnorm"])
    assert np.max(np.abs(got - want["psi"])) < 1e-10 * np.max(np.abs(want["psi"]))


# the field kernels' edges: one and two states a block, a last block of
# padding states, fewer columns than a reduction's 8, a grid whose rows end
# inside a thread's four values
@pytest.mark.parametrize("N,B,radius", [(5, 1, 2.0), (7, 2, 2.1), (13, 8, 2.2), (20, 64, 2.0)])
@pytest.mark.parametrize("m", [2, 3])
def test_step_block_edges_match_oracle(N, B, radius, m):
    w = synthetic.make_workload("sphere_r12_h0.2", radius=radius, nat=2, atom_radius=1.0)
    og, H, g, solver, psi = _setup(w, N, B, m=m, tol=1e-12)
    opts = rmmdiis.Options(m=m, block=B, tol=1e-12)
    for _ in range(2):
        psi = rmmdiis.rmmdiis_step(H, psi, opts)["psi"]
    want = rmmdiis.rmmdiis_step(H, psi, opts)
    t = torch.from_numpy(rsd.to_blocks(psi, B)).to(DEV)
    eig, res, _ = solver.step(t)
    got = rsd.from_blocks(t.cpu().numpy(), N)
    assert np.max(np.abs(eig - want["eig"])) < 1e-12 * np.max(np.abs(want["eig"]))
    assert np.max(np.abs(res - want["resnorm"])) < 1e-10 * np.max(want["resnorm"])
    assert np.max(np.abs(got - want["psi"])) < 1e-10 * np.max(np.abs(want["psi"]))
    assert not np.any(t.cpu().numpy()[-1, :, N - (N - 1) // B * B:])      # padding stays zero


def test_block_stop_freezes_converged_blocks():
    w = synthetic.make_workload("sphere_r12_h0.2", radius=2.4, nat=3, atom_radius=1.2)
    N, B = 16, 8
    og, H, g, solver, psi = _setup(w, N, B, tol=1e9)
    t = torch.from_numpy(rsd.to_blocks(psi, B)).to(DEV)
    eig, res, nconv = solver.step(t)
    assert nconv == N
    lam, xi, p2, _ = linalg.rayleigh_ritz(psi, H.apply(psi), og.dv)
    p2, _, _ = linalg.orthonormalize(p2, og.dv)
    got = rsd.from_blocks(t.cpu().numpy())
    assert np.max(np.abs(got - p2)) < 1e-9 * np.max(np.abs(p2))


@pytest.mark.parametrize("m", [1, 3])
def test_step_with_a_frozen_block_matches_oracle(m):
    """Block stopping rule (Sec. 9) with the lower block frozen and the upper
    one active: the GPU runs the trial step and the DIIS iterations on the
    active block only, the frozen states keep psi up to the final
    orthonormalisation, and the step agrees with the oracle's."""
    w = synthetic.make_workload("sphere_r12_h0.2", radius=2.4, nat=3, atom_radius=1.2)
    N, B = 16, 8
    og, H, g, _, psi = _setup(w, N, B, m=m, tol=1e-12)
    opts0 = rmmdiis.Options(m=m, block=B, tol=1e-12)
    for _ in range(6):
        psi = rmmdiis.rmmdiis_step(H, psi, opts0)["psi"]
    # a tolerance just above the lower block's residuals of the next step
    r = rmmdiis.rmmdiis_step(H, psi, opts0)["resnorm"]
    tol = float(np.max(r[:B])) * (1.0 + 1e-6)
    assert np.max(r[B:]) > 1.01 * tol
    want = rmmdiis.rmmdiis_step(H, psi, rmmdiis.Options(m=m, block=B, tol=tol))
    assert not want["active"][:B].any() and want["active"][B:].all()
    _, _, _, solver, _ = _setup(w, N, B, m=m, tol=tol)
    t = torch.from_numpy(rsd.to_blocks(psi, B)).to(DEV)
    eig, res, nconv = solver.step(t)
    assert solver.stats()["frozen_blocks"] == 1
    got = rsd.from_blocks(t.cpu().numpy())
    assert np.max(np.abs(eig - want["eig"])) < 1e-12 * np.max(np.abs(want["eig"]))
    assert np.max(np.abs(res - want["resnorm"])) < 1e-10 * np.max(want["resnorm"])
    assert np.max(np.abs(got - want["psi"])) < 1e-10 * np.max(np.abs(want["psi"]))


# two active blocks beside a frozen one; all three make 3.1 and 6.1 million values,
# two of 16 states 2.0 (H psi of so few, alone, would take another kernel)
@pytest.mark.parametrize("B,with_net", [(16, False), (32, True)])
def test_active_blocks_do_not_depend_on_the_frozen_ones(B, with_net):
    """Periodic box, no potential: the top block holds plane waves of the highest
    energies, which are eigenvectors, the others smooth states orthogonal to them.
    With the stopping rule the top block is frozen, without it all run: the other
    blocks' states come out the same, bit for bit (orthonormalisation takes the
    states in order, so the top block does not enter them)."""
    n, h = 40, 0.25
    g = rsd.Grid("periodic", h, n=n)
    xyz = np.round(g.xyz() / h).astype(int)
    pts = torch.from_numpy(xyz).to(DEV).double()
    waves = []
    half = n // 2
    for d in sorted(np.ndindex(4, 4, 4), key=sum):
        k = torch.tensor([half - q for q in d], device=DEV, dtype=torch.float64)
        arg = 2.0 * np.pi / n * (pts @ k)
        waves += [torch.cos(arg)] if not any(d) else [torch.cos(arg), torch.sin(arg)]
    top = torch.stack(waves[:B], dim=1)
    rng = np.random.default_rng(31)
    low = torch.zeros((g.np, 2 * B), device=DEV, dtype=torch.float64)
    for s in range(2 * B):
        for _ in range(4):
            k = torch.from_numpy(rng.integers(-6, 7, 3).astype(float)).to(DEV)
            low[:, s] += rng.normal() * torch.cos(2.0 * np.pi / n * (pts @ k) + rng.uniform(0.0, 6.0))
        low[:, s] *= 1.0 + 0.3 * torch.cos(2.0 * np.pi / n * pts[:, s % 3] + s)
    psi = torch.stack([low[:, :B], low[:, B:], top]).contiguous()
    net = None
    if with_net:
        net = rsd.Cnn(2 * B, g.np)
        net.set_params(np.random.default_rng(32).normal(scale=0.2, size=rsd.Cnn.NPARAM))
    out = []
    for stop in (True, False):
        solver = rsd.Eigensolver(g, None, torch.zeros(g.np, device=DEV, dtype=torch.float64), 3 * B, B, tol=1e-6,
                                 block_stop=stop)
        if net is not None:
            solver.set_precond(net)
        x = psi.clone()
        solver.orthonormalize(x)
        _, res, _ = solver.step(x)
        assert solver.stats()["frozen_blocks"] == int(stop)
        assert np.max(res[2 * B:]) < 1e-6 and np.min(res[:2 * B]) > 1e-6
        out.append(x[:2].cpu())
    assert torch.equal(out[0], out[1])


def test_converges_harmonic_box():
    """Lowest four levels of the 32^3 harmonic box from random states."""
    w = synthetic.make_workload("box32_harmonic", nstates=4)
    og, H, g, solver, psi = _setup(w, 4, 4, tol=1e-9)
    t = torch.from_numpy(rsd.to_blocks(psi, 4)).to(DEV)
    want = np.array([1.4999991750, 2.4999964915, 2.4999964915, 2.4999964915])
    for it in range(150):
        eig, res, nconv = solver.step(t)
        if nconv == 4:
            break
    assert np.max(np.abs(eig - want)) < 1e-9
    assert np.max(res) < 1e-9


def _split_floor(ev, npts):
    """Eigenvalue floor of the split-precision solve on a small grid.  Each
    split-BF16 product a b of the subspace matrix carries an error up to
    2^-16 |a| |b| (two bfloat16 terms per operand); over npts points of
    independent rounding an entry <phi|H phi> = eps errs by about
    2^-16 |eps| / sqrt(npts).  Three such deviations, or 1e-6 Ha where that
    is larger (on grids of 1e5 points and more the floor is below 1e-7)."""
    return max(1e-6, 3.0 * 2.0 ** -16 * float(np.max(np.abs(ev))) / np.sqrt(npts))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_converges_dense_bruteforce(dtype):
    """Tiny sphere (2 109 points) with wells and projectors: lowest
    eigenvalues of the dense matrix, to 1e-10 Ha in FP64; the FP32 /
    split-precision solve reaches them to its rounding floor (4e-6 Ha
    here)."""
    w = synthetic.make_workload("sphere_r12_h0.2", radius=1.6, h=0.2, nat=2, atom_radius=0.6, rc=1.0)
    og, H, g, solver, psi = _setup(w, 8, 8, dtype=dtype, tol=1e-9 if dtype == np.float64 else 1e-5)
    ev = np.linalg.eigvalsh(H.dense())[:8]
    etol = 1e-10 if dtype == np.float64 else _split_floor(ev, og.np)
    t = torch.from_numpy(rsd.to_blocks(psi.astype(dtype), 8)).to(DEV)
    best = np.inf
    for it in range(300):
        eig, res, nconv = solver.step(t)
        best = np.max(np.abs(eig - ev))
        if best < etol / 10:
            break
    assert best < etol


def test_partial_last_block_step_matches_oracle():
    """12 states in blocks of 8: the last block holds 4 zero padding states.
    The step agrees with the oracle's on the 12 states (whose stopping rule
    sees a block of 4), and the padding stays exactly zero."""
    w = synthetic.make_workload("sphere_r12_h0.2", radius=2.4, nat=3, atom_radius=1.2)
    N, B = 12, 8
    og, H, g, solver, psi = _setup(w, N, B, tol=1e-12)
    opts = rmmdiis.Options(m=3, block=B, tol=1e-12)
    for _ in range(3):
        psi = rmmdiis.rmmdiis_step(H, psi, opts)["psi"]
    want = rmmdiis.rmmdiis_step(H, psi, opts)
    t = torch.from_numpy(rsd.to_blocks(psi, B)).to(DEV)
    assert tuple(t.shape) == (2, og.np, B)
    eig, res, nconv = solver.step(t)
    assert eig.shape == (N,) and res.shape == (N,)
    full = rsd.from_blocks(t.cpu().numpy())
    assert np.all(full[N:] == 0.0)
    got = full[:N]
    assert np.max(np.abs(eig - want["eig"])) < 1e-12 * np.max(np.abs(want["eig"]))
    assert np.max(np.abs(res - want["resnorm"])) < 1e-10 * np.max(want["resnorm"])
    assert np.max(np.abs(got - want["psi"])) < 1e-10 * np.max(np.abs(want["psi"]))


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_partial_last_block_converges(dtype):
    """6 states in blocks of 4 (two padding states) reach the lowest six
    eigenvalues of the dense matrix of a tiny sphere (FP32: to the split-
    precision floor of that grid)."""
    w = synthetic.make_workload("sphere_r12_h0.2", radius=1.6, h=0.2, nat=2, atom_radius=0.6, rc=1.0)
    og, H, g, solver, psi = _setup(w, 6, 4, dtype=dtype, tol=1e-9 if dtype == np.float64 else 1e-5)
    ev = np.linalg.eigvalsh(H.dense())[:6]
    etol = 1e-10 if dtype == np.float64 else _split_floor(ev, og.np)
    t = torch.from_numpy(rsd.to_blocks(psi.astype(dtype), 4)).to(DEV)
    best = np.inf
    for it in range(300):
        eig, res, nconv = solver.step(t)
        best = np.max(np.abs(eig - ev))
        if best < etol / 10:
            break
    assert best < etol
    assert np.all(rsd.from_blocks(t.cpu().numpy())[6:] == 0.0)


def test_cage_workload_full_size_steps():
    """The largest workload (sphere R 18 at h 0.18, 4.19M points, 60 atoms on
    a cage), 240 FP32 states in blocks of 64 (one padded block): three steps
    run, keep the padding zero, and lower every Rayleigh-Ritz value."""
    w = synthetic.WORKLOADS["sphere_r18_h0.18_cage60"]
    g = rsd.Grid.for_workload(w)
    atoms = synthetic.draw_atoms(w)
    v = synthetic.potential_for(w, g.xyz(), atoms)
    nl = rsd.NonLocal(g, atoms.pos, atoms.D, w.rc, w.sigma, max_states=256)
    tv = torch.from_numpy(v.astype(np.float32)).to(DEV)
    psi = synthetic.draw_states(synthetic.rng_after_atoms(w), w.nstates, g.np).astype(np.float32)
    t = torch.from_numpy(rsd.to_blocks(psi, w.block)).to(DEV)
    del psi
    assert tuple(t.shape) == (4, g.np, 64)
    solver = rsd.Eigensolver(g, nl, tv, w.nstates, w.block)
    solver.orthonormalize(t)
    eigs = [solver.step(t)[0] for _ in range(3)]
    assert all(e.shape == (240,) and np.all(np.isfinite(e)) for e in eigs)
    assert np.all(eigs[2] <= eigs[0] + 1e-6 * np.abs(eigs[0]))
    assert torch.count_nonzero(t[3, :, 48:]).item() == 0


def test_bad_solver_arguments_raise():
    w = synthetic.make_workload("sphere_r12_h0.2", radius=2.4, nat=3, atom_radius=1.2)
    g = rsd.Grid.for_workload(w)
    v = torch.zeros(g.np, dtype=torch.float64, device=DEV)
    for n, B in ((0, 8), (257, 8), (16, 3), (16, 128)):
        with pytest.raises(rsd.RsError) as e:
            rsd.Eigensolver(g, None, v, n, B)
        assert e.value.code == rsd._abi.RS_EINVAL


# ------------------------------------------------- the benchmark's shape
# 128 states in blocks of 32 on a 113k-point sphere: the persistent
# rotations at N = 128 (eight 16-state column blocks, X resident in LDS), and
# the N = 128 LDS Cholesky, triangular inverse and Jacobi, as in the
# benchmark's eigensolver runs.
@pytest.fixture(scope="module")
def bench_shape():
    from oracle import cpu_hpsi
    cpu_hpsi.build()
    w = synthetic.make_workload("sphere_r12_h0.2", radius=6.0, nat=6, atom_radius=4.0)
    og, atoms, H = hamiltonian.build_system(w)
    F = cpu_hpsi.FastHamiltonian(H)
    psi0, _, _ = linalg.orthonormalize(synthetic.draw_states(synthetic.rng_after_atoms(w), 128, og.np), og.dv)
    opts = rmmdiis.Options(m=3, block=32, tol=1e-12)
    first = rmmdiis.rmmdiis_step(F, psi0, opts)      # the step from the random start
    psi = first["psi"]
    for _ in range(4):                                # oracle state after 5 steps
        psi = rmmdiis.rmmdiis_step(F, psi, opts)["psi"]
    after5 = rmmdiis.rmmdiis_step(F, psi, opts)
    return dict(w=w, og=og, atoms=atoms, H=H, psi0=psi0, first=first, psi5=psi, after5=after5)


def _bench_solver(S, dtype):
    w, og, atoms = S["w"], S["og"], S["atoms"]
    g = rsd.Grid.for_workload(w)
    nl = rsd.NonLocal(g, atoms.pos, atoms.D, w.rc, w.sigma, max_states=128)
    v = torch.from_numpy(S["H"].vloc.astype(dtype)).to(DEV)
    return g, nl, v, rsd.Eigensolver(g, nl, v, 128, 32, m=3, tol=1e-12)


def test_step_bench_shape_fp64_random_start(bench_shape):
    """From random orthonormal states the subspace matrix is dense: the
    Jacobi eigensolver runs to FP64 convergence (more than the 6 sweeps an
    earlier version capped it at) and the step matches the oracle's, whose
    Rayleigh-Ritz uses LAPACK."""
    S = bench_shape
    g, nl, v, solver = _bench_solver(S, np.float64)
    want = S["first"]
    t = torch.from_numpy(rsd.to_blocks(S["psi0"], 32)).to(DEV)
    eig, res, _ = solver.step(t)
    st = solver.stats()
    print(f"rr_sweeps {st['rr_sweeps']}")
    assert st["rr_sweeps"] > 6
    got = rsd.from_blocks(t.cpu().numpy())
    print(f"eig {np.max(np.abs(eig - want['eig']) / np.abs(want['eig'])):.2e} "
          f"res {np.max(np.abs(res - want['resnorm']) / want['resnorm']):.2e} "
          f"psi {np.max(np.abs(got - want['psi'])) / np.max(np.abs(want['psi'])):.2e}")
    assert np.max(np.abs(eig - want["eig"])) < 1e-12 * np.max(np.abs(want["eig"]))
    assert np.max(np.abs(res - want["resnorm"])) < 1e-10 * np.max(want["resnorm"])
    assert np.max(np.abs(got - want["psi"])) < 1e-10 * np.max(np.abs(want["psi"]))


def test_step_bench_shape_fp64(bench_shape):
    """One FP64 step from the oracle's state after 5 steps."""
    S = bench_shape
    g, nl, v, solver = _bench_solver(S, np.float64)
    want = S["after5"]
    t = torch.from_numpy(rsd.to_blocks(S["psi5"], 32)).to(DEV)
    eig, res, _ = solver.step(t)
    got = rsd.from_blocks(t.cpu().numpy())
    print(f"rr_sweeps {solver.stats()['rr_sweeps']} eig {np.max(np.abs(eig - want['eig'])):.2e} Ha "
          f"res {np.max(np.abs(res - want['resnorm']) / want['resnorm']):.2e} "
          f"psi {np.max(np.abs(got - want['psi'])) / np.max(np.abs(want['psi'])):.2e}")
    assert np.max(np.abs(eig - want["eig"])) < 1e-12 * np.max(np.abs(want["eig"]))
    assert np.max(np.abs(res - want["resnorm"])) < 1e-10 * np.max(want["resnorm"])
    assert np.max(np.abs(got - want["psi"])) < 1e-10 * np.max(np.abs(want["psi"]))


def test_step_bench_shape_split_precision(bench_shape):
    """The precision form (FP32 fields, split-BF16 contractions, FP64 small
    matrices): H psi of the oracle's 5-step state and one step from it,
    against the FP64 oracle; errors per H psi and per eigenvalue."""
    S = bench_shape
    g, nl, v, solver = _bench_solver(S, np.float32)
    x32 = S["psi5"].astype(np.float32)
    t = torch.from_numpy(rsd.to_blocks(x32, 32)).to(DEV)
    th = torch.empty_like(t)
    rsd.hpsi_block(g, nl, v, t, th)
    hp = rsd.from_blocks(th.cpu().numpy()).astype(np.float64)
    want_h = S["H"].apply(x32.astype(np.float64))
    herr = np.max(np.abs(hp - want_h), axis=1) / np.max(np.abs(want_h), axis=1)
    want = S["after5"]
    eig, res, _ = solver.step(t)
    got = rsd.from_blocks(t.cpu().numpy()).astype(np.float64)
    eerr = np.abs(eig - want["eig"])
    perr = np.max(np.abs(got - want["psi"])) / np.max(np.abs(want["psi"]))
    print(f"H psi max rel err per state {herr.max():.2e}; eigenvalue err max {eerr.max():.2e} Ha "
          f"median {np.median(eerr):.2e}; psi {perr:.2e}")
    assert herr.max() < 1e-5
    assert eerr.max() < 2e-6
    assert np.max(np.abs(res - want["resnorm"]) / want["resnorm"]) < 1e-3
    assert perr < 1e-4


def _harmonic_1d(n=32, h=0.3):
    """Eigenpairs of the 1-D factor of the harmonic box (25-point star =
    sum of three 1-D 9-point operators; Dirichlet, cell-centred)."""
    from oracle import stencil
    c = stencil.fd_weights(4)
    x = (np.arange(n) - 0.5 * (n - 1)) * h
    T = np.zeros((n, n))
    for i in range(n):
        T[i, i] = c[0]
        for m in range(1, 5):
            for j in (i - m, i + m):
                if 0 <= j < n:
                    T[i, j] = c[m]
    A = -0.5 / h ** 2 * T + np.diag(0.5 * x * x)
    return np.linalg.eigh(A)


def test_converges_harmonic_box_eight_states():
    """Config 1 as stated: the lowest 8 states, so state 8 is one member of
    the degenerate triplet at 3.4999938080 Ha, 1e-5 Ha above the triplet at
    3.4999835553.  The solve carries 8 buffer states (16 in blocks of 8): with
    exactly 8 the cut falls inside that 6-state cluster and the lower triplet
    separates from the upper one at a rate set by their 1e-5 Ha gap.  The
    lowest 8 eigenvalues reach the exact separable spectrum; the spectral
    projector of the first triplet matches the exact one built from the 1-D
    eigenvectors (eigenvectors of a degenerate cluster are compared only
    through their projector)."""
    w = synthetic.make_workload("box32_harmonic", nstates=16)
    og, H, g, solver, psi = _setup(w, 16, 8, tol=1e-9)
    t = torch.from_numpy(rsd.to_blocks(psi, 8)).to(DEV)
    want = np.array([1.4999991750] + [2.4999964915] * 3 + [3.4999835553] * 3 + [3.4999938080])
    for it in range(300):
        eig, res, nconv = solver.step(t)
        if res[:8].max() < 1e-9:
            break
    print(f"steps {it + 1}, max res of the lowest 8 {res[:8].max():.2e}")
    assert np.max(np.abs(eig[:8] - want)) < 1e-9
    e1, u1 = _harmonic_1d()
    ix = og.inner[:, 0] - og.inner[:, 0].min()
    iy = og.inner[:, 1] - og.inner[:, 1].min()
    iz = og.inner[:, 2] - og.inner[:, 2].min()
    trip = np.stack([u1[ix, a] * u1[iy, b] * u1[iz, c] for a, b, c in ((1, 0, 0), (0, 1, 0), (0, 0, 1))])
    trip /= og.dv ** 0.5
    got = rsd.from_blocks(t.cpu().numpy())[1:4]
    # projectors compared through their action on a fixed set of vectors
    probe = np.random.default_rng(0).normal(size=(5, og.np))
    Pg = og.dv * (probe @ got.T) @ got
    Pe = og.dv * (probe @ trip.T) @ trip
    assert np.max(np.abs(Pg - Pe)) < 1e-6 * np.max(np.abs(Pe))
