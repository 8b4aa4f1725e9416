"""GPU parity of the learned preconditioner (network forward, training
gradient, Adam, application on grids, training crops) and of the
shifted-kinetic solves against the FP64 oracle, through the C ABI."""
import numpy as np
import pytest

import synthetic
from oracle import cnn as ocnn
from oracle import grid as ogrid
from oracle import stencil

torch = pytest.importorskip("torch")
import paper_1306_2953_amd as rsd  # noqa: E402

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module", autouse=True)
def need_gpu():
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"


def _params(seed, scale=0.3):
    rng = np.random.default_rng(seed)
    p = rng.normal(scale=scale, size=ocnn.NP)
    p[ocnn.NW], p[ocnn.NW + 1] = 0.3, -0.8
    return p.astype(np.float32).astype(np.float64)   # exactly representable in FP32


def _dev(a, dtype=None):
    a = np.ascontiguousarray(a if dtype is None else a.astype(dtype))
    return torch.from_numpy(a).to(DEV)


def _rel(got, want):
    return np.linalg.norm(np.ravel(got - want)) / np.linalg.norm(np.ravel(want))


@pytest.mark.parametrize("dims,periodic", [((10, 12, 9), False), ((8, 8, 8), True), ((5, 3, 7), False)])
def test_forward_matches_oracle(dims, periodic):
    p = _params(1)
    net = rsd.Cnn(4, 2048)
    net.set_params(p)
    assert np.array_equal(net.get_params(), p.astype(np.float32))
    rng = np.random.default_rng(2)
    u = rng.normal(size=(3,) + dims).astype(np.float32)
    f = net.forward(_dev(u), periodic=periodic).cpu().numpy()
    pad = "wrap" if periodic else "zero"
    for i in range(3):
        want, _ = ocnn.forward(p, u[i].astype(np.float64), np.ones(dims), pad)
        assert np.max(np.abs(f[i] - want)) <= 1e-5 * np.max(np.abs(want))


# one point, rows of one column and past it, whole 16 x 16 columns, one point
# past them on each axis, and enough boxes for columns of the full depth, whose
# last one is cut short
@pytest.mark.parametrize("n,dims,periodic", [(1, (1, 1, 1), True), (2, (1, 1, 40), False), (2, (4, 16, 16), True),
                                             (3, (5, 17, 33), False), (2, (3, 18, 17), True),
                                             (1100, (40, 3, 2), True), (1100, (33, 2, 3), False)])
def test_forward_at_column_edges(n, dims, periodic):
    p = _params(15)
    net = rsd.Cnn(n, int(np.prod(dims)))
    net.set_params(p)
    u = np.random.default_rng(16).normal(size=(n,) + dims).astype(np.float32)
    f = net.forward(_dev(u), periodic=periodic).cpu().numpy()
    for i in sorted({0, n // 2, n - 1}):
        want, _ = ocnn.forward(p, u[i].astype(np.float64), np.ones(dims), "wrap" if periodic else "zero")
        # as above: layer 2's split products carry about 2^-16 per term
        assert np.max(np.abs(f[i] - want)) <= 1e-5 * np.max(np.abs(want))


# layer 3 in columns of 8 planes, more than one tile in x and y
@pytest.mark.parametrize("periodic", [False, True])
def test_forward_in_columns_of_several_tiles(periodic):
    n, dims = 300, (9, 17, 18)
    p = _params(25)
    net = rsd.Cnn(n, int(np.prod(dims)))
    net.set_params(p)
    u = np.random.default_rng(26).normal(size=(n,) + dims).astype(np.float32)
    f = net.forward(_dev(u), periodic=periodic).cpu().numpy()
    for i in (0, 1, 149, 298, 299):
        want, _ = ocnn.forward(p, u[i].astype(np.float64), np.ones(dims), "wrap" if periodic else "zero")
        # as above: layer 2's split products carry about 2^-16 per term
        assert np.max(np.abs(f[i] - want)) <= 1e-5 * np.max(np.abs(want))


# the application of the trained network with a mask (or across faces) in columns
# of 8 planes: boxes of 33^3, 21 x 32 x 33 and 32^3, 32 and 64 of them at once
@pytest.mark.parametrize("kind,blocks", [("sphere", 1), ("union", 2), ("periodic", 2)])
def test_precondition_in_masked_columns(kind, blocks):
    kw = {"sphere": dict(radius=4.8), "periodic": dict(n=32),
          "union": dict(radius=3.0, centres=np.array([[0.0, 0.0, 0.0], [3.6, 1.8, 0.0], [0.3, 3.6, 0.1]]))}[kind]
    og, g = ogrid.build_grid(kind, 0.3, **kw), rsd.Grid(kind, 0.3, **kw)
    p = _params(27, scale=0.2)
    B, N = 32, 32 * blocks
    dims = ocnn.box_of(og)[1]
    net = rsd.Cnn(N, int(np.prod(dims)))
    net.set_params(p)
    assert net.box(g) == tuple(dims)
    rng = np.random.default_rng(28)
    r = rng.normal(size=(N, og.np)).astype(np.float32)
    sig = -rng.uniform(0.5, 4.0, size=N)
    out = net.precondition(g, _dev(rsd.to_blocks(r, B)), _dev(sig))
    some = [0, 13, N - 1]
    got = rsd.from_blocks(out.cpu().numpy()).astype(np.float64)[some]
    want = ocnn.precondition(p, og, r[some].astype(np.float64), sig[some])
    assert np.max(np.abs(got - want)) <= 2e-5 * np.max(np.abs(want))


def test_tanh_accuracy():
    """Layer 1's tanh against FP64: with one point, input 1 and layer 2's weights
    zero, the gradient of w2[0][c] at the centre is tanh(w1[c]) times a common
    factor, which channel 7 (tanh 1) gives.  tanh errs by 1.38 units in the last
    place at most, the product's rounding by one of tanh's."""
    rng = np.random.default_rng(29)
    x = np.concatenate([2.0 ** rng.uniform(-20, 4.3, 1300), rng.uniform(0.8, 1.1, 400), rng.uniform(0.0, 10.0, 400)])
    x = (x * rng.choice([-1.0, 1.0], x.size)).astype(np.float32)
    net = rsd.Cnn(1, 1)
    one = torch.ones((1, 1, 1, 1), device=DEV)
    sig = torch.full((1,), -1.0, device=DEV, dtype=torch.float64)
    got = np.empty(x.size)
    for k in range(0, x.size, 7):
        p = np.zeros(ocnn.NP, np.float32)
        p[13:216:27][:7], p[13:216:27][7] = x[k:k + 7], 20.0
        p[1944:2160] = 0.7
        net.set_params(p)
        _, grad, _ = net.loss_grad(one, one, sig, 0.25, 0)
        d = grad[216 + 13:216 + 216:27].astype(np.float64)
        assert d[7] != 0.0
        got[k:k + 7] = d[:7] / d[7]
    want = np.tanh(x.astype(np.float64))
    err = np.abs(got - want) / np.spacing(np.abs(want).astype(np.float32)).astype(np.float64)
    assert np.max(err) <= 2.4, (np.max(err), x[np.argmax(err)])
    assert np.sqrt(np.mean(err ** 2)) <= 0.6


# columns of 8 and of 16 rows: both sides of the line, alone and after whole ones,
# shallow and deep, and more shallow ones than work-groups
@pytest.mark.parametrize("n,dims,periodic", [(2, (4, 8, 17), True), (2, (5, 9, 5), False), (1, (4, 24, 16), False),
                                             (1, (4, 25, 33), True), (1100, (9, 8, 4), False), (1100, (9, 9, 4), True),
                                             (1601, (5, 5, 4), True), (801, (4, 20, 4), False)])
def test_network_at_half_columns(n, dims, periodic):
    p = _params(21)
    net = rsd.Cnn(n, int(np.prod(dims)))
    net.set_params(p)
    rng = np.random.default_rng(22)
    u = rng.normal(size=(n,) + dims).astype(np.float32)
    f = net.forward(_dev(u), periodic=periodic).cpu().numpy()
    for i in sorted({0, n // 2, n - 1}):
        want, _ = ocnn.forward(p, u[i].astype(np.float64), np.ones(dims), "wrap" if periodic else "zero")
        # as above: layer 2's split products carry about 2^-16 per term
        assert np.max(np.abs(f[i] - want)) <= 1e-5 * np.max(np.abs(want))
    t = rng.normal(size=(n,) + dims).astype(np.float32)
    sig = -rng.uniform(0.5, 5.0, n)
    _, grad, du = net.loss_grad(_dev(u), _dev(t), _dev(sig), 0.25, 0, want_du=True)
    _, wg, wdu = ocnn.loss_and_grad(p, u.astype(np.float64), t.astype(np.float64), sig, 0.25, 0)
    for a, b in ((0, 216), (216, 1944), (1944, 2160), (2160, 2162)):
        assert _rel(grad[a:b], wg[a:b]) <= 1e-4, (a, b)
    assert _rel(du.cpu().numpy(), wdu) <= 1e-4


# rows of a pair on both sides of the point, in the first, the last and an inner
# row of a column, and across the periodic faces
@pytest.mark.parametrize("periodic", [False, True])
@pytest.mark.parametrize("at", [(2, 0, 3), (3, 7, 0), (0, 8, 16), (6, 15, 9), (4, 17, 5)])
def test_nonfinite_inputs_reach_three_points(at, periodic):
    dims, p = (7, 18, 17), _params(17)
    net = rsd.Cnn(2, int(np.prod(dims)))
    net.set_params(p)
    u = np.random.default_rng(18).normal(size=(2,) + dims).astype(np.float32)
    pad = "wrap" if periodic else "zero"
    far = np.ones(dims, bool)
    near = [np.arange(c - 3, c + 4) for c in at]
    near = [a % d if periodic else a[(a >= 0) & (a < d)] for a, d in zip(near, dims)]
    far[np.ix_(*near)] = False
    u[(1,) + at] = 0.0
    want, _ = ocnn.forward(p, u[1].astype(np.float64), np.ones(dims), pad)
    u[(1,) + at] = np.nan
    f = net.forward(_dev(u), periodic=periodic).cpu().numpy()
    # three layers of reach one; the split products of layer 2 as above
    assert np.all(np.isnan(f[1][~far])) and np.all(np.isfinite(f[0]))
    assert np.max(np.abs(f[1] - want)[far], initial=0.0) <= 1e-5 * np.max(np.abs(want))
    # layer 1 takes an infinity to +-1, as it does any large number
    u[(1,) + at] = 1e9
    want, _ = ocnn.forward(p, u[1].astype(np.float64), np.ones(dims), pad)
    u[(1,) + at] = np.inf
    f = net.forward(_dev(u), periodic=periodic).cpu().numpy()
    assert np.max(np.abs(f[1] - want)) <= 1e-5 * np.max(np.abs(want))


def test_nonfinite_input_and_the_gradients_it_is_no_part_of():
    dims, p = (6, 9, 17), _params(19)
    net = rsd.Cnn(2, int(np.prod(dims)))
    net.set_params(p)
    rng = np.random.default_rng(20)
    u = rng.normal(size=(2,) + dims).astype(np.float32)
    t = rng.normal(size=(2,) + dims).astype(np.float32)
    sig = np.array([-0.7, -2.0])
    # at the first point of a box layer 1's delta is zero and only taps up to the
    # centre meet the input: 0 x Inf is NaN there, the others do not have it
    u[1, 0, 0, 0] = 1e9
    _, want, wdu = ocnn.loss_and_grad(p, u.astype(np.float64), t.astype(np.float64), sig, 0.25, 1)
    u[1, 0, 0, 0] = np.inf
    _, got, du = net.loss_grad(_dev(u), _dev(t), _dev(sig), 0.25, 1, want_du=True)
    past = np.zeros((3, 3, 3), bool)
    past[2], past[:, 2], past[:, :, 2] = True, True, True
    past = np.tile(past.ravel(), 8)
    assert np.all(np.isnan(got[:216][~past]))
    assert _rel(got[:216][past], want[:216][past]) <= 1e-4
    assert _rel(got[216:1944], want[216:1944]) <= 1e-4 and _rel(got[1944:2160], want[1944:2160]) <= 1e-4
    assert _rel(du.cpu().numpy(), wdu) <= 1e-4


def test_loss_gradient_and_adam_match_oracle():
    p = _params(3)
    net = rsd.Cnn(4, 4096)
    net.set_params(p)
    rng = np.random.default_rng(4)
    dims = (12, 11, 13)
    u = rng.normal(size=(3,) + dims).astype(np.float32)
    t = rng.normal(size=(3,) + dims).astype(np.float32)
    sig = np.array([-0.7, -2.0, -5.5])
    h, margin = 0.25, 2
    loss, grad, du = net.loss_grad(_dev(u), _dev(t), _dev(sig), h, margin, want_du=True)
    wl, wg, wdu = ocnn.loss_and_grad(p, u.astype(np.float64), t.astype(np.float64), sig, h, margin)
    assert loss == pytest.approx(wl, rel=1e-5)
    for a, b in ((0, 216), (216, 1944), (1944, 2160), (2160, 2162)):
        assert _rel(grad[a:b], wg[a:b]) <= 1e-4, (a, b)
    assert _rel(du.cpu().numpy(), wdu) <= 1e-4
    # Adam from zero moments with the GPU's own gradient
    net.adam_step(1e-3)
    want, _, _ = ocnn.adam_step(p, grad.astype(np.float64), np.zeros(ocnn.NP), np.zeros(ocnn.NP), 1, 1e-3)
    got = net.get_params()
    assert np.max(np.abs(got - want)) <= 1e-6 * np.max(np.abs(p))


# one-point axes, exactly one 4 x 8 x 16 block, one point past it on each
# axis, and more blocks than work-groups (each then sums several)
@pytest.mark.parametrize("n,dims,margin", [(2, (1, 1, 40), 0), (1, (4, 8, 16), 0), (3, (5, 9, 17), 1),
                                           (300, (9, 9, 17), 2)])
def test_weight_gradients_at_block_edges(n, dims, margin):
    p = _params(13)
    net = rsd.Cnn(n, int(np.prod(dims)))
    net.set_params(p)
    rng = np.random.default_rng(14)
    u = rng.normal(size=(n,) + dims).astype(np.float32)
    t = rng.normal(size=(n,) + dims).astype(np.float32)
    sig = -rng.uniform(0.5, 5.0, n)
    loss, grad, _ = net.loss_grad(_dev(u), _dev(t), _dev(sig), 0.25, margin)
    wl, wg, _ = ocnn.loss_and_grad(p, u.astype(np.float64), t.astype(np.float64), sig, 0.25, margin)
    # layer 2's split products carry about 2^-16 per term: 1e-5 of the sums
    assert loss == pytest.approx(wl, rel=1e-5)
    for a, b in ((0, 216), (216, 1944), (1944, 2160), (2160, 2162)):
        assert _rel(grad[a:b], wg[a:b]) <= 1e-4, (a, b)


@pytest.mark.parametrize("kind,dtype,B", [("sphere", np.float64, 8), ("sphere", np.float32, 16),
                                          ("periodic", np.float32, 8)])
def test_precondition_matches_oracle(kind, dtype, B):
    if kind == "sphere":
        og = ogrid.build_grid("sphere", 0.3, radius=2.4)
        g = rsd.Grid("sphere", 0.3, radius=2.4)
    else:
        og = ogrid.build_grid("periodic", 0.25, n=16)
        g = rsd.Grid("periodic", 0.25, n=16)
    p = _params(5, scale=0.2)
    N = 2 * B
    rng = np.random.default_rng(6)
    r = rng.normal(size=(N, og.np)).astype(dtype)
    r[3] = 0.0                                   # a zero residual maps to zero
    sig = -rng.uniform(0.5, 4.0, size=N)
    net = rsd.Cnn(16, 40000)
    net.set_params(p)
    assert net.box(g) == ocnn.box_of(og)[1]
    out = net.precondition(g, _dev(rsd.to_blocks(r, B)), _dev(sig))
    got = rsd.from_blocks(out.cpu().numpy()).astype(np.float64)
    want = ocnn.precondition(p, og, r.astype(np.float64), sig)
    assert np.all(got[3] == 0.0)
    assert np.max(np.abs(got - want)) <= 2e-5 * np.max(np.abs(want))


def test_fewer_blocks_need_no_new_scratch():
    """A call with fewer blocks of a grid than one before it allocates nothing
    (a capture would refuse it), and its replays give the eager results: those of
    the same blocks in the larger call."""
    g = rsd.Grid("periodic", 0.25, n=40)
    net = rsd.Cnn(32, 40 ** 3)
    net.set_params(_params(23, scale=0.2))
    gen = torch.Generator(device=DEV).manual_seed(24)
    r = torch.randn((3, g.np, 32), generator=gen, device=DEV)
    sig = -0.5 - torch.rand(96, generator=gen, device=DEV, dtype=torch.float64)
    want = net.precondition(g, r, sig)
    r2, s2 = r[:2].clone(), sig[:64].clone()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = net.precondition(g, r2, s2)
    for k in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[:2]), k
        net.precondition(g, r[1:], sig[32:].clone())     # the program's own work in between


def test_box_follows_the_grid_not_its_address():
    """A grid made after another one was destroyed may get its address; the
    network's box has to be the new grid's (dims only: no field is read)."""
    net = rsd.Cnn(1, 40000)
    reused = 0
    for k in range(40):
        g = rsd.Grid("box", 0.3, n=12)
        assert net.box(g) == (12, 12, 12)
        first = g.handle.value
        del g
        g = rsd.Grid("box", 0.3, n=8 + k % 3)
        assert net.box(g) == (8 + k % 3,) * 3
        reused += g.handle.value == first
        del g
    if not reused:
        pytest.skip("the allocator gave out no address twice")


def test_crops_match_direct_indexing():
    og = ogrid.build_grid("sphere", 0.3, radius=2.4)
    g = rsd.Grid("sphere", 0.3, radius=2.4)
    _, dims, idx, mask = ocnn.box_of(og)
    rng = np.random.default_rng(7)
    B, N = 8, 16
    r = rng.normal(size=(N, og.np))
    x = rng.normal(size=(N, og.np))
    net = rsd.Cnn(4, 40000)
    desc = np.array([[0, 0, 0, 0], [5, 3, 7, 2], [15, dims[2] - 2, dims[1] - 3, dims[0] - 1]], dtype=np.int32)
    cd = (4, 5, 6)
    u, t = net.crops(g, _dev(rsd.to_blocks(r, B)), _dev(rsd.to_blocks(x, B)), desc, cd)
    u, t = u.cpu().numpy(), t.cpu().numpy()
    for c, (k, x0, y0, z0) in enumerate(desc):
        s = np.sqrt(np.mean(r[k] ** 2))
        rb = np.zeros(int(np.prod(dims)))
        xb = np.zeros_like(rb)
        rb[idx], xb[idx] = r[k] / s, x[k] / s
        rb, xb = rb.reshape(dims), xb.reshape(dims)
        wu = np.zeros(cd)
        wt = np.zeros(cd)
        for zz in range(cd[0]):
            for yy in range(cd[1]):
                for xx in range(cd[2]):
                    Z, Y, X = z0 + zz, y0 + yy, x0 + xx
                    if Z < dims[0] and Y < dims[1] and X < dims[2]:
                        wu[zz, yy, xx] = rb[Z, Y, X]
                        wt[zz, yy, xx] = xb[Z, Y, X]
        assert np.allclose(u[c], wu, rtol=1e-6, atol=1e-6)
        assert np.allclose(t[c], wt, rtol=1e-6, atol=1e-6)


def test_shifted_solve_periodic_matches_closed_form():
    og = ogrid.build_grid("periodic", 0.25, n=24)
    g = rsd.Grid("periodic", 0.25, n=24)
    rng = np.random.default_rng(8)
    B, N = 8, 16
    r = rng.normal(size=(N, og.np))
    sig = -rng.uniform(0.3, 6.0, size=N)
    x, it = rsd.shifted_solve(g, _dev(rsd.to_blocks(r, B)), _dev(sig), tol=1e-12, maxit=3000)
    got = rsd.from_blocks(x.cpu().numpy())
    want = ocnn.shifted_inverse_periodic(og, r, sig)
    assert np.max(np.abs(got - want)) <= 1e-10 * np.max(np.abs(want))
    assert 0 < it < 3000


@pytest.mark.parametrize("dtype,tol,bound", [(np.float64, 1e-10, 1e-9), (np.float32, 1e-5, 1e-4)])
def test_shifted_solve_sphere_residual(dtype, tol, bound):
    og = ogrid.build_grid("sphere", 0.3, radius=3.0)
    g = rsd.Grid("sphere", 0.3, radius=3.0)
    rng = np.random.default_rng(9)
    B, N = 8, 8
    r = rng.normal(size=(N, og.np)).astype(dtype)
    r[2] = 0.0                                   # zero right-hand side -> zero solution
    sig = -rng.uniform(0.5, 3.0, size=N)
    x, it = rsd.shifted_solve(g, _dev(rsd.to_blocks(r, B)), _dev(sig), tol=tol, maxit=2000)
    got = rsd.from_blocks(x.cpu().numpy()).astype(np.float64)
    assert np.all(got[2] == 0.0)
    back = stencil.apply_kinetic(og, got) - sig[:, None] * got
    r64 = r.astype(np.float64)
    for k in range(N):
        if k != 2:
            assert np.linalg.norm(back[k] - r64[k]) <= bound * np.linalg.norm(r64[k])


def test_shifted_solve_reports_nonconvergence():
    g = rsd.Grid("periodic", 0.25, n=16)
    r = _dev(rsd.to_blocks(np.random.default_rng(10).normal(size=(8, g.np)), 8))
    with pytest.raises(rsd.RsError) as e:
        rsd.shifted_solve(g, r, _dev(np.full(8, -1.0)), tol=1e-14, maxit=3)
    assert e.value.code == rsd._abi.RS_ENOTCONV


def test_bad_arguments_raise():
    with pytest.raises(rsd.RsError):
        rsd.Cnn(0, 100)
    net = rsd.Cnn(2, 100)
    with pytest.raises(rsd.RsError):
        net.forward(_dev(np.zeros((3, 4, 4, 4), np.float32)))    # batch above max_batch
    g = rsd.Grid("periodic", 0.25, n=16)                          # box 4096 > max_box
    with pytest.raises(rsd.RsError):
        net.precondition(g, _dev(np.zeros((1, g.np, 2), np.float32)), _dev(-np.ones(2)))


def test_checkpoint_restores_training_state(tmp_path):
    """save/load carry the parameters, both Adam moments and the step count:
    after a restore, the next Adam step gives the same parameters as on the
    network that was saved; a file of another layout is refused."""
    p = _params(8, scale=0.2)
    a = rsd.Cnn(4, 4096)
    a.set_params(p)
    u = _dev(np.random.default_rng(1).normal(size=(2, 8, 8, 8)), np.float32)
    t = _dev(np.random.default_rng(2).normal(size=(2, 8, 8, 8)), np.float32)
    sig = _dev(np.array([-1.0, -2.0]))
    for _ in range(3):
        a.loss_grad(u, t, sig, 0.25, 1)
        a.adam_step(1e-3)
    path = str(tmp_path / "net.rscnn")
    a.save(path)
    b = rsd.Cnn(4, 4096)
    b.load(path)
    assert np.array_equal(a.get_params(), b.get_params())
    for net in (a, b):
        net.loss_grad(u, t, sig, 0.25, 1)
        net.adam_step(1e-3)
    assert np.array_equal(a.get_params(), b.get_params())
    bad = tmp_path / "bad.rscnn"
    bad.write_bytes(b"RSCNN001" + b"\0" * 16)
    with pytest.raises(rsd.RsError) as e:
        b.load(str(bad))
    assert e.value.code == rsd._abi.RS_EINVAL
