"""Line derivatives as matrix products (sets of independent patches): sizes at
the edges of their tiles -- the smallest line, 16-row and 32-pair blocks, both
kernels' largest lines, the first length that runs as a transform, periodic
lines, lengths without a radix plan -- against the FP64 oracle, and columns of
extreme scale.

Tolerance: the operands carry 22 bits (each partial product's relative error is
at most 2^-22), the FP32 sums add at most ten roundings a block of 32 pairs,
2^-24 each of the running sum; the sum of |kernel x difference| over a line is
at most about 1 + log(L) < 8 times its largest derivative for smooth lines.
8 (2^-22 + 2^-23) < 3e-6 of a line's largest derivative, pointwise; the input's
own rounding to FP32 enters the oracle too.  Ends of short lines with d = 5 add
the continuation's condition (rows of the derivative reach 1e2 of the interior's
there, exact in FP64 up to one FP32 rounding): twice that."""
import numpy as np
import pytest

from oracle import fcgram

pytestmark = pytest.mark.gpu
TOL = 6e-6


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2506_16076_amd import api
    ctx = api.Context(0)
    yield api, ctx, torch
    ctx.sync()


def make(api, ctx, sides, d, C, layout):
    from paper_2506_16076_amd._lib import blocked_layout
    n1 = np.array([s[0] for s in sides], np.int32)
    n2 = np.array([s[1] for s in sides], np.int32)
    if layout:
        off, plane = blocked_layout(n1, n2)
    else:
        off = np.concatenate([[0], np.cumsum(n1.astype(np.int64) * n2)])[:-1]
        plane = int(np.sum(n1.astype(np.int64) * n2))
    one = np.ones(len(sides))
    s = api.PatchSet(ctx, n1, n2, [C] * len(sides), [C] * len(sides), off, one, one, np.zeros((len(sides), 4), np.uint8),
                     d, plane, 0, 0, layout)
    return s, off, plane


def place(x, n1, off, plane, layout):
    """Patch arrays [nf, n2, n1] -> flat planes in the storage."""
    nf = x[0].shape[0]
    out = np.zeros((nf, plane), np.float32)
    idx = []
    for v, o in zip(x, off):
        b, a = v.shape[1:]
        j, i = np.meshgrid(np.arange(b), np.arange(a), indexing="ij")
        k = o + (((j // 4) * ((a + 7) // 8) + i // 8) * 32 + (j % 4) * 8 + i % 8 if layout else j * a + i)
        idx.append(k)
        out[:, k.ravel()] = v.reshape(nf, -1)
    return out, idx


def lines(rng, nf, b, a, direction):
    """Smooth lines along a direction, other lines other functions."""
    n, m = (a, b) if direction == 1 else (b, a)
    x = np.linspace(0, 1, n)
    f = np.ones((nf, m, n))
    for _ in range(3):
        f += rng.uniform(-.3, .3, (nf, m, 1)) * np.sin(2 * np.pi * rng.uniform(0, 1.5, (nf, m, 1)) * x +
                                                       rng.uniform(0, 6, (nf, m, 1)))
    return (f if direction == 1 else np.swapaxes(f, 1, 2)).astype(np.float32)


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("d,C,nf,sides", [
    (5, 27, 1, [(11, 13), (15, 16), (17, 31)]),
    (2, 27, 5, [(5, 33), (32, 47), (65, 101)]),
    (5, 28, 3, [(64, 63), (96, 130), (255, 35)]),
    (5, 27, 4, [(256, 34), (33, 257)]),
    (5, 28, 2, [(511, 17), (18, 512)]),
    (5, 27, 4, [(513, 12), (64, 545)]),
    (5, 0, 3, [(30, 64), (49, 96), (12, 200)]),
])
def test_matrix_lines(env, d, C, nf, sides, layout):
    api, ctx, torch = env
    rng = np.random.default_rng(7)
    s, off, plane = make(api, ctx, sides, d, C, layout)
    for direction in (1, 2):
        x = [lines(rng, nf, b, a, direction) for a, b in sides]
        inp, idx = place(x, None, off, plane, layout)
        ti = torch.from_numpy(inp.reshape(-1)).cuda()
        to = torch.full((nf * plane,), 7.0, device="cuda:0")
        api.fc_diff(s, direction, ti, to, nf)
        got = to.cpu().numpy().reshape(nf, plane)
        inside = np.zeros(plane, bool)
        for v, k in zip(x, idx):
            inside[k.ravel()] = True
            f = v.astype(np.float64) if direction == 1 else np.swapaxes(v, 1, 2).astype(np.float64)
            want = fcgram.diff_lines(f, d, C)
            g = got[:, k.ravel()].reshape(v.shape)
            g = g if direction == 1 else np.swapaxes(g, 1, 2)
            scale = np.maximum(np.abs(want).max(-1, keepdims=True), np.abs(f).max(-1, keepdims=True))
            err = float((np.abs(g - want) / scale).max())
            print("side", v.shape, "dir", direction, "max err", err, flush=True)
            assert err <= TOL
        assert np.all(got[:, ~inside] == 7.0)
    s.close()


def test_matrix_columns_keep_apart(env):
    """A column's scale is its own: columns of 1e-30 and 1e30, a zero one, and
    one with an infinity or a NaN next to an ordinary one."""
    api, ctx, torch = env
    n, m, d, C = 96, 12, 5, 27
    s, off, plane = make(api, ctx, [(n, m)], d, C, 0)
    rng = np.random.default_rng(3)
    base = lines(rng, 1, m, n, 1)[0]
    x = base.copy()
    x[1] *= np.float32(1e-30)
    x[2] *= np.float32(1e30)
    x[3] = 0
    x[4, 40] = np.inf
    x[5, 0] = np.nan
    to = torch.zeros(plane, device="cuda:0")
    api.fc_diff(s, 1, torch.from_numpy(x.reshape(-1)).cuda(), to, 1)
    got = to.cpu().numpy().reshape(m, n).astype(np.float64)
    fine = [0, 1, 2, 6, 7, 8, 9, 10, 11]
    want = fcgram.diff_lines(x[fine].astype(np.float64), d, C)
    scale = np.abs(want).max(-1, keepdims=True)
    assert float((np.abs(got[fine] - want) / scale).max()) <= TOL
    assert np.all(got[3] == 0)
    assert not np.isfinite(got[4]).any() and not np.isfinite(got[5]).any()
    s.close()


def operand_norm(x, d, C):
    """Norm of the products' terms Me xe, Mo xo of lines x over that of their
    sum, the derivative: what the terms' independent rounding errors are
    relative to."""
    M, N = x.shape
    L = N + C
    m, k = np.arange(L), np.arange(1, (L - 1) // 2 + 1)
    kappa = np.cos(2 * np.pi * (np.outer(2 * m - 1, k) % (2 * L)) / (2 * L)) @ (
        2 * np.pi * k * (N - 1) / L / np.sin(np.pi * k / L)) / L
    ext = fcgram.extend(x, fcgram.continuation_matrix(d, C))
    dx = np.roll(ext, -1, 1) - ext
    n = np.arange(L)
    nm = (N - 2 - n) % L
    a = n[n <= nm]
    b = nm[a]
    own = a == b
    K = kappa[(np.arange(N)[:, None] - n) % L]
    Ka, Kb = K[:(N + 1) // 2][:, a], np.where(own, K[:(N + 1) // 2][:, a], K[:(N + 1) // 2][:, b])
    xa, xb = dx[:, a], np.where(own, 0, dx[:, b])
    terms = ((Ka + Kb) / 2) ** 2 @ ((xa + xb) ** 2).T + ((Ka - Kb) / 2) ** 2 @ ((xa - xb) ** 2).T
    return np.sqrt(2 * terms.sum()) / np.linalg.norm(dx @ K.T)


@pytest.mark.parametrize("d", [2, 5])
@pytest.mark.parametrize("N", [48, 101, 256, 512])
@pytest.mark.parametrize("amp", [1e-5, 1e-6, 3e-7])
def test_nearly_uniform_lines(env, d, N, amp):
    """Lines 1.4 (1 + amp sin): the differences are far below the samples, and
    keep their bits.  Both operands of a term carry a relative rounding of at
    most 2^-22 and the dropped product is as small; at most 36 roundings of
    2^-24 of the FP32 sums, of independent sign: (2^-22 + 6 2^-24) of the norm
    of the terms (no less than the derivative's) in the L2 norm."""
    api, ctx, torch = env
    M, C = 48, 27
    rng = np.random.default_rng(11)
    x = np.linspace(0, 1, N)
    f = (1.4 * (1 + amp * np.sin(2 * np.pi * rng.uniform(.3, 2, (M, 1)) * x + rng.uniform(0, 6, (M, 1))))).astype(
        np.float32)
    s, off, plane = make(api, ctx, [(N, M)], d, C, 0)
    to = torch.zeros(plane, device="cuda:0")
    api.fc_diff(s, 1, torch.from_numpy(f.reshape(-1)).cuda(), to, 1)
    got = to.cpu().numpy().reshape(M, N).astype(np.float64)
    want = fcgram.diff_lines(f.astype(np.float64), d, C)
    err = np.linalg.norm(got - want) / np.linalg.norm(want)
    tol = (2.0 ** -22 + 6 * 2.0 ** -24) * max(1.0, operand_norm(f.astype(np.float64), d, C))
    print("d", d, "N", N, "amp", amp, "rel L2", err, "bar", tol, flush=True)
    assert err <= tol
    s.close()


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("d,C,sides", [
    (5, 27, [(11, 13), (17, 31), (256, 34)]),
    (2, 28, [(511, 17), (18, 512), (257, 12)]),
    (5, 27, [(513, 20), (40, 100)]),
    (5, 0, [(30, 64), (49, 12)]),
])
def test_any_number_of_fields_gives_the_same_bits(env, d, C, sides, layout):
    """One or two fields run on narrower tiles than three and more: the bits of
    a field do not depend on how many others are differentiated with it."""
    api, ctx, torch = env
    rng = np.random.default_rng(9)
    s, off, plane = make(api, ctx, sides, d, C, layout)
    for direction in (1, 2):
        inp, idx = place([lines(rng, 5, b, a, direction) for a, b in sides], None, off, plane, layout)
        ti = torch.from_numpy(inp.reshape(-1)).cuda()
        outs = {}
        for nf in (1, 2, 3, 5):
            to = torch.full((nf * plane,), 7.0, device="cuda:0")
            api.fc_diff(s, direction, ti, to, nf)
            outs[nf] = to.cpu().numpy().reshape(nf, plane)
        for k, side in zip(idx, sides):
            pairs = side[direction - 1] > 512    # transforms take two fields as one complex line
            for nf in (1, 2, 3):
                n = nf // 2 * 2 if pairs else nf
                assert np.array_equal(outs[nf][:n, k.ravel()], outs[5][:n, k.ravel()])
        inside = np.zeros(plane, bool)
        for k in idx:
            inside[k.ravel()] = True
        assert np.all(outs[1][:, ~inside] == 7.0) and not np.any(outs[1][:, inside] == 7.0)
    s.close()
