"""Set-up at the edges of its kernels' blocks (slices of 64, scans of 2048,
sorts padded to powers of two): neighbour lists and row pointers against the
oracle, and the velocity groups' lists through their diagnostics (counts
exact, means of the exported displacements to the rounding of a sum)."""
import numpy as np
import pytest

from paper_1901_07374_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def tl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1901_07374_amd import tlsph
    return tlsph


def beam(n, groups):
    """The first n particles of a beam of 4 x 4 particles per layer, in no
    group, all in one, or the last in the second of two."""
    dx = 1e-3
    rng = np.random.default_rng(n)
    q = np.arange(n)
    X = np.stack([q % 4, q // 4 % 4, q // 16], axis=1) * dx
    X = X + rng.uniform(-0.05 * dx, 0.05 * dx, X.shape)
    bc = np.full(n, 0 if groups == "all" else -1, np.int32)
    if groups == "last":
        bc[-1] = 1
    table = [I.bc_group(4, (0.0, 0.0, 1.0))] * {"none": 0, "all": 1, "last": 2}[groups]
    return I.Problem("beam", X, np.full(n, dx ** 3), np.array([0, n], np.int64),
                     [I.material(dx, I.DMG_NONE)], bc, table, np.zeros((n, 3)), steps=1,
                     dx=np.array([dx]))


@pytest.mark.parametrize("n,groups", [(33, "all"), (64, "none"), (65, "last"), (2047, "all"),
                                      (2048, "last"), (2049, "all"), (4097, "none"),
                                      (131073, "last")])
def test_lists_at_block_edges(tl, orc, n, groups):
    p = beam(n, groups)
    print(n, groups, flush=True)
    g, o = tl.Sim(p), orc.Sim(p)
    rp, col = g.neighbors()
    assert np.array_equal(rp, o.row_ptr)
    assert np.array_equal(col, o.col[: o.row_ptr[-1]])
    assert g.info()["nnz"] == o.row_ptr[-1]
    g.step(2)
    u, bd = g.get("u"), g.diagnostics()[1]
    for k in range(len(p.bc_groups)):
        sel = p.bc_group == k
        assert bd[k, 6] == sel.sum()
        if sel.any():
            assert np.allclose(bd[k, 3:6], u[sel].mean(0), rtol=1e-12, atol=1e-18)


def test_export_leaves_the_workspace_alone(tl):
    """The export's scan works in the caller's arrays: nothing of the context
    changes, so that it may run beside diagnostics or another export."""
    import torch
    p = beam(131073, "last")
    g = tl.Sim(p)
    rp, col = g.neighbors()
    ref = g.diagnostics()
    before = g.ws.clone()
    g.neighbors()
    assert torch.equal(g.ws, before)
    streams = [torch.cuda.Stream() for _ in range(3)]
    outs = [(torch.empty(p.n + 1, dtype=torch.int64, device="cuda"),
             torch.empty(len(col), dtype=torch.int32, device="cuda")) for _ in streams]
    torch.cuda.synchronize()
    for s, (r, c) in zip(streams, outs):
        assert tl.lib().tlsph_get_neighbors(g.ctx, r.data_ptr(), c.data_ptr(), s.cuda_stream) == 0
    got = g.diagnostics()
    torch.cuda.synchronize()
    for r, c in outs:
        assert np.array_equal(r.cpu().numpy(), rp) and np.array_equal(c.cpu().numpy(), col)
    assert all(np.array_equal(a, b) for a, b in zip(got, ref))


def test_many_specimens(tl):
    """More specimens than a grid may have rows: cubes of eight particles each,
    against their pair distances."""
    m, dx = 70000, 1e-3
    rng = np.random.default_rng(7)
    corner = np.array([[q & 1, q >> 1 & 1, q >> 2] for q in range(8)]) * dx
    X = corner + rng.uniform(-0.05 * dx, 0.05 * dx, (m, 8, 3))
    mat = I.material(dx, I.DMG_NONE)
    p = I.Problem("cubes", X.reshape(-1, 3), np.full(8 * m, dx ** 3), 8 * np.arange(m + 1),
                  [mat] * m, np.full(8 * m, -1, np.int32), [], np.zeros((8 * m, 3)), steps=1,
                  dx=np.full(m, dx))
    rp, col = tl.Sim(p, k_cap=8).neighbors()
    d = X[:, None] - X[:, :, None]
    near = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1] + d[..., 2] * d[..., 2]
            < mat["h"] * mat["h"]) & ~np.eye(8, dtype=bool)
    s, _, j = np.nonzero(near)
    assert np.array_equal(np.diff(rp), near.sum(2).ravel())
    assert np.array_equal(col, 8 * s + j)
