"""Host side of meshes whose nodes are not numbered line by line (CPU): what the ABI returns is in the caller's
numbering and does not depend on the order the unknowns get on the device."""
import numpy as np
import pytest

import qh_inputs as qi


def _host(xyz, tets):
    import paper_2103_06737_amd as qh
    ctx = qh.Context(-1)
    ctx.mesh_upload(xyz, tets)
    ctx.set_physics(qi.EPS0, qi.MU0, 1e-11, 1.0, 2.0 ** -56)
    return ctx


@pytest.mark.parametrize("extra", [[], [np.nan] * 3, [np.inf, 0.0, -np.inf]])
def test_scattered_box(extra):
    """A 10^3 box (6130 unknowns) numbered at random, also with a node of no tet whose coordinates are not
    finite: the assembled matrices are those of the box with its nodes in order, renumbered."""
    box = qi.BoxMesh(10)
    n = box.xyz.shape[0]
    perm = np.random.default_rng(3).permutation(n)
    inv = np.empty_like(perm)
    inv[perm] = np.arange(n)
    xyz = np.concatenate([box.xyz[perm], np.array(extra).reshape(-1, 3)])
    a, b = _host(box.xyz, box.tets), _host(xyz, inv[box.tets].astype(np.int32))
    ta, tb = a.topology(), b.topology()
    ia, ib = (t["edges"][~t["wall_edge"].astype(bool)] for t in (ta, tb))
    at = {tuple(e): k for k, e in enumerate(ib)}
    ends = inv[ia]
    sign = np.where(ends[:, 0] < ends[:, 1], 1.0, -1.0)
    k = np.array([at[tuple(sorted(e))] for e in ends])
    for which in (0, 1, 2):
        A, B = a.matrix(which), b.matrix(which)[k][:, k]
        D = abs(A - B.multiply(sign[:, None]).multiply(sign[None, :]).tocsr())
        assert D.max() <= 1e-13 * abs(A).max()
