"""Non-finite values in the iterate: a patch whose closure holds one (Dirichlet nodes apart) becomes
non-finite as a whole, colour by colour, as the residual b - A x would make it (Sec. 2.2, Alg. 3), although
the eigenbasis form of the multiplicative pass needs no old interior value."""
import numpy as np
import pytest

import synth
from oracle import mesh

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2405_19004_amd as vps  # noqa: E402


def spread(bad, d, k, L, colours):
    """The non-finite nodes after the colours' passes."""
    bad = bad & ~mesh.boundary_mask(d, k, L)
    for c in colours:
        verts = mesh.patches_of_colour(d, L, c)
        closure = mesh.patch_box_ids_many(d, k, L, verts, interior=False)
        inner = mesh.patch_box_ids_many(d, k, L, verts, interior=True)
        bad[inner[bad[closure].any(axis=1)].reshape(-1)] = True
    return bad


@pytest.mark.parametrize("dtype", ["float32", "float64"])
@pytest.mark.parametrize("d,k,L", [(2, 1, 4), (2, 3, 3), (2, 7, 3), (3, 1, 3), (3, 2, 3), (3, 4, 2), (3, 4, 3)])
def test_non_finite_values_spread_by_patches(d, k, L, dtype):
    print("case non-finite", d, k, L, dtype, flush=True)
    dt = getattr(torch, dtype)
    P = vps.Problem(d, k, L)
    n = k * 2 ** L + 1
    b = torch.from_numpy(synth.random_interior(d, k, L, 3)).to("cuda", dt)
    x0 = synth.random_interior(d, k, L, 4)
    everything = list(range(2 ** d))
    # a cell-interior or vertex node, the first and last interior nodes, a cell face, a Dirichlet node
    for node, value in [((n // 2 + 1,) * d, np.nan), ((1,) * d, np.inf), ((n - 2,) * d, -np.inf),
                        ((k,) + (k + 1,) * (d - 1), np.nan), ((0,) + (k + 1,) * (d - 1), np.nan)]:
        at = sum(i * n ** a for a, i in enumerate(node))
        xh = x0.copy()
        xh[at] = value
        start = ~np.isfinite(xh)
        runs = [("ascending", everything, lambda x: P.smoother_apply(b, x)),
                ("descending", everything[::-1], lambda x: P.smoother_apply(b, x, reverse=True)),
                ("colour 0", [0], lambda x: P.color_pass(b, x, 0)),
                ("last colour", [2 ** d - 1], lambda x: P.color_pass(b, x, 2 ** d - 1))]
        for name, colours, run in runs:
            x = torch.from_numpy(xh).to("cuda", dt)
            run(x)
            got = ~np.isfinite(x.double().cpu().numpy())
            want = spread(start.copy(), d, k, L, colours)
            want |= start  # a Dirichlet entry stays as it is
            assert np.array_equal(got, want), (node, value, name, int(got.sum()), int(want.sum()))
    P.close()
