"""The batch's step graph runs the groups of one order as parallel branches.
The groups share nothing, so the replays give the bits of the eager steps,
whatever groups are present: one order alone, two, all four, with several
steps per call, calls back to back on one stream, and the states read and
written between calls."""
import numpy as np
import pytest

from oracle import fr, mesh as om
from paper_1409_0405_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

NAMES = ("tet", "pri")


def _run(orders, precision, graph):
    from paper_1409_0405_amd import frlib
    meshes = [inputs.mixed_box(m, m, m, m, (1.0, 1.0, 1.0), z_split=0.5, jitter=0.05, seed=40 + i)
              for i, m in enumerate((2, 3, 4, 2, 3)[:len(orders)])]
    B = frlib.Batch(list(zip(meshes, orders)), system="euler", precision=precision)
    B.set_graph(graph)
    dtype = torch.float64 if precision == "fp64" else torch.float32
    for i, (mesh, p) in enumerate(zip(meshes, orders)):
        U = fr.initial_state(om.build_mesh(mesh, p), inputs.isentropic_vortex, centre=(0.5, 0.5), radius=0.15)
        for t, n in enumerate(NAMES):
            x = B.state_tensor(i, t)
            ne = B.query(i, t)["nelem"]
            x[:, :, :ne] = torch.as_tensor(np.transpose(U[n], (1, 2, 0)), dtype=dtype)
            x[:, :, ne:] = x[:, :, :1]
            B.set_solution(i, t, x.data_ptr())
    torch.cuda.synchronize()
    B.set_dt([1e-3 * (i + 1) for i in range(len(orders))])
    out = []
    for calls in ((1,), (3, 2), (1, 1, 1)):
        for n in calls:
            B.rk_step(frlib.FR_RK45_2RP, n)
        for i in range(len(orders)):
            for t in range(2):
                x = B.state_tensor(i, t)
                B.get_solution(i, t, x.data_ptr())
                out.append(x.clone())
                x[:, 0] += 1e-3                      # and on from a changed state
                B.set_solution(i, t, x.data_ptr())
        torch.cuda.synchronize()
    B.close()
    return out


@pytest.mark.parametrize("orders,precision", [((3,), "fp32"), ((1, 4), "fp32"), ((1, 2, 3, 4, 2), "fp32"),
                                              ((1, 2, 3, 4, 2), "fp64")])
def test_parallel_groups_give_the_bits_of_the_eager_steps(orders, precision):
    print(f"orders {orders} {precision}", flush=True)
    a, b = (_run(orders, precision, g) for g in (True, False))
    it = torch.int64 if precision == "fp64" else torch.int32
    assert all(bool(torch.isfinite(x).all()) for x in b)
    assert all(torch.equal(x.view(it), y.view(it)) for x, y in zip(a, b))
