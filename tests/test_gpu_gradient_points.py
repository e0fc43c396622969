"""fr_intermediate's gradient at the flux points on a mesh that nobody has
tuned: at the orders where the gradient operator has fewer than four 16-row
blocks (tets of orders 1 and 2, prisms and hexahedra of order 1) every flux
point holds the gradient, bit for bit as the separate kernels leave it; at
higher orders the read faces do.  Meshes on both sides of the small-mesh
launches (256 tiles of 16 elements), ragged against the tiles."""
import math

import numpy as np
import pytest

from gradient_points import read_points
from oracle import fr, mesh as om
from paper_1409_0405_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

NAMES = ("tet", "pri", "hex")
ARRAYS = {
    "hybrid": lambda: inputs.hybrid_box(6, 4, 6, 3, 3, (2 * math.pi,) * 3, jitter=0.1, seed=5),
    # 5,292 tets and prisms: above 256 tiles, 12 past a tile of 16
    "wide": lambda: inputs.small_mixed_box(nxy=21, n_pri_layers=6, n_tet_layers=2, jitter=0.1, seed=5),
}


def _gradient(arrays, O, p, prec, steps, **kw):
    from paper_1409_0405_amd import frlib
    U = fr.initial_state(O, inputs.taylor_green, mach=0.3)
    ts = [NAMES.index(n) for n in O.types]
    M = frlib.Mesh(arrays, p, system="ns", precision=prec, mu=0.02, **kw)
    u = {t: frlib.to_device_state(M, t, np.transpose(U[NAMES[t]], (1, 2, 0))) for t in ts}
    r = {t: frlib.state_tensor(M, t) for t in ts}
    if steps:
        for t in ts:
            M.set_solution(t, u[t].data_ptr())
        M.rk_step(frlib.FR_RK45_2RP, 1e-3, steps)
    else:
        M.rhs([u[t].data_ptr() if t in u else 0 for t in range(3)],
              [r[t].data_ptr() if t in r else 0 for t in range(3)])
    out = {}
    for t in ts:
        q = M.query(t)
        out[t] = torch.zeros((q["nfpts"], 15, q["ld"]), dtype=r[t].dtype, device="cuda")
        M.intermediate(t, 2, out[t].data_ptr())
        out[t] = out[t][:, :, :q["nelem"]]
    nupts = {t: M.query(t)["nupts"] for t in ts}
    torch.cuda.synchronize()
    M.close()
    return out, nupts


@pytest.mark.parametrize("kind,p,prec,steps", [("hybrid", 1, "fp32", 0), ("hybrid", 2, "fp32", 0), ("hybrid", 1, "fp64", 2),
                                               ("hybrid", 3, "fp32", 0), ("wide", 1, "fp32", 0), ("wide", 1, "fp64", 0),
                                               ("wide", 2, "fp32", 2)])
def test_untuned_low_orders_hold_the_gradient_at_every_flux_point(kind, p, prec, steps):
    print(f"{kind} p{p} {prec} steps {steps}", flush=True)
    arrays = ARRAYS[kind]()
    O = om.build_mesh(arrays, p)
    got, nupts = _gradient(arrays, O, p, prec, steps)
    want, _ = _gradient(arrays, O, p, prec, steps, separate_gradient=True)
    read = read_points(O)
    it = torch.int64 if prec == "fp64" else torch.int32
    for t in got:
        mask = torch.from_numpy(np.ascontiguousarray(read[NAMES[t]].T)).to("cuda")[:, None, :]
        every = 3 * nupts[t] <= 48
        a, b = ((x if every else torch.where(mask, x, 0)).contiguous() for x in (got[t], want[t]))
        assert torch.equal(a.view(it), b.view(it)), NAMES[t]
        assert bool(torch.where(mask, 0, want[t]).any()), NAMES[t]
