"""The kernels on element tiles where the other tests do not take them, bit
for bit against the separate kernels (the same arithmetic on the same values
in the same order; raw bits, a zero's sign included):

* LDG weights with beta = 0 (both sides' gradients are read and both sides
  get a jump) and beta = -1/2 (side R only), every order and element type,
  with the oracle's FP64 residual as well;
* meshes above the small-mesh launches (256 tiles of 16 elements per type)
  whose element counts leave ragged tiles of 16 and of 32, straight and
  curved with walls, Navier-Stokes and Euler, FP32 and FP64;
* hexahedra of order 4 in FP64 for the Euler equations, whose tile does not
  fit a CU: the products run.

The launches of a step are counted, so that tiles cannot be compared with
themselves: with the divergence stage on tiles only a step's first stage has
an interpolation kernel, and no update kernel runs."""
import functools
import math

import numpy as np
import pytest

from gradient_points import read_points
from oracle import fr, mesh as om
from paper_1409_0405_amd import inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

NAMES = ("tet", "pri", "hex")
L3 = (2 * math.pi,) * 3
P0 = 1.0 / (1.4 * 0.09)


@functools.lru_cache(maxsize=None)
def _arrays(kind):
    if kind == "hybrid":           # 36 hexahedra, 144 prisms, 216 tets
        return inputs.hybrid_box(6, 4, 6, 3, 3, L3, jitter=0.1, seed=5)
    if kind == "ragged":           # 6,348 tets, 5,290 prisms: 12 and 10 past whole tiles of 32
        return inputs.small_mixed_box(nxy=23, n_pri_layers=5, n_tet_layers=2, jitter=0.1, seed=5)
    if kind == "hex5":             # 125 hexahedra
        return inputs.hex_box(5, jitter=0.1, seed=5)
    # 4,284 tets, 7,038 prisms, 4,335 hexahedra: 28, 30 and 15 past whole tiles of 32
    return inputs.curve(inputs.hybrid_box(24, 17, 21, 17, 15, L3, jitter=0.1, seed=5, y_bc="wall"), 0.02)


def _bits(x, y):
    it = torch.int64 if x.dtype == torch.float64 else torch.int32
    return torch.equal(x.contiguous().view(it), y.contiguous().view(it))


def _run(kind, p, system, prec, separate, beta=0.5):
    """Residual, flux-point values and steps of one mesh, and the launches of
    one RK45 step by kernel class."""
    from paper_1409_0405_amd import frlib
    arrays = _arrays(kind)
    M = frlib.Mesh(arrays, p, system=system, precision=prec, mu=0.02, ldg_beta=beta, t_wall=P0,
                   p_ref=0.0 if kind == "curved" else P0, separate_update=separate, separate_gradient=separate)
    ts = [t for t in range(3) if M.query(t)["nelem"]]
    u, r = {}, {}
    for t in ts:
        x = M.upts_coords(t)
        U = np.stack(inputs.taylor_green(x[:, 0], x[:, 1], x[:, 2], mach=0.3), 1)
        U[:, 3] += 0.3 * U[:, 0]      # every field nonzero, so that no product vanishes
        u[t] = frlib.to_device_state(M, t, U * inputs.random_perturbation(U.shape, 4, 0.01))
        r[t] = frlib.state_tensor(M, t)
        if separate:                  # the interpolation as a product of its own
            M.set_blocking(t, 0, 2, 0)
        elif system == "ns":
            M.set_gradient_form(t, 1)
    ptr = lambda d: [d[t].data_ptr() if t in d else 0 for t in range(3)]
    M.rhs(ptr(u), ptr(r))
    out = {("rhs", NAMES[t]): r[t][:, :, :M.query(t)["nelem"]] for t in ts}
    for t in ts:
        q = M.query(t)
        for which, nv in ((0, 5), (1, 5)) + (((2, 15),) if system == "ns" else ()):
            f = torch.zeros((q["nfpts"], nv, q["ld"]), dtype=r[t].dtype, device="cuda")
            M.intermediate(t, which, f.data_ptr())
            out[(("state", "flux", "gradient")[which], NAMES[t])] = f[:, :, :q["nelem"]]
        M.set_solution(t, u[t].data_ptr())
    for scheme, n in ((frlib.FR_RK45_2RP, 2), (frlib.FR_RK4, 1), (frlib.FR_FWD_EULER, 2)):
        M.rk_step(scheme, 1e-4, n)
    for t in ts:
        s = frlib.state_tensor(M, t)
        M.get_solution(t, s.data_ptr())
        out[("steps", NAMES[t])] = s[:, :, :M.query(t)["nelem"]]
    M.profile(True)
    M.rk_step(frlib.FR_RK45_2RP, 1e-4, 1)
    count = {k: n for k, (_, n) in M.profile_read().items()}
    torch.cuda.synchronize()
    M.close()
    return out, count, ts


def _compare(kind, p, system, prec, tiles=True, beta=0.5, gradient_mask=None):
    print(f"{kind} p{p} {system} {prec} beta {beta}", flush=True)
    (a, ca, ts), (b, cb, _) = (_run(kind, p, system, prec, sep, beta) for sep in (False, True))
    for t in ts:
        n = NAMES[t]
        assert ca["interp_" + n] == (1 if tiles else 5) and ca["negdivconf_" + n] == 0, (n, ca)
        assert cb["interp_" + n] == 5 and cb["negdivconf_" + n] == 5, (n, cb)
        if system == "ns":
            assert ca["gradflux_" + n] == 5 and ca["grad_" + n] == 0 and cb["grad_" + n] == 5, (n, ca, cb)
    for k, x in a.items():
        y = b[k]
        assert bool(torch.isfinite(y).all()), k
        if k[0] == "gradient":
            if gradient_mask is None:
                continue
            mask = gradient_mask[k[1]]
            assert not bool(torch.where(mask, 0, x).any()), k      # (a fresh mesh: zeros elsewhere)
            x, y = torch.where(mask, x, 0), torch.where(mask, y, 0)
        assert _bits(x, y), k
    return a


@pytest.mark.parametrize("beta", (0.0, -0.5))
@pytest.mark.parametrize("p,prec", [(1, "fp32"), (2, "fp32"), (3, "fp32"), (4, "fp32"), (1, "fp64"), (2, "fp64"),
                                    (3, "fp64"), (4, "fp64")])
def test_ldg_weights(p, prec, beta):
    O = om.build_mesh(_arrays("hybrid"), p)
    # the points whose gradient has a weight: every one, or the sides R
    left = read_points(O)
    mask = {n: torch.from_numpy(np.ascontiguousarray((np.ones_like(m) if beta == 0.0 else ~m).T)).to("cuda")[:, None, :]
            for n, m in left.items()}
    a = _compare("hybrid", p, "ns", prec, beta=beta, gradient_mask=mask)
    if prec == "fp32" or p > 3:
        return
    # against the oracle: 1e-11 of each field's norm, as at beta = 1/2
    U = fr.initial_state(O, inputs.taylor_green, mach=0.3)
    for n in U:
        U[n][..., 3] += 0.3 * U[n][..., 0]
        U[n] = U[n] * np.transpose(inputs.random_perturbation(np.transpose(U[n], (1, 2, 0)).shape, 4, 0.01), (2, 0, 1))
    R = fr.rhs(O, U, fr.Params(system="ns", mu=0.02, beta=beta))
    num, den = np.zeros(5), np.zeros(5)
    for n in R:
        g = np.transpose(a[("rhs", n)].cpu().numpy(), (2, 0, 1))
        num += ((g - R[n]) ** 2).sum(axis=(0, 1))
        den += (R[n] ** 2).sum(axis=(0, 1))
    err = np.sqrt(num / den)
    print("  against the oracle:", err, flush=True)
    assert (err < 1e-11).all(), err


@pytest.mark.parametrize("p,system,prec", [(1, "ns", "fp32"), (2, "ns", "fp32"), (3, "ns", "fp32"), (4, "ns", "fp32"),
                                           (1, "ns", "fp64"), (2, "ns", "fp64"), (3, "ns", "fp64"), (4, "ns", "fp64"),
                                           (1, "euler", "fp32"), (2, "euler", "fp32"), (3, "euler", "fp32"),
                                           (4, "euler", "fp32"), (1, "euler", "fp64"), (2, "euler", "fp64"),
                                           (3, "euler", "fp64"), (4, "euler", "fp64")])
def test_ragged_meshes_above_the_small_launches(p, system, prec):
    n = _arrays("ragged")
    assert all(len(n[k]) > 4096 and len(n[k]) % 16 for k in ("tet_v", "pri_v"))
    _compare("ragged", p, system, prec)


@pytest.mark.parametrize("p,system,prec", [(1, "ns", "fp32"), (2, "ns", "fp32"), (3, "ns", "fp32"), (4, "ns", "fp32"),
                                           (2, "ns", "fp64"), (3, "ns", "fp64"), (2, "euler", "fp32"),
                                           (3, "euler", "fp32"), (4, "euler", "fp32"), (3, "euler", "fp64")])
def test_curved_walls_above_the_small_launches(p, system, prec):
    n = _arrays("curved")
    assert all(len(n[k]) > 4096 and len(n[k]) % 16 for k in ("tet_v", "pri_v", "hex_v"))
    _compare("curved", p, system, prec)


def test_euler_hexahedra_whose_tile_does_not_fit():
    _compare("hex5", 4, "euler", "fp64", tiles=False)
