"""GPU parity of the two inverse-map paths (closed form, and Newton's method
for tighter solver settings or points near a fold of the bilinear map) with
the oracle, on interfaces whose quads are far from parallelograms."""

import numpy as np
import pytest
import scipy.sparse as sp
import torch

import oracle
import synth
from tests.gpu_util import TOL, assert_forward_parity, csr_weights, oracle_params, rel_err, weight_fns

pytestmark = pytest.mark.gpu


def run(itf, seed=None, **kw):
    from paper_2202_03933_amd import MortarInterface, default_params
    print(f"[gpu] {itf.name} {kw}", flush=True)
    it = MortarInterface(itf.slave.X, itf.slave.conn, itf.master.X, itf.master.conn,
                         params=default_params(delta=float(itf.delta), **kw), device="cuda:0")
    it.build_pairs()
    cs, cm, cnv = (t.cpu().numpy() for t in it.candidates())
    ps, pm, nv = (t.cpu().numpy() for t in it.pairs())
    it.csr_pattern()
    D, M, g = it.integrate()
    ns, nm = itf.slave.n_nodes, itf.master.n_nodes
    Dc = sp.csr_matrix((D.cpu().numpy(), it.D_col.cpu().numpy(), it.D_rowptr.cpu().numpy()), shape=(ns, ns))
    Mc = sp.csr_matrix((M.cpu().numpy(), it.M_col.cpu().numpy(), it.M_rowptr.cpu().numpy()), shape=(ns, nm))
    out = {"cand_s": cs, "cand_m": cm, "cand_nv": cnv, "pair_s": ps, "pair_m": pm, "nverts": nv, "D": Dc, "M": Mc,
           "g": g.cpu().numpy(), "stats": it.stats()}
    if seed is not None:
        w = (torch.from_numpy(x).to("cuda:0") for x in csr_weights(Dc, Mc, ns, seed))
        out["grads"] = [x.cpu().numpy().T for x in it.backward(*w)]
    return out


def distorted(seed):
    """Wavy interface, the nodes of both sides moved in plane by up to a
    quarter of an element."""
    itf = synth.wavy(24, 19)
    rng = np.random.default_rng(seed)
    for mesh, n in ((itf.slave, 24), (itf.master, 19)):
        mesh.X[:, :2] += rng.uniform(-0.25 / n, 0.25 / n, size=(mesh.n_nodes, 2))
    return itf


# newton_maxit 30 is the least, and newton_tol 1e-14 the smallest, that the
# closed form serves; one below each runs Newton's method
@pytest.mark.parametrize("kw", [{"newton_maxit": 30}, {"newton_maxit": 29}, {"newton_tol": 9e-15}, {"rule": 3},
                                {"dual": True}, {"dual": True, "newton_maxit": 29}])
def test_distorted_quads(kw):
    itf = distorted(5)
    prm = oracle_params(itf, dual=kw.get("dual", False), rule=kw.get("rule", 7))
    o = oracle.evaluate(itf, prm)
    g = run(itf, seed=3100, **kw)
    assert_forward_parity(g, o)
    w = oracle.pair_weights(itf.slave, itf.master, o["pair_s"], o["pair_m"], *weight_fns(3100))
    g24, _ = oracle.pair_grads(itf.slave, itf.master, prm, o["pair_s"], o["pair_m"], w)
    ref = oracle.scatter_grads(itf.slave, itf.master, o["pair_s"], o["pair_m"], g24)
    for a, b in zip(g["grads"], ref):
        assert rel_err(a, b) <= TOL


# One master quad whose corner at (1/2 + eps, 1/2 + eps) is nearly straight:
# its Jacobian vanishes there with eps, and a slave patch around the corner
# has rule points on both sides of the bound between the two paths (slave
# edge 4e-2: determinants from ~0 to 1/4 of that at the centre).
@pytest.mark.parametrize("eps,opposing", [(1e-3, False), (1e-7, False), (1e-3, True)])
@pytest.mark.parametrize("element_rule", [0, 4])
def test_points_near_a_fold(eps, opposing, element_rule):
    s, t, conn, _ = synth.tensor_grid(7, 6)
    Xs = np.stack([0.4 + 0.25 * s, 0.37 + 0.25 * t, 0.02 * s * t], 1)
    Xm = np.array([[0.0, 0, 0.01], [1, 0, 0.01], [0.5 + eps, 0.5 + eps, 0.02], [0, 1, 0.01]])
    itf = synth.Interface(synth.Mesh(Xs, conn), synth.Mesh(Xm, np.array([[0, 1, 2, 3]], dtype=np.int32)), 0.05,
                          name=f"corner {eps}")
    if opposing:
        itf = synth.opposing(itf)
    prm = oracle_params(itf)
    o = oracle.evaluate(itf, prm)
    g = run(itf, element_rule=element_rule)
    if not element_rule:
        assert_forward_parity(g, o)
        return
    e = oracle.evaluate_elements(itf, element_rule, prm)
    for k in ("D", "M", "g"):
        a, b = (x[k].data if k != "g" else x[k] for x in (g, e))
        assert rel_err(a, b) <= TOL
