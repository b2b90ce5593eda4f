"""Batches and served requests that differ in collision and blended diffusivity:
every member's state, objective and gradient equal its run alone bitwise (the same
device code on the same values)."""
import numpy as np
import pytest
import torch

from paper_1501_04741_amd import inputs
from paper_1501_04741_amd import lbm as L
from paper_1501_04741_amd.lbm import Lbm
from paper_1501_04741_amd.serve import DONE, GpuExecutor, Job, Server

pytestmark = pytest.mark.gpu

HEAT = dict(tau=0.8, tau_s=0.6, u_in=0.02, switch_fn="ramp", switch_param=0.05, c_dp=0.1, c_var=1.0, s_in_lo=0.0,
            s_in_hi=1.0, s_split_axis=1)
KINDS = {
    "d3q19_d3q7": [dict(HEAT, flow=19, scalar=7, nx=33, ny=8, nz=7, **kw)
                   for kw in ({}, dict(collision="mrt"), dict(tau_s_solid=2.0), dict(collision="mrt", tau_s_solid=2.0),
                              dict(tau_s_solid=3.0))],
    "d2q9_d2q5": [dict(HEAT, flow=9, scalar=5, nx=70, ny=21, nz=1, **kw) for kw in (dict(tau_s_solid=2.0), {})],
}


def _alone(p, w, steps, prec, interval, inplace):
    c = Lbm(p, nsteps=steps, precision=prec, checkpoint_interval=interval, inplace=inplace)
    J, g = c.value_and_grad(torch.from_numpy(w))
    return J, g.cpu().numpy()


@pytest.mark.parametrize("inplace", [False, True], ids=["pp", "ip"])
@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_mixed_batch_bitwise_equals_alone(kind, prec, inplace):
    ps, steps = KINDS[kind], 23
    ws = [inputs.porosity(p["nx"], p["ny"], p["nz"], k, 3, np.float32 if prec == "fp32" else np.float64)
          for k, p in enumerate(ps)]
    intervals = [(0, 5, 9)[k % 3] for k in range(len(ps))]
    cs = [Lbm(p, nsteps=steps, precision=prec, checkpoint_interval=i, inplace=inplace) for p, i in zip(ps, intervals)]
    for c, w in zip(cs, ws):
        c.set_design(torch.from_numpy(w))
        c.reset()
    handles = [c.ctx for c in cs]
    for k in (7, 1, steps - 8):
        L.lbm_primal_steps_batch(handles, k, record=True)
    Js = [c.objective()[0] for c in cs]
    for k in (0, 6, steps - 6):
        L.lbm_adjoint_steps_batch(handles, k)
    for c, p, w, i, J in zip(cs, ps, ws, intervals, Js):
        Ja, ga = _alone(p, w, steps, prec, i, inplace)
        assert J == Ja
        assert np.array_equal(c.gradient().cpu().numpy(), ga)


def test_mixed_requests_served_equal_alone_bitwise():
    jobs = [Job(rid=k, params=p, steps=20 + 3 * k, design=inputs.porosity(p["nx"], p["ny"], p["nz"], k, 3),
                precision="fp32", arrival=0.0) for k, p in enumerate(KINDS["d3q19_d3q7"] + KINDS["d2q9_d2q5"])]
    srv = Server(GpuExecutor(), hbm_budget_bytes=4 << 30, quantum=9)
    srv.replay(jobs, realtime=False)
    for j in jobs:
        assert j.state == DONE, (j.rid, j.error)
        J, g = _alone(j.params, np.asarray(j.design, dtype=np.float32), j.steps, "fp32", j.steps, False)
        assert j.J == J and np.array_equal(j.grad, g), j.rid
