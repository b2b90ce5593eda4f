"""Several steps of a 2D lattice in one launch, alone and batched, against the
one-step kernels, bitwise (both evaluate the same node expressions in the same
order, so no tolerance): recorded run, recomputed segments, adjoint state and
gradient, at lattices smaller than one region of a tile, of whole tiles, and one
node more or less; and captured calls replayed."""
import numpy as np
import pytest
import torch

from paper_1501_04741_amd import inputs
from paper_1501_04741_amd import lbm as L
from paper_1501_04741_amd.lbm import Lbm

pytestmark = pytest.mark.gpu

FLOW = dict(flow=9, scalar=0, tau=0.8, u_in=0.02, switch_fn="ramp", switch_param=0.05, c_dp=1.0)
HEAT = dict(FLOW, scalar=5, tau_s=0.6, c_hf=0.5, c_var=1.0, s_in_lo=0.0, s_in_hi=1.0, s_split_axis=1)
CASES = [  # parameters, sizes, precision, in place, steps, checkpoint interval
    (FLOW, (5, 4), "fp32", False, 23, 0),
    (FLOW, (129, 33), "fp32", False, 41, 13),
    (FLOW, (256, 128), "fp32", True, 29, 0),
    (dict(FLOW, inlet="pressure", rho_in=1.02, u_cap=0.012), (61, 47), "fp64", True, 33, 11),
    (FLOW, (64, 32), "fp64", False, 30, 7),
    (dict(HEAT, scalar_wall="dirichlet", s_wall=1.0), (97, 31), "fp32", True, 31, 10),
    (dict(HEAT, tau_s_solid=3.0), (130, 65), "fp32", False, 22, 0),
    (dict(HEAT, periodic=1, c_dp=0.0, c_hf=0.0, c_var=0.0), (7, 12), "fp64", False, 19, 6),
    (HEAT, (48, 96), "fp64", True, 24, 9),
]


def _context(p, size, prec, inplace, steps, interval, seed):
    w = torch.from_numpy(inputs.porosity(size[0], size[1], 1, seed, 3, np.float32 if prec == "fp32" else np.float64))
    c = Lbm(dict(p, nx=size[0], ny=size[1], nz=1), nsteps=steps, precision=prec, checkpoint_interval=interval,
            inplace=inplace)
    c.set_design(w)
    c.reset()
    return c


def _arrays(*groups):
    return [t.cpu().numpy() for g in groups for t in g if t is not None]


def _same(a, b):
    assert len(a) == len(b) and all(np.array_equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("batch", [False, True], ids=["alone", "batch"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "d2q9%s_%dx%d_%s" % (("_d2q5" if c[0]["scalar"] else "",) + c[1] + c[2:3]))
def test_many_steps_per_launch_bitwise_equal_one(case, batch):
    p, (nx, ny), prec, inplace, steps, interval = case
    sizes = [(nx, ny), (nx + 1, ny), (2 * nx, ny + 3)] if batch else [(nx, ny)]
    ones = [_context(p, s, prec, inplace, steps, interval, k) for k, s in enumerate(sizes)]
    many = [_context(p, s, prec, inplace, steps, interval, k) for k, s in enumerate(sizes)]
    for c in ones:
        for _ in range(steps):
            c.primal_steps(1, record=True)
    handles = [c.ctx for c in many]
    for k in (1, steps - 3, 2):  # an odd start, and a call that ends amid a segment
        if batch:
            L.lbm_primal_steps_batch(handles, k, record=True)
        else:
            many[0].primal_steps(k, record=True)
    for a, b in zip(ones, many):
        _same(_arrays(a.get_state(), a.fields()), _arrays(b.get_state(), b.fields()))
        assert a.objective() == b.objective()
    for k in (steps - 6, 1, 5):
        for c in ones:
            for _ in range(k):
                c.adjoint_steps(1)
        if batch:
            L.lbm_adjoint_steps_batch(handles, k)
        else:
            many[0].adjoint_steps(k)
        for a, b in zip(ones, many):
            _same(_arrays(a.get_adjoint()), _arrays(b.get_adjoint()))
    for a, b in zip(ones, many):
        _same(_arrays([a.gradient()]), _arrays([b.gradient()]))


@pytest.mark.parametrize("inplace", [False, True])
def test_captured_even_call_replays(inplace):
    """An even number of steps leaves the state in the buffer it came from, whatever
    the number of launches: the captured call advances the state again on each replay."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        w = torch.from_numpy(inputs.porosity(100, 60, 1, 0, 3, np.float32))
        a, b = [Lbm(dict(FLOW, nx=100, ny=60, nz=1), nsteps=0, precision="fp32", inplace=inplace, stream=stream)
                for _ in range(2)]
        for c in (a, b):
            c.set_design(w)
            c.reset()
            c.primal_steps(18)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            b.primal_steps(18)
        for _ in range(3):
            graph.replay()
            a.primal_steps(18)
            stream.synchronize()
            _same(_arrays(a.get_state()), _arrays(b.get_state()))


def _steps(c, batch, call, *args):
    if batch:
        getattr(L, "lbm_%s_steps_batch" % call)([c.ctx], *args)
    else:
        getattr(c, call + "_steps")(*args)


@pytest.mark.parametrize("batch", [False, True], ids=["alone", "batch"])
def test_captured_inplace_steps_replayed_between_oneshot_iterations(batch):
    """The adjoint buffer is free when the primal steps are captured and holds the
    one-shot iteration's cotangent when the graph is replayed."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        w = torch.from_numpy(inputs.porosity(100, 60, 1, 0, 3, np.float32))
        a, b = [Lbm(dict(HEAT, nx=100, ny=60, nz=1), nsteps=0, precision="fp32", inplace=True, stream=stream)
                for _ in range(2)]
        for c in (a, b):
            c.set_design(w)
            c.reset()
            c.primal_steps(4)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            _steps(b, batch, "primal", 18)
        for _ in range(3):
            graph.replay()
            a.primal_steps(18)
            for c in (a, b):
                c.oneshot_steps(6, 1e-3)
            stream.synchronize()
            _same(_arrays(a.get_state(), a.get_adjoint(), [a.design(), a.gradient()]),
                  _arrays(b.get_state(), b.get_adjoint(), [b.design(), b.gradient()]))


@pytest.mark.parametrize("batch", [False, True], ids=["alone", "batch"])
def test_captured_inplace_adjoint_replays_from_the_recorded_state(batch):
    """Each replay of a captured adjoint seeds from the state that the run ended in."""
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        w = torch.from_numpy(inputs.porosity(100, 60, 1, 0, 3, np.float32))
        a, b = [Lbm(dict(HEAT, nx=100, ny=60, nz=1), nsteps=400, precision="fp32", inplace=True, stream=stream)
                for _ in range(2)]
        for c in (a, b):
            c.set_design(w)
            c.reset()
            c.primal_steps(400, record=True)
        a.adjoint_steps(400)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            _steps(b, batch, "adjoint", 400)
        for _ in range(3):
            graph.replay()
            stream.synchronize()
            _same(_arrays(a.get_adjoint(), [a.gradient()]), _arrays(b.get_adjoint(), [b.gradient()]))


@pytest.mark.parametrize("size, prec, inplace, solid", [
    ((1021, 509), "fp32", False, 3.0), ((1024, 512), "fp32", True, 3.0), ((701, 353), "fp64", True, 0.0),
    ((704, 352), "fp64", True, 3.0)], ids=["vd_pp", "vd_ip", "fp64_ip", "fp64_vd_ip"])
def test_tiles_of_whole_rows_bitwise_equal_one_step_launches(size, prec, inplace, solid):
    """States beyond the L2s with D2Q5: recorded runs (and all in place in FP64) take tiles of
    whole 64-byte rows, the blended FP32 adjoint in place one step per launch."""
    one, many = [_context(dict(HEAT, tau_s_solid=solid), size, prec, inplace, 16, 0, 0) for _ in range(2)]
    for _ in range(16):
        one.primal_steps(1, record=True)
    many.primal_steps(16, record=True)
    _same(_arrays(one.get_state()), _arrays(many.get_state()))
    for _ in range(16):
        one.adjoint_steps(1)
    many.adjoint_steps(16)
    _same(_arrays(one.get_adjoint(), [one.gradient()]), _arrays(many.get_adjoint(), [many.gradient()]))


@pytest.mark.parametrize("batch", [False, True], ids=["alone", "batch"])
@pytest.mark.parametrize("case", [c for c in CASES if c[5]], ids=lambda c: "%dx%d_%s" % (c[1] + c[2:3]))
def test_recomputed_segments_bitwise_equal_a_run_that_recomputes_nothing(case, batch):
    """The reference holds every step's moments and takes one step per call; the segments of
    the others, recomputed in launches of several steps, start at odd and at even times."""
    p, (nx, ny), prec, inplace, steps, interval = case
    sizes = [(nx, ny), (nx + 1, ny), (2 * nx, ny + 3)] if batch else [(nx, ny)]
    whole = [_context(p, s, prec, inplace, steps, steps, k) for k, s in enumerate(sizes)]
    parts = [_context(p, s, prec, inplace, steps, interval, k) for k, s in enumerate(sizes)]
    assert whole[0].plan()["interval"] == steps and parts[0].plan()["interval"] == interval
    handles = [c.ctx for c in parts]
    for c in whole:
        for _ in range(steps):
            c.primal_steps(1, record=True)
    if batch:
        L.lbm_primal_steps_batch(handles, steps, record=True)
    else:
        parts[0].primal_steps(steps, record=True)
    for k in (interval + 3, 1, steps - interval - 4):
        for c in whole:
            for _ in range(k):
                c.adjoint_steps(1)
        if batch:
            L.lbm_adjoint_steps_batch(handles, k)
        else:
            parts[0].adjoint_steps(k)
        for a, b in zip(whole, parts):
            _same(_arrays(a.get_adjoint()), _arrays(b.get_adjoint()))
    for a, b in zip(whole, parts):
        _same(_arrays([a.gradient()]), _arrays([b.gradient()]))
