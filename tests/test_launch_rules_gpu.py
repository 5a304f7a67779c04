"""The launches that a call makes: steps per launch, block and kernel, read
from a captured graph of the call (nothing of it runs).  Calls that should
take the same form are compared with each other by kernel, so the tests name
no kernel; the rules' reasons stand at rollout_lanes, rollout_spaced and
default_shape.
"""
import ctypes as C

import numpy as np
import pytest

from paper_2308_12698_amd import inputs as I

pytestmark = pytest.mark.gpu


class Dim3(C.Structure):
    _fields_ = [("x", C.c_uint32), ("y", C.c_uint32), ("z", C.c_uint32)]


class KernelNode(C.Structure):
    _fields_ = [("block", Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", Dim3),
                ("params", C.c_void_p), ("shared", C.c_uint)]


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch, torch.device("cuda:0")


@pytest.fixture(scope="module")
def hip(torch_dev):
    torch, dev = torch_dev
    torch.zeros(1, device=dev)
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return C.CDLL(path)


def launches(torch_dev, hip, sim, n, steps, *, mode=1, types=0, perm=False, alive=False, carry=True, gains=False):
    """(kernel, blocks, threads) of every launch of one call on n agents."""
    torch, dev = torch_dev
    st, wp = torch.zeros((30, n), device=dev), torch.zeros((1, 3, n), device=dev)
    ti = torch.zeros(n, dtype=torch.uint8, device=dev) if types else None
    kw = dict(type_idx=ti, perm=sim.order_by_type(ti) if perm else None,
              alive=torch.ones(n, dtype=torch.uint8, device=dev) if alive else None,
              carry=torch.zeros((10, n), device=dev) if carry else None,
              gains=torch.ones((9, n), device=dev) if gains else None,
              wp=wp if mode else None, motor_cmd=None if mode else torch.zeros((4, n), device=dev))
    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    handle, graph = C.c_void_p(stream.cuda_stream), C.c_void_p()
    assert hip.hipStreamBeginCapture(handle, 2) == 0
    try:
        sim.step(st, steps, 1e-3, stream=stream, **kw)
    finally:
        assert hip.hipStreamEndCapture(handle, C.byref(graph)) == 0
    count = C.c_size_t()
    assert hip.hipGraphGetNodes(graph, None, C.byref(count)) == 0
    nodes = (C.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(count)) == 0
    out = []
    for node in nodes:
        p = KernelNode()
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
        out.append((p.func, p.grid.x, p.block.x))
    hip.hipGraphDestroy(graph)
    return out


def simulator(types=None, mode=1, **kw):
    from paper_2308_12698_amd.sim import Simulator
    return Simulator(types or [I.base_type()], I.globals_f32(), mode=mode, **kw)


@pytest.mark.parametrize("n", [5000, 100000, 131073, 200000])
def test_quadrotors_of_a_table_with_vehicles(torch_dev, hip, n):
    """A call without a type index advances quadrotors of type 0, whatever
    else the table holds: the launches of a table of that type alone."""
    one, table = simulator(), simulator([I.base_type(), I.car_type(), I.wing_type()])
    assert launches(torch_dev, hip, one, n, 1000) == launches(torch_dev, hip, table, n, 1000)
    one.close()
    table.close()


@pytest.mark.parametrize("n", [131073, 300000])
@pytest.mark.parametrize("carry", [True, False])
def test_masked_swarms_run_the_form_of_fewer_agents(torch_dev, hip, n, carry):
    """With an alive mask a swarm may hold any number of live agents, all of
    them in a few waves for instance: its launches take the kernel of swarms
    of at most 131,072, and up to 250 steps."""
    sim = simulator()
    few = launches(torch_dev, hip, sim, 131072, 1000, carry=carry)
    masked = launches(torch_dev, hip, sim, n, 1000, carry=carry, alive=True)
    assert [k[0] for k in masked] == 4 * [k[0] for k in few]
    assert {k[0] for k in launches(torch_dev, hip, sim, n, 1000, carry=carry)} != {k[0] for k in few}
    sim.close()


@pytest.mark.parametrize("tuned,other", [(5000, 200000), (5000, 100000), (140000, 5000), (140000, 20000)])
def test_a_tuned_shape_stays_with_its_form(torch_dev, hip, tuned, other):
    """Tuning a swarm of one size fixes the launches of that size and of
    those that run the same form, and leaves the default of the others."""
    torch, dev = torch_dev
    fresh, sim = simulator(), simulator()
    st, wp = torch.zeros((30, tuned), device=dev), torch.zeros((1, 3, tuned), device=dev)
    st[6] = 1.0
    best = sim.autotune(st, 1e-3, probe_steps=25, wp=wp, carry=torch.zeros((10, tuned), device=dev), cache="")
    for n in (tuned, tuned + 7):
        got = launches(torch_dev, hip, sim, n, 100)
        assert [k[2] for k in got] == [best["block"]] * (100 // best["steps_per_launch"])
    assert launches(torch_dev, hip, sim, other, 1000) == launches(torch_dev, hip, fresh, other, 1000)
    fresh.close()
    sim.close()


@pytest.mark.parametrize("kinds,n,threads", [(True, 1000, 512), (True, 65536, 512), (True, 65537, 512),
                                             (True, 131072, 512), (True, 131073, 1024), (False, 16385, 256),
                                             (False, 262144, 256), (False, 262145, 1024)])
def test_blocks_of_grouped_launches(torch_dev, hip, kinds, n, threads):
    """Agents of several kinds, or of one kind with several budgets, in the
    caller's order: the measured block widths, in one launch."""
    types = [I.base_type(), I.car_type(), I.wing_type()] if kinds else [dict(I.base_type(), budget=b) for b in (90, 800)]
    sim = simulator(types)
    got = launches(torch_dev, hip, sim, n, 1000, types=len(types))
    assert len(got) == 1 and got[0][2] == threads and got[0][1] <= -(-n // threads)
    sim.close()
