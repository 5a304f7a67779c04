"""Parity of the HIP path (through the C ABI) with the FP64 reference.

Tolerance: relative state error <= 1e-4 per agent and state group after the
stated number of steps (groups and floors in tests/_util.py).  Determinism
and decomposition checks compare GPU results with each other bitwise: each
lane's arithmetic does not depend on the launch shape, so any difference
would expose an indexing, LDS or ordering bug.
"""
import numpy as np
import pytest

from paper_2308_12698_amd import inputs as I
from tests._util import OPEN_LOOP_GROUPS, rel_errors

pytestmark = pytest.mark.gpu

TOL = 1e-4


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch, torch.device("cuda:0")


def _dev(torch, dev, a):
    return None if a is None else torch.from_numpy(np.ascontiguousarray(a)).to(dev)


def gpu_rollout(torch_dev, sw, n_steps, form="fused", state=None, sim=None, step0=0, ld=None,
                carry=True, **opts):
    """Run the workload on the GPU.  ``state`` (default the workload's) has
    30 rows, or 40 with its rounding carries in rows 30-39.  With ``carry``
    the call keeps the carries in a buffer and the result is float64 [40, N]
    (state, then carries); without, the updates are uncompensated and the
    result is [30, N].  ``ld`` > N pads both buffers with columns of 7.0."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    own = sim is None
    if own:
        sim = Simulator(sw.types, sw.glob, mode=sw.mode, form=form, debug=True, **opts)
    s0 = sw.state if state is None else state
    n = s0.shape[1]
    c0 = s0[30:40] if s0.shape[0] == 40 else np.zeros((10, n), dtype=np.float32)
    s0 = s0[:30]
    if ld is not None and ld > n:
        buf = np.full((30, ld), 7.0, dtype=np.float32)
        buf[:, :n] = s0
        s0 = buf
        cbuf = np.full((10, ld), 7.0, dtype=np.float32)
        cbuf[:, :n] = c0
        c0 = cbuf
    st = _dev(torch, dev, s0)
    ct = _dev(torch, dev, c0) if carry else None
    sim.step(st, n_steps, sw.dt, n_agents=n, type_idx=_dev(torch, dev, sw.type_idx),
             gains=_dev(torch, dev, sw.gains), motor_cmd=_pad(torch, dev, sw.motor_cmd, st.shape[1]),
             wp=_pad3(torch, dev, sw.wp, st.shape[1]), resample_every=sw.resample_every, step0=step0,
             carry=ct)
    torch.cuda.synchronize()
    out = st.cpu().numpy()
    if carry:
        out = np.concatenate([out, ct.cpu().numpy()])
    if own:
        sim.close()
    return out.astype(np.float64)


def carry_zeros(torch_dev, n):
    torch, dev = torch_dev
    return torch.zeros((10, n), dtype=torch.float32, device=dev)


def _pad(torch, dev, a, ld):
    if a is None:
        return None
    if a.shape[-1] == ld:
        return _dev(torch, dev, a)
    b = np.zeros(a.shape[:-1] + (ld,), dtype=a.dtype)
    b[..., :a.shape[-1]] = a
    return _dev(torch, dev, b)


_pad3 = _pad


def oracle_rollout(oracle, sw, n_steps, state=None, step0=0):
    s = sw.state if state is None else state
    return oracle.rollout(s, sw.types, sw.glob, sw.mode, sw.dt, n_steps, type_idx=sw.type_idx,
                          gains=sw.gains, motor_cmd=sw.motor_cmd, wp=sw.wp,
                          resample_every=sw.resample_every, step0=step0)


def assert_parity(got, ref, sw, groups=None, tol=TOL):
    errs = rel_errors(got, ref, sw.types, sw.type_idx, groups)
    worst = max(v[0] for v in errs.values())
    print("parity", sw.name, {k: f"{v[0]:.2e}" for k, v in errs.items()}, flush=True)
    assert worst <= tol, errs


# --- parity with the oracle --------------------------------------------------

@pytest.mark.parametrize("form", ["plain", "fused"])
def test_open_loop_1000_agents_1000_steps(oracle, torch_dev, form):
    sw = I.config0()
    got = gpu_rollout(torch_dev, sw, 1000, form=form, steps_per_launch=128)
    ref = oracle_rollout(oracle, sw, 1000)
    assert_parity(got, ref, sw, OPEN_LOOP_GROUPS)
    # rows the open loop does not own are left alone (state rows 17-29, the
    # carries of J and of the position-loop integral)
    assert np.array_equal(got[17:30], sw.state[17:30].astype(np.float64))
    assert not got[36:].any()


def test_open_loop_full_size_every_agent(oracle, torch_dev):
    """The open-loop swarm at 1,048,576 agents, 1,000 steps, in the plain
    form (1,000 launches) and the fused form: the two agree bit for bit and
    every agent matches the oracle."""
    sw = I.config0(n=1 << 20)
    plain = gpu_rollout(torch_dev, sw, 1000, form="plain", block=128)
    fused = gpu_rollout(torch_dev, sw, 1000, form="fused", steps_per_launch=250)
    assert np.array_equal(plain, fused)
    ref = oracle_rollout(oracle, sw, 1000)
    assert_parity(fused, ref, sw, OPEN_LOOP_GROUPS)


@pytest.mark.parametrize("form", ["plain", "fused"])
def test_closed_loop_5000_agents_1000_steps(oracle, torch_dev, form):
    sw = I.config1()
    got = gpu_rollout(torch_dev, sw, 1000, form=form, steps_per_launch=100)
    ref = oracle_rollout(oracle, sw, 1000)
    assert_parity(got, ref, sw)


def test_closed_loop_10000_steps_sampled(oracle, torch_dev):
    """The full closed-loop rollout length, on a sample of agents."""
    sw = I.subset(I.config1(), np.arange(0, 5000, 5))
    got = gpu_rollout(torch_dev, sw, 10000, steps_per_launch=250)
    ref = oracle_rollout(oracle, sw, 10000)
    assert_parity(got, ref, sw)


def test_waypoint_epochs_ragged_agents(oracle, torch_dev):
    """Epoch switches that fall inside launches, a ragged agent count and a
    padded leading dimension."""
    sw = I.config2(n=3 * 256 + 37, n_steps=2500, resample_every=700)
    got = gpu_rollout(torch_dev, sw, 2500, steps_per_launch=333, block=128, ld=1024)
    ref = oracle_rollout(oracle, sw, 2500)
    assert_parity(got[:, :sw.n], ref, sw)
    assert np.all(got[:, sw.n:] == 7.0)            # columns past n_agents untouched


@pytest.mark.parametrize("form", ["plain", "fused"])
def test_controller_limits_match_oracle(oracle, torch_dev, form):
    """Agents held at the rotor speed limit, at the vertical-acceleration
    floor, with attitude and rate integrals in their clamps and rotors at 0
    and the limit, and tumbling towards far waypoints (inputs.limits_swarm),
    with per-agent gains; every agent against the oracle after 1,000 steps."""
    sw = I.limits_swarm()
    got = gpu_rollout(torch_dev, sw, sw.n_steps, form=form, steps_per_launch=250)
    ref = oracle_rollout(oracle, sw, sw.n_steps)
    for k, name in enumerate(sw.extra["groups"]):
        idx = np.arange(k * sw.n // 4, (k + 1) * sw.n // 4)
        sub = I.subset(sw, idx)
        print(name, end=" ")
        assert_parity(got[:, idx], ref[:, idx], sub)


def test_arbitrary_attitudes_match_oracle(oracle, torch_dev):
    """Attitudes drawn uniformly over all rotations, stored with either sign
    of the scalar part (half start upside down or with attitude errors past
    a half turn, so the short-arc choice of the error quaternion is taken
    from the first step), body rates up to 3 rad/s, waypoints 2 m away:
    every agent against the oracle after 1,000 steps."""
    sw = I.config1(n=512, n_steps=1000)
    r = np.random.default_rng(41)
    q = r.normal(size=(4, sw.n))
    q /= np.linalg.norm(q, axis=0)
    st = sw.state.astype(np.float64)
    st[6:10] = q
    st[10:13] = r.uniform(-3.0, 3.0, (3, sw.n))
    st[26:29] = st[10:13]
    d = r.normal(size=(3, sw.n))
    wp = st[0:3] + 2.0 * d / np.linalg.norm(d, axis=0)
    sw = I.Swarm(sw.name, sw.mode, sw.dt, sw.n_steps, I.f32(st), sw.types, sw.glob, wp=I.f32(wp[None]))
    assert (sw.state[6] < 0).sum() > 100
    got = gpu_rollout(torch_dev, sw, 1000, steps_per_launch=250)
    ref = oracle_rollout(oracle, sw, 1000)
    assert_parity(got, ref, sw)


def test_scale_workload_full_size_every_agent(oracle, torch_dev):
    """1,048,576 agents, 1,000 steps with the bench's launch shape (tuned,
    graph-captured); every agent against the oracle (about 1e9 FP64
    agent-steps on the host's cores)."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config2()
    sim = Simulator(sw.types, sw.glob, mode=1, form="fused", use_graph=True)
    st = _dev(torch, dev, sw.state)
    ct = carry_zeros(torch_dev, sw.n)
    wp = _dev(torch, dev, sw.wp)
    sim.autotune(st, sw.dt, 200, wp=wp, resample_every=sw.resample_every, carry=ct)
    sim.step(st, 1000, sw.dt, wp=wp, resample_every=sw.resample_every, carry=ct)
    torch.cuda.synchronize()
    got = st.cpu().numpy().astype(np.float64)
    sim.close()
    assert np.isfinite(got).all()
    ref = oracle_rollout(oracle, sw, 1000)
    assert_parity(got[:30], ref, sw)


def test_heterogeneous_batch_matches_oracle(oracle, torch_dev):
    """Eight types, step budgets 1,000-8,000, one launch, with and without the
    type-grouped processing order."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config3(scale=256)
    ref = oracle_rollout(oracle, sw, sw.n_steps)
    for use_perm in (False, True):
        sim = Simulator(sw.types, sw.glob, mode=1, form="fused", steps_per_launch=sw.n_steps,
                        debug=True)
        st = _dev(torch, dev, sw.state)
        ti = _dev(torch, dev, sw.type_idx)
        perm = sim.order_by_type(ti) if use_perm else None
        sim.step(st, sw.n_steps, sw.dt, type_idx=ti, perm=perm, wp=_dev(torch, dev, sw.wp),
                 resample_every=sw.resample_every, carry=carry_zeros(torch_dev, sw.n))
        torch.cuda.synchronize()
        got = st.cpu().numpy().astype(np.float64)
        sim.close()
        assert_parity(got, ref, sw)


def test_heterogeneous_full_size_every_agent(oracle, torch_dev):
    """The full heterogeneous swarm (1,007,616 agents, 8 types) for its
    first 1,000 steps in the type order, one launch: every agent against the
    oracle (about 1e9 FP64 agent-steps on the host); the same launch in the
    caller's order (grouped per block) gives the same bits."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config3()
    sim = Simulator(sw.types, sw.glob, mode=1, form="fused", steps_per_launch=1000)
    st = _dev(torch, dev, sw.state)
    ti = _dev(torch, dev, sw.type_idx)
    perm = sim.order_by_type(ti)
    sim.step(st, 1000, sw.dt, type_idx=ti, perm=perm, wp=_dev(torch, dev, sw.wp),
             resample_every=sw.resample_every, carry=carry_zeros(torch_dev, sw.n))
    # the caller's order: each block groups its agents by budget class
    su = _dev(torch, dev, sw.state)
    sim.step(su, 1000, sw.dt, type_idx=ti, wp=_dev(torch, dev, sw.wp), resample_every=sw.resample_every,
             carry=carry_zeros(torch_dev, sw.n))
    torch.cuda.synchronize()
    assert torch.equal(st, su)
    del su
    got = st.cpu().numpy().astype(np.float64)
    sim.close()
    assert np.isfinite(got).all()
    ref = oracle_rollout(oracle, sw, 1000)
    assert_parity(got[:30], ref, sw)


def test_hover_fixed_point_on_gpu(torch_dev):
    """wp = p, level, at rest, rotors at the reference speed: nothing moves
    beyond FP32 rounding of the hover balance."""
    sw = I.config1(n=512)
    sw.wp = sw.state[0:3][None].copy()
    got = gpu_rollout(torch_dev, sw, 1000)
    assert np.abs(got[0:3] - sw.state[0:3]).max() <= 1e-4        # positions ~ 100 m
    assert np.abs(got[3:6]).max() <= 1e-5
    assert np.abs(got[10:13]).max() <= 1e-5
    assert np.abs(got[13:17]).max() <= 1e-3                        # rad/s around ~634
    assert np.abs(got[6] - 1.0).max() <= 1e-6


@pytest.mark.parametrize("mode,form", [(1, "plain"), (1, "fused"), (0, "fused")])
def test_nothing_is_written_past_the_state_and_carry_rows(oracle, torch_dev, mode, form):
    """The state is 30 rows and the carries 10: both sit at the top of
    larger buffers whose extra rows are guard rows holding a sentinel; after
    the rollout (10,000 steps closed loop) every guard element is the
    sentinel bit for bit and the state matches the oracle."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.subset(I.config1(), np.arange(0, 5000, 10)) if mode == 1 else I.config0(n=500)
    n_steps = 10000 if mode == 1 else 1000
    n, guard, sentinel = sw.n, 6, -12345.678
    buf = torch.full((30 + guard, n), sentinel, dtype=torch.float32, device=dev)
    cbuf = torch.full((10 + guard, n), sentinel, dtype=torch.float32, device=dev)
    buf[:30] = _dev(torch, dev, sw.state)
    cbuf[:10] = 0.0
    st, ct = buf[:30], cbuf[:10]
    assert st.is_contiguous() and ct.is_contiguous()
    sim = Simulator(sw.types, sw.glob, mode=mode, form=form, steps_per_launch=500)
    sim.step(st, n_steps, sw.dt, wp=_dev(torch, dev, sw.wp), motor_cmd=_dev(torch, dev, sw.motor_cmd),
             carry=ct)
    torch.cuda.synchronize()
    sim.close()
    assert bool((buf[30:] == sentinel).all()) and bool((cbuf[10:] == sentinel).all())
    ref = oracle_rollout(oracle, sw, n_steps)
    assert_parity(buf[:30].cpu().numpy().astype(np.float64), ref, sw,
                  None if mode == 1 else OPEN_LOOP_GROUPS)


def test_uncompensated_updates_without_a_carry_buffer(oracle, torch_dev):
    """Without a carry buffer the integrator's updates are plain FP32 sums
    (the documented accuracy of that mode: ~1e-4 relative after 1,000 steps
    of the closed-loop swarm, ~2e-3 after 10,000); with carries the same
    runs stay near 1e-6.  Both results are printed."""
    sw = I.config1()
    ref = oracle_rollout(oracle, sw, 1000)
    plain = gpu_rollout(torch_dev, sw, 1000, carry=False, steps_per_launch=250)
    comp = gpu_rollout(torch_dev, sw, 1000, carry=True, steps_per_launch=250)
    e_plain = max(v[0] for v in rel_errors(plain, ref, sw.types).values())
    e_comp = max(v[0] for v in rel_errors(comp, ref, sw.types).values())
    sub = I.subset(sw, np.arange(0, 5000, 10))
    ref10 = oracle_rollout(oracle, sub, 10000)
    e10 = max(v[0] for v in rel_errors(gpu_rollout(torch_dev, sub, 10000, carry=False, steps_per_launch=500),
                                      ref10, sub.types).values())
    print(f"without carries: {e_plain:.2e} (1,000 steps), {e10:.2e} (10,000 steps); "
          f"with: {e_comp:.2e} (1,000 steps)", flush=True)
    assert e_comp <= TOL and e_plain <= 1e-3 and e10 <= 2e-2
    assert e_comp < e_plain


# --- GPU-side invariants and decompositions -------------------------------------

def test_launch_shape_does_not_change_results(torch_dev):
    sw = I.config2(n=2000, n_steps=600, resample_every=250)
    base = gpu_rollout(torch_dev, sw, 600, form="fused", block=256, steps_per_launch=100)
    for kw in (dict(form="plain", block=64), dict(form="fused", block=512, steps_per_launch=7),
               dict(form="fused", block=64, steps_per_launch=600, grid_blocks=5),
               dict(form="fused", block=128, steps_per_launch=50, use_graph=True)):
        assert np.array_equal(gpu_rollout(torch_dev, sw, 600, **kw), base), kw


def test_split_rollout_is_bitwise_equal(torch_dev):
    sw = I.config2(n=1500, n_steps=1000, resample_every=300)
    full = gpu_rollout(torch_dev, sw, 1000, steps_per_launch=64)
    half = gpu_rollout(torch_dev, sw, 450, steps_per_launch=64).astype(np.float32)
    rest = gpu_rollout(torch_dev, sw, 550, state=half, step0=450, steps_per_launch=64)
    assert np.array_equal(full, rest)


def test_graph_replay_matches_eager(torch_dev):
    """A cached hipGraph replayed several times, with eager work between
    replays, gives the eager result each time."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config1(n=3000)
    wp = _dev(torch, dev, sw.wp)
    eager = Simulator(sw.types, sw.glob, mode=1, steps_per_launch=40)
    graph = Simulator(sw.types, sw.glob, mode=1, steps_per_launch=40, use_graph=True)
    a = _dev(torch, dev, sw.state)
    b = _dev(torch, dev, sw.state)
    ca, cb = carry_zeros(torch_dev, sw.n), carry_zeros(torch_dev, sw.n)
    for _ in range(4):
        eager.step(a, 200, sw.dt, wp=wp, carry=ca)
        graph.step(b, 200, sw.dt, wp=wp, carry=cb)
        torch.cuda.synchronize()
        assert torch.equal(a, b) and torch.equal(ca, cb)
        a.mul_(1.0)                    # eager work between replays
    eager.close(); graph.close()


def test_types_match_single_type_runs(torch_dev):
    """Each type's agents in the mixed launch equal a run of the same agents
    with that type alone: bitwise through the same (type-indexed) kernel,
    and to FP32 rounding through the homogeneous kernel, whose compiled
    instruction sequence (FMA contraction) may differ."""
    sw = I.config3(scale=512)
    mixed = gpu_rollout(torch_dev, sw, sw.n_steps, steps_per_launch=1000)
    for t in range(len(sw.types)):
        idx = np.where(sw.type_idx == t)[0]
        sub = I.subset(sw, idx)
        sub.types = [sw.types[t]]
        sub.type_idx = np.zeros(idx.size, dtype=np.uint8)
        alone = gpu_rollout(torch_dev, sub, sw.n_steps, steps_per_launch=1000)
        assert np.array_equal(mixed[:, idx], alone), t
        sub.type_idx = None
        homo = gpu_rollout(torch_dev, sub, sw.n_steps, steps_per_launch=1000)
        assert_parity(homo, alone, sub, tol=1e-5)


def test_grouped_launch_equals_the_type_order(torch_dev):
    """In the caller's order the eight types (eight step budgets, so eight
    classes) are grouped within each block; the result equals the
    type-ordered launch bit for bit, whatever the launch shape (one round of
    blocks, one block holding several chunks, two 1024-thread blocks,
    64-thread blocks with a few chunks each, a captured graph, one step per
    launch), also with dead
    agents, which stay as they were."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config3(scale=300)
    steps = 2500

    def run(ordered, alive=None, **opts):
        sim = Simulator(sw.types, sw.glob, mode=1, debug=True, **opts)
        st = _dev(torch, dev, sw.state)
        ti = _dev(torch, dev, sw.type_idx)
        perm = sim.order_by_type(ti) if ordered else None
        sim.step(st, steps, sw.dt, type_idx=ti, perm=perm, wp=_dev(torch, dev, sw.wp),
                 resample_every=sw.resample_every, carry=carry_zeros(torch_dev, sw.n),
                 alive=_dev(torch, dev, alive))
        torch.cuda.synchronize()
        out = st.cpu().numpy()
        sim.close()
        return out

    print(f"grouped launch: {sw.n} agents, {steps} steps", flush=True)
    ref = run(True, form="fused", steps_per_launch=500)
    for opts in (dict(form="fused", steps_per_launch=500),
                 dict(form="fused", block=512, steps_per_launch=1000, grid_blocks=1),
                 dict(form="fused", block=1024, steps_per_launch=1000, grid_blocks=2),
                 dict(form="fused", block=64, steps_per_launch=2500, grid_blocks=3),
                 dict(form="fused", block=128, steps_per_launch=250, use_graph=True),
                 dict(form="plain")):
        assert np.array_equal(run(False, **opts), ref), opts
    alive = (np.arange(sw.n) % 7 != 3).astype(np.uint8)
    got = run(False, alive, form="fused", steps_per_launch=1000)
    assert np.array_equal(got, run(True, alive, form="fused", steps_per_launch=1000))
    assert np.array_equal(got[:, alive == 0], sw.state[:, alive == 0])


def test_grouped_launch_with_per_agent_gains(oracle, torch_dev):
    """Per-agent gains beside three budget classes, in the caller's order:
    the per-block grouping carries each agent's gains with it (bitwise the
    type order; within 1e-4 of the oracle)."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    dw = I.config4(n=3000, n_steps=600)
    types = [dict(t, budget=b) for t, b in zip(I.hetero_types(3, seed_stream=2), (600, 250, 430))]
    labels = np.random.default_rng(4).integers(0, 3, dw.n).astype(np.uint8)
    sw = I.Swarm("gains3", 1, dw.dt, 600, dw.state, types, dw.glob, type_idx=labels, gains=dw.gains, wp=dw.wp,
                 resample_every=0)
    outs = []
    for ordered in (False, True):
        sim = Simulator(types, sw.glob, mode=1, steps_per_launch=200, debug=True)
        st = _dev(torch, dev, sw.state)
        ti = _dev(torch, dev, labels)
        sim.step(st, 600, sw.dt, type_idx=ti, perm=sim.order_by_type(ti) if ordered else None,
                 gains=_dev(torch, dev, sw.gains), wp=_dev(torch, dev, sw.wp), carry=carry_zeros(torch_dev, sw.n))
        torch.cuda.synchronize()
        outs.append(st.cpu().numpy())
        sim.close()
    assert np.array_equal(outs[0], outs[1])
    assert_parity(outs[0].astype(np.float64), oracle_rollout(oracle, sw, 600), sw)


def test_ungrouped_launch_beyond_eight_classes(oracle, torch_dev):
    """Twelve types of twelve step budgets (more classes than a block
    groups): the caller's order runs the launch's plain 64-agent groups,
    bitwise equal to the type order and within 1e-4 of the oracle."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    types = I.hetero_types(12, seed_stream=5)
    for t, ty in enumerate(types):
        ty["budget"] = 100 * (t + 1)
    r = I.rng(3, 7)
    n = 2500
    labels = r.integers(0, 12, n).astype(np.uint8)
    state = I.hover_state(I._box_positions(r, n))
    wp = I.f32(I._box_positions(r, n)[None])
    sw = I.Swarm("twelve", 1, 1e-3, 1200, state, types, I.globals_f32(), type_idx=labels, wp=wp,
                 resample_every=0)
    outs = []
    for ordered in (False, True):
        sim = Simulator(types, sw.glob, mode=1, steps_per_launch=400, debug=True)
        st = _dev(torch, dev, state)
        ti = _dev(torch, dev, labels)
        sim.step(st, 1200, sw.dt, type_idx=ti, perm=sim.order_by_type(ti) if ordered else None,
                 wp=_dev(torch, dev, wp), carry=carry_zeros(torch_dev, n))
        torch.cuda.synchronize()
        outs.append(st.cpu().numpy())
        sim.close()
    assert np.array_equal(outs[0], outs[1])
    ref = oracle_rollout(oracle, sw, 1200)
    assert_parity(outs[0].astype(np.float64), ref, sw)


def test_order_by_type_is_the_stable_budget_order(torch_dev):
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config3(scale=16)
    sim = Simulator(sw.types, sw.glob, mode=1)
    perm = sim.order_by_type(_dev(torch, dev, sw.type_idx)).cpu().numpy()
    sim.close()
    budgets = np.array([t["budget"] for t in sw.types])
    rank = np.argsort(np.argsort(-budgets, kind="stable"), kind="stable")
    expect = np.lexsort((np.arange(sw.n), rank[sw.type_idx]))
    assert np.array_equal(perm, expect)


def test_out_of_range_type_and_order_entries(torch_dev):
    """The device clamps a type index >= n_types to the last type and an
    order entry outside [0, n) to the last agent, so bad inputs address
    nothing outside the table and the state rows."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config3(scale=256)
    n, steps = sw.n, 300
    bad_types = sw.type_idx.copy()
    bad_types[::50] = 200
    clamped = np.minimum(bad_types, len(sw.types) - 1).astype(np.uint8)
    sim = Simulator(sw.types, sw.glob, mode=1, steps_per_launch=100)
    wp = _pad3(torch, dev, sw.wp, n)
    runs = {}
    for label, ti in (("bad", bad_types), ("clamped", clamped)):
        st = _dev(torch, dev, sw.state)
        t = _dev(torch, dev, ti)
        perm = sim.order_by_type(t)
        sim.step(st, steps, sw.dt, type_idx=t, perm=perm, wp=wp, resample_every=sw.resample_every)
        runs[label] = (st.cpu().numpy(), perm.cpu().numpy())
    assert np.array_equal(runs["bad"][1], runs["clamped"][1])
    assert np.array_equal(np.sort(runs["bad"][1]), np.arange(n))
    assert np.array_equal(runs["bad"][0], runs["clamped"][0])
    # an order that is not a permutation: entries 5 and 6 point outside [0, n)
    perm = np.arange(n, dtype=np.int32)
    perm[5], perm[6] = np.iinfo(np.int32).max, -3
    t = _dev(torch, dev, clamped)
    st = _dev(torch, dev, sw.state)
    sim.step(st, steps, sw.dt, type_idx=t, perm=_dev(torch, dev, perm), wp=wp, resample_every=sw.resample_every)
    ref = _dev(torch, dev, sw.state)
    sim.step(ref, steps, sw.dt, type_idx=t, perm=_dev(torch, dev, np.arange(n, dtype=np.int32)), wp=wp,
             resample_every=sw.resample_every)
    torch.cuda.synchronize()
    got, want = st.cpu().numpy(), ref.cpu().numpy()
    sim.close()
    keep = np.ones(n, bool)
    keep[[5, 6, n - 1]] = False        # 5, 6: no lane; n - 1: three lanes
    assert np.array_equal(got[:, keep], want[:, keep])
    assert np.array_equal(got[:, [5, 6]], sw.state[:, [5, 6]])
    assert np.isfinite(got[:30]).all()


def test_budget_zero_and_nan_agents(torch_dev):
    sw = I.config1(n=700)
    t0 = dict(sw.types[0]); t0["budget"] = 0
    sw.types = [sw.types[0], t0]
    sw.type_idx = (np.arange(700) % 3 == 0).astype(np.uint8)
    bad = sw.state.copy()
    bad[3, 5] = np.nan
    got = gpu_rollout(torch_dev, sw, 300, state=bad)
    frozen = sw.type_idx == 1
    assert np.array_equal(got[:30, frozen], bad[:, frozen].astype(np.float64))
    assert not got[30:, frozen].any()
    clean = gpu_rollout(torch_dev, sw, 300)
    keep = np.arange(700) != 5
    assert np.array_equal(got[:, keep], clean[:, keep])
    assert np.isnan(got[:, 5]).any()


def test_count_nonfinite_agents(torch_dev):
    """Failure detection: the device count of diverged agents, over the rows
    each mode integrates, before and after a rollout (NaN stays confined)."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    n = 1000 + 37
    sw = I.config1(n=n)
    bad = sw.state.copy()
    bad[0, 3] = np.nan           # position
    bad[15, 700] = np.inf        # rotor
    bad[29, 1036] = -np.inf      # cost (last agent, ragged tail)
    carry = np.zeros((10, n), dtype=np.float32)
    carry[5, 10] = np.nan        # a rounding carry (of v_z): not a state row, not counted ...
    closed = Simulator(sw.types, sw.glob, mode=1)
    st = _dev(torch, dev, bad)
    assert int(closed.count_nonfinite(st).item()) == 3
    closed.step(st, 200, sw.dt, wp=_dev(torch, dev, sw.wp), carry=_dev(torch, dev, carry))
    torch.cuda.synchronize()
    got = st.cpu().numpy()
    # ... but the integrator adds it to the velocity, so agent 10 diverges too
    assert not np.isfinite(got[:30, 10]).all()
    c = closed.count_nonfinite(st)
    closed.count_nonfinite(st, count=c)                 # accumulates
    assert int(c.item()) == 8
    finite = np.ones(n, bool)
    finite[[3, 10, 700, 1036]] = False
    assert np.isfinite(got[:30, finite]).all()          # nothing else is touched
    closed.close()
    open_loop = Simulator(sw.types, sw.glob, mode=0)
    assert int(open_loop.count_nonfinite(_dev(torch, dev, bad)).item()) == 2   # rows 0-16 only
    open_loop.close()


def test_zero_steps_and_single_agent(oracle, torch_dev):
    sw = I.config1(n=1)
    zero = gpu_rollout(torch_dev, sw, 0)
    assert np.array_equal(zero[:30], sw.state.astype(np.float64)) and not zero[30:].any()
    got = gpu_rollout(torch_dev, sw, 500)
    assert_parity(got, oracle_rollout(oracle, sw, 500), sw)


def test_step_rejects_invalid_arguments(torch_dev):
    torch, dev = torch_dev
    from paper_2308_12698_amd import _lib as L
    from paper_2308_12698_amd.sim import Simulator
    import ctypes as C
    sw = I.config1(n=64)
    sim = Simulator(sw.types, sw.glob, mode=1)
    st = _dev(torch, dev, sw.state)
    wp = _dev(torch, dev, sw.wp)
    before = st.clone()
    lib = L.load()
    S = L.State(C.c_void_p(st.data_ptr()), 64)
    P = L.Params(None, None, None, 0)
    Cm = L.Cmds(None, C.c_void_p(wp.data_ptr()), 1, 0, 64, 0)
    h = sim._h
    assert lib.potato_step(h, C.byref(S), C.byref(P), C.byref(Cm), 1e-3, 65, 10, None, 0, None) == L.EINVAL
    assert lib.potato_step(h, C.byref(S), C.byref(P), C.byref(Cm), 0.0, 64, 10, None, 0, None) == L.EINVAL
    assert lib.potato_step(h, C.byref(S), C.byref(P), C.byref(Cm), float("nan"), 64, 10, None, 0, None) == L.EINVAL
    assert lib.potato_step(h, C.byref(S), C.byref(P), C.byref(Cm), 1e-3, 64, -1, None, 0, None) == L.EINVAL
    assert lib.potato_step(h, C.byref(S), C.byref(P), C.byref(Cm), 1e-3, 64, 10, C.c_void_p(st.data_ptr()), 0, None) == L.EINVAL
    Cm0 = L.Cmds(None, None, 0, 0, 64, 0)
    assert lib.potato_step(h, C.byref(S), C.byref(P), C.byref(Cm0), 1e-3, 64, 10, None, 0, None) == L.EINVAL
    # checkpoints without a carry buffer; a carry buffer narrower than the swarm
    ck = torch.empty((1, 40, 64), device=dev)
    assert lib.potato_step(h, C.byref(S), C.byref(P), C.byref(Cm), 1e-3, 64, 10, C.c_void_p(ck.data_ptr()),
                           10, None) == L.EINVAL
    assert b"carr" in lib.potato_last_error(None)
    carry = torch.zeros((10, 64), device=dev)
    Sc = L.State(C.c_void_p(st.data_ptr()), 64, C.c_void_p(carry.data_ptr()), 63)
    assert lib.potato_step(h, C.byref(Sc), C.byref(P), C.byref(Cm), 1e-3, 64, 10, None, 0, None) == L.EINVAL
    # more than 2^30 agents: rejected before any device access (byte offsets are 32-bit)
    big = (1 << 30) + 1
    Sb = L.State(C.c_void_p(st.data_ptr()), big)
    Cb = L.Cmds(None, C.c_void_p(wp.data_ptr()), 1, 0, big, 0)
    assert lib.potato_step(h, C.byref(Sb), C.byref(P), C.byref(Cb), 1e-3, big, 10, None, 0, None) == L.EINVAL
    assert b"2^30" in lib.potato_last_error(None)
    torch.cuda.synchronize()
    assert torch.equal(st, before)
    with pytest.raises(ValueError):
        bad_t = torch.full((64,), 3, dtype=torch.uint8, device=dev)
        sim.debug = True
        sim.step(st, 10, sw.dt, wp=wp, type_idx=bad_t)
    sim.close()


def test_checkpoints_are_the_intermediate_states(torch_dev):
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config4(n=1000, n_steps=230)
    K = 50
    sim = Simulator(sw.types, sw.glob, mode=1, steps_per_launch=37)
    st = _dev(torch, dev, sw.state)
    ck = torch.full((5, 40, 1000), float("nan"), device=dev)
    sim.step(st, 230, sw.dt, wp=_dev(torch, dev, sw.wp), gains=_dev(torch, dev, sw.gains),
             ckpt=ck, ckpt_every=K, carry=carry_zeros(torch_dev, 1000))
    torch.cuda.synchronize()
    ck = ck.cpu().numpy()
    sim.close()
    for c in range(5):
        ref = gpu_rollout(torch_dev, sw, c * K, steps_per_launch=37)
        assert np.array_equal(ck[c].astype(np.float64), ref), c


def test_autotune_cache_round_trip(torch_dev, tmp_path):
    """A cached launch shape is returned without timing and runs the same
    rollout bit for bit."""
    import time
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config1(n=4096)
    sim = Simulator(sw.types, sw.glob, mode=1, form="fused")
    st = _dev(torch, dev, sw.state)
    wp = _dev(torch, dev, sw.wp)
    path = str(tmp_path / "tune.json")
    first = sim.autotune(st, sw.dt, 100, wp=wp, cache=path)
    t0 = time.perf_counter()
    again = sim.autotune(st, sw.dt, 100, wp=wp, cache=path)
    assert again == first and time.perf_counter() - t0 < 0.5
    out = []
    for shape in (first, again):
        sim.set_options(form="fused", **shape)
        x = _dev(torch, dev, sw.state)
        sim.step(x, 300, sw.dt, wp=wp)
        out.append(x.cpu().numpy())
    sim.close()
    assert np.array_equal(out[0], out[1])


LANE_KINDS = ("closed", "open", "uncompensated", "types", "order", "gains", "dead", "plain", "snapshot", "ckpt")


@pytest.mark.parametrize("n", [1, 15, 16, 17, 65, 1000, 16384])
@pytest.mark.parametrize("kind", LANE_KINDS)
def test_four_lanes_per_agent_give_the_bits_of_one(torch_dev, n, kind):
    """Swarms of up to 16,384 quadrotors run four lanes per agent.  The same
    agents inside a swarm of 16,600 run one lane per agent; states, carries,
    snapshots and checkpoints must agree bit for bit: saturated and
    inverted attitudes, clamped integrals, epoch changes, budgets that end
    inside the call, out-of-range types, dead agents, NaN and infinite
    states, a row stride beyond the agent count."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Pipe, Simulator
    N, steps, every = 16600, 37, 10
    rng = np.random.default_rng(77)
    s = np.zeros((30, N))
    s[0:3] = rng.uniform(0.0, 50.0, (3, N))
    s[3:6] = rng.normal(0.0, 2.0, (3, N))
    s[6:10] = rng.normal(0.0, 1.0, (4, N)) + np.array([[2.0], [0.0], [0.0], [0.0]])
    s[6:10] /= np.linalg.norm(s[6:10], axis=0)
    s[10:13] = rng.normal(0.0, 2.0, (3, N))
    s[13:17] = rng.normal(0.0, 80.0, (4, N))
    s[17:20] = rng.uniform(-5.0, 5.0, (3, N))
    s[20:26] = rng.uniform(-1.0, 1.0, (6, N))
    s[26:29] = s[10:13] + rng.normal(0.0, 0.1, (3, N))
    s[29] = rng.uniform(0.0, 1e6, N)
    bad = np.arange(3, N, 97)
    for k, i in enumerate(bad):
        s[k % 30, i] = (np.nan, np.inf, -np.inf)[k % 3]
    state = I.f32(s)
    carry = I.f32(rng.normal(0.0, 1e-7, (10, N)))
    wp = I.f32(rng.uniform(0.0, 50.0, (3, 3, N)))
    cmd = I.f32(rng.uniform(-200.0, 200.0, (4, N)))
    gains = I.f32(np.asarray(I.DEFAULT_GAINS)[:, None] * rng.uniform(0.5, 3.0, (9, N)))
    types = [I.base_type()]
    ti = None
    if kind in ("types", "order", "ckpt"):
        types = I.hetero_types()
        for t, ty in enumerate(types):
            ty["budget"] = 10 + 6 * t
        ti = rng.integers(0, 10, N).astype(np.uint8)
    alive = (rng.random(N) > 0.3).astype(np.uint8)
    mode = 0 if kind == "open" else 1

    def run(m):
        """The first m agents of the swarm (a row stride of m + 5)."""
        ld = m + 5

        def up(a):
            b = np.full(a.shape[:-1] + (ld,), 7.0, dtype=a.dtype)
            b[..., :m] = a[..., :m]
            return _dev(torch, dev, b)

        st, ct = up(state), None if kind == "uncompensated" else up(carry)
        tt = None if ti is None else _dev(torch, dev, ti[:m])
        sim = Simulator(types, I.globals_f32(), mode=mode, form="plain" if kind == "plain" else "fused",
                        steps_per_launch=16)
        out = {}
        if kind == "snapshot":
            pipe = Pipe(sim, m)
            snaps = torch.empty((3, 3, m), pin_memory=True)
            pipe.push(wp[0, :, :m])
            pipe.run(st, steps, 1e-3, snap_every=12, snaps=snaps, carry=ct, alive=_dev(torch, dev, alive[:m]))
            pipe.wait_snapshots(3)
            out["snaps"] = snaps.numpy().copy()
        else:
            ck = torch.full((4, 40, ld), 7.0, device=dev) if kind == "ckpt" else None
            sim.step(st, steps, 1e-3, n_agents=m, type_idx=tt, carry=ct,
                     perm=sim.order_by_type(tt) if kind in ("order", "ckpt") else None,
                     gains=up(gains) if kind in ("gains", "ckpt") else None,
                     motor_cmd=up(cmd) if mode == 0 else None, wp=up(wp) if mode == 1 else None,
                     resample_every=15, step0=4, ckpt=ck, ckpt_every=every if kind == "ckpt" else 0,
                     alive=_dev(torch, dev, alive[:m]) if kind == "dead" else None)
            torch.cuda.synchronize()
            if ck is not None:
                out["ckpt"] = ck.cpu().numpy()
        out["state"] = st.cpu().numpy()
        if ct is not None:
            out["carry"] = ct.cpu().numpy()
        sim.close()
        for a in out.values():
            if a.shape[-1] == ld:
                assert (a[..., m:] == 7.0).all()              # columns past the agents
        return {k: a[..., :n] for k, a in out.items()}

    one, four = run(N), run(n)
    for k in one:
        a, b = one[k], four[k]
        same = (a.view(np.int32) == b.view(np.int32)) | (np.isnan(a) & np.isnan(b))
        assert same.all(), (k, np.argwhere(~same)[:5])


@pytest.mark.parametrize("kind", ["closed", "uncompensated", "gains", "kinds", "kinds_order"])
def test_rollouts_of_many_agents_keep_their_bits(torch_dev, kind):
    """Closed-loop swarms of more than 131,072 agents take the spaced rsq and
    sqrt: the first 131,072 agents of one more must come out bit for bit as
    in a swarm of their own (far way-points, thrust at its bounds, NaN and
    infinite states, zero and unnormalised attitudes)."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    n = 131072
    rng = np.random.default_rng(78)
    N = n + 1
    s = np.zeros((30, N))
    s[0:3] = rng.uniform(0.0, 50.0, (3, N))
    s[3:6] = rng.normal(0.0, 2.0, (3, N))
    s[6:10] = rng.normal(0.0, 1.0, (4, N)) + np.array([[2.0], [0.0], [0.0], [0.0]])
    s[6:10, ::2] /= np.linalg.norm(s[6:10, ::2], axis=0)
    s[6:10, 5::1000] = 0.0
    s[10:13] = rng.normal(0.0, 2.0, (3, N))
    s[13:17] = rng.normal(0.0, 80.0, (4, N))
    s[17:29] = rng.uniform(-1.0, 1.0, (12, N))
    bad = np.arange(3, N, 997)
    for k, i in enumerate(bad):
        s[k % 30, i] = (np.nan, np.inf, -np.inf)[k % 3]
    state = I.f32(s)
    wp = I.f32(rng.uniform(-50.0, 100.0, (2, 3, N)))
    wp[:, :, ::4] = state[0:3, ::4]
    carry = None if kind == "uncompensated" else I.f32(rng.normal(0.0, 1e-7, (10, N)))
    gains = I.f32(np.asarray(I.DEFAULT_GAINS)[:, None] * rng.uniform(0.5, 3.0, (9, N)))
    types, ti = [I.base_type()], None
    if kind.startswith("kinds"):
        types = [I.base_type(), I.car_type(lam=1.0), I.wing_type(lam=-1.0), I.base_type(), I.car_type(lam=-1.0)]
        ti = rng.integers(0, 5, N).astype(np.uint8)
    out = []
    for m in (n, N):
        sim = Simulator(types, I.globals_f32(), mode=1, form="fused")
        st = _dev(torch, dev, state[:, :m])
        ct = None if carry is None else _dev(torch, dev, carry[:, :m])
        tt = None if ti is None else _dev(torch, dev, ti[:m])
        sim.step(st, 23, 1e-3, type_idx=tt, carry=ct, perm=sim.order_by_type(tt) if kind == "kinds_order" else None,
                 gains=_dev(torch, dev, gains[:, :m]) if kind == "gains" else None,
                 wp=_dev(torch, dev, wp[:, :, :m]), resample_every=11)
        torch.cuda.synchronize()
        out.append([st.cpu().numpy()[:, :n]] + ([] if ct is None else [ct.cpu().numpy()[:, :n]]))
        sim.close()
    for a, b in zip(*out):
        same = (a.view(np.int32) == b.view(np.int32)) | (np.isnan(a) & np.isnan(b))
        assert same.all(), np.argwhere(~same)[:5]


@pytest.mark.parametrize("n", [1, 257, 10000, 16384])
@pytest.mark.parametrize("mode", [0, 1])
def test_single_step_launches_of_small_swarms(torch_dev, n, mode):
    """Launches of one step take one agent per lane, longer ones four lanes:
    17 steps in launches of 17, 16 and 1, and of 1 (twice, the second time in
    the plain form) must agree bit for bit."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    rng = np.random.default_rng(n + mode)
    state = I.hover_state(rng.uniform(0.0, 50.0, (3, n)))
    wp = _dev(torch, dev, I.f32(rng.uniform(0.0, 50.0, (2, 3, n))))
    cmd = _dev(torch, dev, I.f32(rng.uniform(-200.0, 200.0, (4, n))))
    out = []
    for form, per_launch in (("fused", 17), ("fused", 16), ("fused", 1), ("plain", 1)):
        sim = Simulator([I.base_type()], I.globals_f32(), mode=mode, form=form, steps_per_launch=per_launch)
        st, ct = _dev(torch, dev, state), torch.zeros((10, n), device=dev)
        sim.step(st, 17, 1e-3, carry=ct, motor_cmd=cmd if mode == 0 else None, wp=wp if mode == 1 else None,
                 resample_every=9)
        torch.cuda.synchronize()
        out.append(torch.cat([st, ct]).cpu().numpy())
        sim.close()
    assert np.isfinite(out[0]).all()
    for other in out[1:]:
        assert np.array_equal(out[0], other)


@pytest.mark.parametrize("dead", ["none", "scattered", "three quarters in front", "all but the last"])
@pytest.mark.parametrize("carry", [True, False])
def test_masked_swarms_of_many_agents(torch_dev, dead, carry):
    """131,203 quadrotors of one type with an alive mask, agents dead here and
    there and in one piece: the live ones have the bits that they have
    without a mask, the dead ones those that they came with."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    n, steps = 131203, 23
    rng = np.random.default_rng(79)
    state = I.hover_state(rng.uniform(0.0, 50.0, (3, n)))
    state[10:13] = I.f32(rng.normal(0.0, 0.5, (3, n)))
    wp = _dev(torch, dev, I.f32(rng.uniform(0.0, 50.0, (1, 3, n))))
    alive = {"none": np.ones(n), "scattered": rng.random(n) > 0.4, "three quarters in front": np.arange(n) >= 3 * n // 4,
             "all but the last": np.arange(n) == n - 1}[dead].astype(np.uint8)
    sim = Simulator([I.base_type()], I.globals_f32(), mode=1)
    out = []
    for mask in (None, alive):
        st, ct = _dev(torch, dev, state), torch.zeros((10, n), device=dev) if carry else None
        sim.step(st, steps, 1e-3, wp=wp, carry=ct, alive=_dev(torch, dev, mask))
        torch.cuda.synchronize()
        out.append(st.cpu().numpy())
    sim.close()
    live = alive == 1
    assert np.array_equal(out[0][:, live], out[1][:, live])
    assert np.array_equal(out[1][:, ~live], state[:, ~live])


def budget_swarm(n, budgets, seed, steps):
    """Quadrotors of len(budgets) airframes with these step budgets, labels
    shuffled with uneven shares, waypoints redrawn halfway; more than 16,384
    of them, so that a launch takes one lane per agent."""
    assert n > 16384
    types = [dict(t, budget=b) for t, b in zip(I.hetero_types(len(budgets), seed_stream=5), budgets)]
    rng = np.random.default_rng(seed)
    share = rng.uniform(0.2, 1.0, len(budgets))
    labels = rng.choice(len(budgets), n, p=share / share.sum()).astype(np.uint8)
    pos = rng.uniform(0.0, 30.0, (3, n))
    return I.Swarm("budgets", 1, 1e-3, steps, I.hover_state(pos), types, I.globals_f32(), type_idx=labels,
                   wp=I.f32(pos + rng.uniform(-3.0, 3.0, (2, 3, n))), resample_every=steps // 2)


def run_budgets(torch_dev, sw, ordered, *, alive=None, gains=None, carry=True, **opts):
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sim = Simulator(sw.types, sw.glob, mode=1, debug=True, **opts)
    st, ti = _dev(torch, dev, sw.state), _dev(torch, dev, sw.type_idx)
    sim.step(st, sw.n_steps, sw.dt, type_idx=ti, perm=sim.order_by_type(ti) if ordered else None,
             wp=_dev(torch, dev, sw.wp), resample_every=sw.resample_every, gains=_dev(torch, dev, gains),
             carry=carry_zeros(torch_dev, sw.n) if carry else None, alive=_dev(torch, dev, alive))
    torch.cuda.synchronize()
    out = st.cpu().numpy()
    sim.close()
    return out


EIGHT = (200, 180, 150, 120, 90, 60, 30, 1)


@pytest.mark.parametrize("opts", [dict(), dict(block=512, grid_blocks=1), dict(block=1024, grid_blocks=2),
                                  dict(block=64, steps_per_launch=200, grid_blocks=3), dict(block=256, grid_blocks=7),
                                  dict(block=128, steps_per_launch=25, use_graph=True), dict(form="plain")])
def test_grouped_one_lane_launches_equal_the_type_order(torch_dev, opts):
    """Eight budget classes of 16,601 agents in the caller's order, grouped
    per block (k_rollout with group_agents), against the type order: one
    round of blocks, one to seven blocks of several chunks each, all block
    widths, a captured graph, one step per launch; then with dead agents,
    per-agent gains and no carries."""
    sw = budget_swarm(16601, EIGHT, 1, 200)
    opts = dict(dict(form="fused", steps_per_launch=50), **opts)
    assert np.array_equal(run_budgets(torch_dev, sw, False, **opts), run_budgets(torch_dev, sw, True, steps_per_launch=50))
    rng = np.random.default_rng(2)
    gains = I.f32(np.asarray(I.DEFAULT_GAINS)[:, None] * rng.uniform(0.8, 1.2, (9, sw.n)))
    alive = (rng.random(sw.n) > 0.2).astype(np.uint8)
    for kw in (dict(alive=alive), dict(gains=gains), dict(alive=alive, gains=gains, carry=False)):
        got = run_budgets(torch_dev, sw, False, **kw, **opts)
        assert np.array_equal(got, run_budgets(torch_dev, sw, True, **kw))
        if "alive" in kw:
            assert np.array_equal(got[:, alive == 0], sw.state[:, alive == 0])


@pytest.mark.parametrize("budgets", [EIGHT, (200, 120, 60), (200, 200), tuple(range(12, 156, 12))])
def test_one_lane_launches_of_several_budgets_match_oracle(oracle, torch_dev, budgets):
    """Eight and three budget classes (grouped per block), one class and
    twelve (not grouped: the plain groups of 64 of k_rollout), 20,011 agents
    in the caller's order: bitwise the type order, and 2,000 sampled agents
    within the tolerance of the reference."""
    sw = budget_swarm(20011, budgets, len(budgets), 200)
    got = run_budgets(torch_dev, sw, False)
    assert np.array_equal(got, run_budgets(torch_dev, sw, True, steps_per_launch=30))
    pick = np.sort(np.random.default_rng(3).choice(sw.n, 2000, replace=False))
    sub = I.subset(sw, pick)
    assert_parity(got[:, pick].astype(np.float64), oracle_rollout(oracle, sub, 200), sub)
