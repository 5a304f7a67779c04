"""Cars and fixed-wing aircraft in the quadrotors' type-indexed launch (the
three robot kinds of Sec. II-B; aircraft circling as in the first
demonstration of Sec. IV), through the C ABI, against the FP64 references
(quadrotors through the quadrotor reference, cars and aircraft through the
vehicle reference, each on its own agents).

Tolerance: relative state error <= 1e-4 per agent and state group (the
quadrotor groups of tests/_util.py for quadrotors; position, speed,
heading, actuator angle and flight-path angle for the others).  Plain and
fused launches, ordered and unordered launches, and a kind's agents run
alone are compared bitwise: a lane's arithmetic does not depend on the
launch or on its neighbours' kinds.
"""
import numpy as np
import pytest

from paper_2308_12698_amd import inputs as I
from tests._util import OPEN_LOOP_GROUPS, rel_errors, vehicle_rel_errors

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


def agent_kinds(sw):
    kinds = np.array([int(t.get("kind", 0)) for t in sw.types])
    ti = np.zeros(sw.n, dtype=np.int64) if sw.type_idx is None else sw.type_idx.astype(np.int64)
    return kinds[ti]


def gpu_run(torch_dev, sw, n_steps, *, form="fused", steps_per_launch=0, ordered=False, carry=True,
            alive=None, state=None):
    """The workload on the GPU: float64 [30, N] after n_steps."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sim = Simulator(sw.types, sw.glob, mode=sw.mode, form=form, steps_per_launch=steps_per_launch,
                    debug=True)
    st = _dev(torch, dev, sw.state if state is None else state)
    ti = _dev(torch, dev, sw.type_idx)
    perm = sim.order_by_type(ti) if ordered else None
    ct = torch.zeros((10, sw.n), dtype=torch.float32, device=dev) if carry else None
    sim.step(st, n_steps, sw.dt, type_idx=ti, perm=perm, motor_cmd=_dev(torch, dev, sw.motor_cmd),
             wp=_dev(torch, dev, sw.wp), resample_every=sw.resample_every, carry=ct,
             alive=_dev(torch, dev, alive))
    torch.cuda.synchronize()
    got = st.cpu().numpy().astype(np.float64)
    sim.close()
    return got


def oracle_run(oracle, sw, n_steps, agents=None):
    sub = sw if agents is None else I.subset(sw, agents)
    return oracle.rollout_kinds(sub.state, sub.types, sub.glob, sub.mode, sub.dt, n_steps,
                                type_idx=sub.type_idx, gains=sub.gains, motor_cmd=sub.motor_cmd, wp=sub.wp,
                                resample_every=sub.resample_every)


def assert_kinds_parity(got, ref, sw, agents=None, tol=TOL):
    """got, ref: [30, len(agents)] of the agents `agents` (default all)."""
    kinds = agent_kinds(sw)
    if agents is not None:
        kinds = kinds[agents]
    ti = (np.zeros(sw.n, dtype=np.int64) if sw.type_idx is None else sw.type_idx.astype(np.int64))
    if agents is not None:
        ti = ti[agents]
    quad = kinds == 0
    worst = {}
    if quad.any():
        qtypes = [k for k, t in enumerate(sw.types) if int(t.get("kind", 0)) == 0]
        remap = np.full(len(sw.types), -1)
        remap[qtypes] = np.arange(len(qtypes))
        groups = OPEN_LOOP_GROUPS if sw.mode == 0 else None
        errs = rel_errors(got[:30, quad], ref[:30, quad], [sw.types[k] for k in qtypes], remap[ti[quad]], groups)
        worst.update({f"quad {g}": v for g, v in errs.items()})
    for kind, name in ((1, "car"), (2, "wing")):
        sel = kinds == kind
        if sel.any():
            errs = vehicle_rel_errors(got[:7, sel], ref[:7, sel])
            worst.update({f"{name} {g}": v for g, v in errs.items()})
    print("worst relative errors:", {k: f"{v[0]:.2e}" for k, v in worst.items()}, flush=True)
    bad = {k: v for k, v in worst.items() if not v[0] <= tol}
    assert not bad, bad


def open_loop_kinds(n=6000, seed=11):
    """Open-loop quadrotors (rotor commands within 10 % of hover), cars
    (constant acceleration and steering commands) and aircraft (constant
    airspeed, bank and flight-path commands), labels shuffled."""
    r = np.random.default_rng(seed)
    types = [I.base_type(), I.car_type(), I.wing_type()]
    labels = r.integers(0, 3, n).astype(np.uint8)
    s = np.zeros((30, n))
    s[0:3] = np.stack([r.uniform(0, 100, n), r.uniform(0, 100, n), r.uniform(0, 20, n)])
    s[6] = 1.0
    cmd = np.zeros((4, n))
    w_ref = float(types[0]["w_ref"])
    cmd[:, labels == 0] = r.uniform(-0.1, 0.1, (4, int((labels == 0).sum()))) * w_ref
    for kind in (1, 2):
        idx = np.where(labels == kind)[0]
        centre = np.stack([r.uniform(0, 100, idx.size), r.uniform(0, 100, idx.size),
                           np.zeros(idx.size) if kind == 1 else r.uniform(40, 60, idx.size)])
        s[:, idx] = 0.0
        s[0:7, idx] = I.orbit_starts(r, types[kind], centre)
        if kind == 1:
            cmd[0, idx] = r.uniform(-1.0, 1.0, idx.size)
            cmd[1, idx] = r.uniform(-0.4, 0.4, idx.size)
        else:
            cmd[0, idx] = r.uniform(15.0, 21.0, idx.size)
            cmd[1, idx] = r.uniform(-0.5, 0.5, idx.size)
            cmd[2, idx] = r.uniform(-0.1, 0.1, idx.size)
    return I.Swarm("kinds_open", 0, 1e-3, 2000, I.f32(s), types, I.globals_f32(), type_idx=labels,
                   motor_cmd=I.f32(cmd))


def test_mixed_kinds_closed_loop_matches_oracle(oracle, torch_dev):
    """Quadrotors, cars and aircraft shuffled in one launch, 1,000 steps, in
    index order and in the type order; vehicles leave rows 7-29 (and a car
    rows 2 and 6) exactly as they were."""
    sw = I.config_kinds(n=6000, n_steps=1000)
    ref = oracle_run(oracle, sw, 1000)
    kinds = agent_kinds(sw)
    outs = []
    for ordered in (False, True):
        got = gpu_run(torch_dev, sw, 1000, steps_per_launch=250, ordered=ordered)
        assert_kinds_parity(got, ref, sw)
        veh = kinds != 0
        assert np.array_equal(got[7:, veh], sw.state[7:, veh].astype(np.float64))
        car = kinds == 1
        assert np.array_equal(got[[2, 6]][:, car], sw.state[[2, 6]][:, car].astype(np.float64))
        outs.append(got)
    assert np.array_equal(outs[0], outs[1])


def test_mixed_kinds_open_loop_matches_oracle(oracle, torch_dev):
    sw = open_loop_kinds()
    ref = oracle_run(oracle, sw, sw.n_steps)
    got = gpu_run(torch_dev, sw, sw.n_steps, steps_per_launch=500)
    assert_kinds_parity(got, ref, sw)


def test_vehicles_settle_on_their_orbits(torch_dev):
    """Closed loop, 20,000 steps (20 s) from starts up to half a radius off
    the orbit and 60 degrees off its direction: every car ends within 1 cm
    of its orbit's radius around its waypoint, every aircraft within 0.5 m
    of its orbit and 1 cm of its altitude (the circles of the paper's
    demonstration; the FP64 reference ends within 0.06 mm and 0.18 m)."""
    sw = I.config_kinds(n=4000, n_steps=20000)
    got = gpu_run(torch_dev, sw, 20000, steps_per_launch=1000)
    kinds = agent_kinds(sw)
    for kind, tol in ((1, 0.01), (2, 0.5)):
        sel = kinds == kind
        t = sw.types[1] if kind == 1 else sw.types[3]
        rho = I.veh_param(t, "rho")
        c = sw.wp[-1][:, sel].astype(np.float64)
        d = np.hypot(got[0, sel] - c[0], got[1, sel] - c[1])
        assert np.abs(d - rho).max() < tol, (kind, np.abs(d - rho).max())
        if kind == 2:
            assert np.abs(got[2, sel] - c[2]).max() < 0.01


def test_plain_equals_fused_bitwise(torch_dev):
    sw = I.config_kinds(n=3000, n_steps=200)
    a = gpu_run(torch_dev, sw, 200, form="plain")
    b = gpu_run(torch_dev, sw, 200, steps_per_launch=37)
    assert np.array_equal(a, b)
    ol = open_loop_kinds(n=2000, seed=3)
    a = gpu_run(torch_dev, ol, 150, form="plain", carry=False)
    b = gpu_run(torch_dev, ol, 150, steps_per_launch=150, carry=False)
    assert np.array_equal(a, b)


def test_each_kind_equals_its_own_launch(torch_dev):
    """A kind's agents advanced in a mixed launch equal the same agents
    advanced alone (a type table and launch of their kind only), bitwise."""
    sw = I.config_kinds(n=4000, n_steps=300)
    mixed = gpu_run(torch_dev, sw, 300, steps_per_launch=100)
    kinds = agent_kinds(sw)
    for group in ((0,), (1,), (2,)):
        idx = np.where(np.isin(kinds, group))[0]
        sub = I.subset(sw, idx)
        keep = sorted({int(t) for t in sub.type_idx})
        remap = np.zeros(len(sw.types), dtype=np.uint8)
        remap[keep] = np.arange(len(keep))
        alone = I.Swarm(sub.name, sub.mode, sub.dt, sub.n_steps, sub.state, [sw.types[k] for k in keep], sub.glob,
                        type_idx=remap[sub.type_idx], wp=sub.wp, resample_every=sub.resample_every)
        got = gpu_run(torch_dev, alone, 300, steps_per_launch=100)
        assert np.array_equal(got, mixed[:, idx]), group


def test_kinds_full_size(oracle, torch_dev):
    """1,048,576 agents (half quadrotors, a quarter cars, a quarter
    aircraft) in the type order: every agent against the references after
    1,000 steps, then 2,048 sampled agents after 10,000 steps (waypoints
    redrawn every 2,000 steps for the quadrotors); the launch in index
    order equals the type-ordered one bitwise."""
    torch, dev = torch_dev
    sw = I.config_kinds()
    print("kinds full size: 1,048,576 agents, 1,000 steps then 10,000", flush=True)
    got = gpu_run(torch_dev, sw, 1000, steps_per_launch=1000, ordered=True)
    assert np.isfinite(got).all()
    ref = oracle_run(oracle, sw, 1000)
    assert_kinds_parity(got, ref, sw)
    del ref
    # the kinds shuffled in index order: each block groups its agents by kind
    assert np.array_equal(gpu_run(torch_dev, sw, 1000, steps_per_launch=1000), got)
    got = gpu_run(torch_dev, sw, 10000, steps_per_launch=1000, ordered=True)
    sample = np.sort(np.random.default_rng(21).choice(sw.n, 2048, replace=False))
    ref = oracle_run(oracle, sw, 10000, agents=sample)
    assert_kinds_parity(got[:, sample], ref, sw, agents=sample)


def test_vehicle_budgets_and_dead_agents(oracle, torch_dev):
    """Per-type step budgets (cars 300, counter-clockwise aircraft 700) and
    dead agents: each live agent takes min(steps, budget) steps, dead ones
    none."""
    sw = I.config_kinds(n=3000, n_steps=1000)
    types = [dict(t) for t in sw.types]
    types[1]["budget"] = 300
    types[2]["budget"] = 300
    types[3]["budget"] = 700
    sw = I.Swarm(sw.name, sw.mode, sw.dt, sw.n_steps, sw.state, types, sw.glob, type_idx=sw.type_idx, wp=sw.wp,
                 resample_every=sw.resample_every)
    alive = (np.arange(sw.n) % 5 != 0).astype(np.uint8)
    got = gpu_run(torch_dev, sw, 1000, steps_per_launch=400, alive=alive)
    live = np.where(alive == 1)[0]
    ref = oracle_run(oracle, sw, 1000, agents=live)
    assert_kinds_parity(got[:, live], ref, sw, agents=live)
    dead = alive == 0
    assert np.array_equal(got[:, dead], sw.state[:, dead].astype(np.float64))


def test_kinds_reject_checkpoints_and_the_adjoint(torch_dev):
    torch, dev = torch_dev
    from paper_2308_12698_amd import _lib as L
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config_kinds(n=256, n_steps=100)
    sim = Simulator(sw.types, sw.glob, mode=1)
    st = _dev(torch, dev, sw.state)
    ti = _dev(torch, dev, sw.type_idx)
    wp = _dev(torch, dev, sw.wp)
    ck = torch.empty((2, 40, sw.n), device=dev)
    with pytest.raises(L.PotatoError) as e:
        sim.step(st, 100, sw.dt, type_idx=ti, wp=wp, ckpt=ck, ckpt_every=50,
                 carry=torch.zeros((10, sw.n), device=dev))
    assert e.value.status == L.EUNSUPPORTED
    with pytest.raises(L.PotatoError) as e:
        sim.step_backward(ck, 50, 100, sw.dt, torch.zeros((30, sw.n), device=dev), type_idx=ti, wp=wp)
    assert e.value.status == L.EUNSUPPORTED
    sim.close()


def test_collision_radius_of_vehicle_types(oracle, torch_dev):
    """Vehicle types carry their own collision radius through the type index."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config_kinds(n=20000, n_steps=10)
    r = np.random.default_rng(4)
    state = sw.state.copy()
    state[0:3] = I.f32(np.stack([r.uniform(0, 40, sw.n), r.uniform(0, 40, sw.n), r.uniform(0, 4, sw.n)]))
    sim = Simulator(sw.types, sw.glob, mode=1)
    st = _dev(torch, dev, state)
    alive = torch.ones(sw.n, dtype=torch.uint8, device=dev)
    died = torch.zeros(1, dtype=torch.int64, device=dev)
    sim.detect_collisions(st, alive, type_idx=_dev(torch, dev, sw.type_idx), died=died)
    torch.cuda.synchronize()
    got = alive.cpu().numpy()
    sim.close()
    ref, ref_died = oracle.detect_collisions(state, [t["radius"] for t in sw.types], np.ones(sw.n, np.uint8),
                                             type_idx=sw.type_idx)
    assert np.array_equal(got, ref) and int(died.item()) == ref_died > 0


@pytest.mark.parametrize("dt,steps,turns", [(1e-3, 50, 0.0), (0.05, 40, 0.0), (0.1, 40, 0.0), (0.25, 20, 0.0),
                                            (1e-3, 1, 1e5), (1e-3, 1, 1e6)])
def test_vehicle_angle_ranges(oracle, torch_dev, dt, steps, turns):
    """The ranges of the vehicles' trigonometry: stage offsets within the
    short series (dt = 1 ms), the longer ones and beyond (dt up to 0.25 s,
    steering far from its command), headings up to and past the reduction's
    range (one step, so that the heading's own rounding does not enter),
    orbit directions other than +-1, agents at the very centre of their
    orbit and on its axes."""
    r = np.random.default_rng(int(steps + 1000 * dt))
    types = [I.car_type(lam=1.0), I.car_type(lam=-1.0), I.car_type(lam=0.5), I.wing_type(lam=1.0),
             I.wing_type(lam=-1.0), I.wing_type(lam=-0.75)]
    n = 1200
    labels = r.integers(0, len(types), n).astype(np.uint8)
    s = np.zeros((30, n))
    wp = np.zeros((1, 3, n))
    for t, ty in enumerate(types):
        idx = np.where(labels == t)[0]
        centre = np.stack([r.uniform(0, 100, idx.size), r.uniform(0, 100, idx.size),
                           np.zeros(idx.size) if ty["kind"] == 1 else r.uniform(40, 60, idx.size)])
        s[0:7, idx] = I.orbit_starts(r, ty, centre)
        s[5, idx] = r.uniform(-0.5, 0.5, idx.size)
        wp[0][:, idx] = centre
    special = np.arange(0, n, 10)
    s[0:2, special] = np.round(s[0:2, special])
    wp[0, 0:2, special] = s[0:2, special].T                 # at the centre
    wp[0, 0, special[::3]] += 30.0                           # on an axis, behind and ahead
    wp[0, 1, special[1::3]] -= 30.0
    s[4] += r.choice([-1.0, 1.0], n) * r.uniform(0.5, 1.0, n) * turns
    sw = I.Swarm("angles", 1, dt, steps, I.f32(s), types, I.globals_f32(), type_idx=labels, wp=I.f32(wp))
    got = gpu_run(torch_dev, sw, steps)
    assert_kinds_parity(got, oracle_run(oracle, sw, steps), sw)
    assert np.array_equal(got, gpu_run(torch_dev, sw, steps, form="plain"))


def one_kind(kind, state, wp=None, cmd=None, dt=float(np.float32(1e-3)), **params):
    """A swarm of one car or aircraft type: rows 0-6 of its agents and their
    waypoints [3, n] (closed loop) or commands [4, n] (open loop).  The time
    step is the float32 that the call takes, for the reference too."""
    n = state.shape[1]
    s = np.zeros((30, n))
    s[0:7] = state
    ty = I.car_type(**params) if kind == 1 else I.wing_type(**params)
    return I.Swarm("one_kind", 0 if wp is None else 1, dt, 1, I.f32(s), [ty], I.globals_f32(),
                   wp=None if wp is None else I.f32(wp[None]), motor_cmd=None if cmd is None else I.f32(cmd))


@pytest.mark.parametrize("n", [1, 300])
def test_aircraft_nearly_at_rest(oracle, torch_dev, n):
    """Airspeeds down to the smallest subnormal, commanded to stop, wings
    level (the course rate g tan(bank) / V is zero whatever V is, so the
    heading stays what it is) or at banks as small as their speeds (a
    quotient of two subnormals of some rad/s).  Speeds of 1e-39 m/s keep 19
    bits, so 20 steps' roundings of speed and bank are 20 x 2^-20 x the
    0.2 rad turned at most, well inside the tolerance."""
    r = np.random.default_rng(n)
    x = np.zeros((7, n))
    x[0:3] = r.uniform(10.0, 60.0, (3, n))
    x[3] = 10.0 ** r.uniform(-39.0, -36.0, n)
    x[5] = x[3] * r.uniform(-1.0, 1.0, n)
    level = np.arange(n) % 3 == 1
    x[3, level] = 10.0 ** r.uniform(-44.0, 1.0, int(level.sum()))
    x[5, level] = 0.0
    x[4] = r.uniform(-3.0, 3.0, n)
    x[6] = r.uniform(-0.1, 0.1, n)
    sw = one_kind(2, x, cmd=np.zeros((4, n)))
    ref = oracle_run(oracle, sw, 20)
    for form in ("fused", "plain"):
        got = gpu_run(torch_dev, sw, 20, form=form)
        assert np.isfinite(got).all()
        assert np.array_equal(got[4, level], sw.state[4, level].astype(np.float64))
        assert_kinds_parity(got, ref, sw)


@pytest.mark.parametrize("kind", [1, 2])
@pytest.mark.parametrize("far", [0.9e19, 1.2e19])
def test_orbits_beyond_the_reciprocals_range(oracle, torch_dev, kind, far):
    """Agents so far from their orbit that the course error's product of
    complex numbers exceeds 2^126, whose reciprocal is no normal number: they
    still steer towards it."""
    r = np.random.default_rng(int(far / 1e18) + kind)
    n = 500
    rho = 25.0 if kind == 1 else 80.0
    th, off = r.uniform(-np.pi, np.pi, n), r.uniform(-0.25, 0.25, n)
    x = np.zeros((7, n))
    x[0:2] = far * r.uniform(0.97, 1.03, n) * np.stack([np.cos(th), np.sin(th)])
    x[2] = 50.0
    x[3] = 15.0
    x[4] = th + np.pi + off
    wp = np.zeros((3, n))
    wp[2] = 50.0
    sw = one_kind(kind, x, wp=wp, rho=rho, k_orb=rho)
    ref = oracle_run(oracle, sw, 20)
    assert (np.abs(ref[5]) > 1e-3).mean() > 0.5              # they do steer
    assert_kinds_parity(gpu_run(torch_dev, sw, 20), ref, sw)


def test_vehicles_that_are_not_finite_keep_to_themselves(torch_dev):
    """NaN and infinite rows (speed, heading, actuator, flight path, position)
    of cars and aircraft: those agents stay not finite, and every other agent
    of their waves has the bits it has without them."""
    r = np.random.default_rng(6)
    sw = I.config_kinds(n=3000, n_steps=100)
    veh = np.where(agent_kinds(sw) != 0)[0]
    bad = r.choice(veh, 300, replace=False)
    state = sw.state.copy()
    for k, i in enumerate(bad):
        state[(3, 4, 5, 0, 1)[k % 5], i] = (np.nan, np.inf, -np.inf)[k % 3]
    clean = gpu_run(torch_dev, sw, 100)
    got = gpu_run(torch_dev, sw, 100, state=state)
    rest = np.setdiff1d(np.arange(sw.n), bad)
    assert np.array_equal(got[:, rest], clean[:, rest])
    assert (~np.isfinite(got[0:7, bad])).any(axis=0).all()
    assert np.array_equal(got, gpu_run(torch_dev, sw, 100, state=state, form="plain"), equal_nan=True)


def test_course_rate_has_the_tangents_rounding(torch_dev):
    """Aircraft at 16 m/s whose inputs hold their bank and flight path: one
    step turns them by dt g tan(bank) / V, all four stages alike.  The same
    operations in float32 with a correctly rounded tangent in their place
    give the same bits for at least 19 in 20 banks (0.26 ulp in the mean
    where the best possible is 0.25; an emulation of its operations gives 98
    in 100, of the rounded sine over the rounded cosine 61)."""
    r = np.random.default_rng(8)
    n, f, dt = 20000, np.float32, np.float32(1e-3)
    x = np.zeros((7, n))
    x[3] = 16.0
    x[5] = I.f32(r.uniform(-0.7, 0.7, n))
    cmd = np.zeros((4, n))
    cmd[0], cmd[1] = 16.0, x[5]
    sw = one_kind(2, x, cmd=cmd)
    k = f(sw.glob["g"]) * np.tan(x[5]).astype(f) / f(16.0)
    acc = f(3.0) * k
    acc = (acc.astype(np.float64) + 2.0 * k).astype(f) + k
    dt6 = dt / f(6.0)
    lo = f(np.float64(dt) / 6.0 - np.float64(dt6))
    want = (np.float64(dt6) * acc + (np.float64(lo) * acc).astype(f)).astype(f)
    got = gpu_run(torch_dev, sw, 1)[4]
    assert np.abs(got - want).max() <= 4 * 2.0 ** -24 * np.abs(want).max()
    assert (got == want).mean() >= 0.95


@pytest.mark.parametrize("kind", [1, 2])
def test_increments_are_not_rounded_before_the_carry(oracle, torch_dev, kind):
    """500 steps of 1 ms on and around orbits.  Rounding dt/6, as float32
    must, moves an agent by 0.49 x 2^-24 of the way it flies: 0.26 um in the 9
    m of an aircraft, 0.1 um in the 3.6 m of a car.  The mean error of the
    position (with its carry) stays below half of that."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    r = np.random.default_rng(9)
    n, steps = 20000, 500
    ty = I.car_type() if kind == 1 else I.wing_type()
    centre = np.stack([r.uniform(0, 100, n), r.uniform(0, 100, n), np.full(n, 0.0 if kind == 1 else 50.0)])
    x = I.orbit_starts(r, ty, centre)
    if kind == 1:
        x[3] = r.uniform(6.5, 8.0, n)
    sw = one_kind(kind, x, wp=centre)
    sim = Simulator(sw.types, sw.glob, mode=1)
    st, ct = _dev(torch, dev, sw.state), torch.zeros((10, n), device=dev)
    sim.step(st, steps, sw.dt, wp=_dev(torch, dev, sw.wp), carry=ct)
    torch.cuda.synchronize()
    got = st.cpu().numpy()[0:3].astype(np.float64) + ct.cpu().numpy()[0:3]
    sim.close()
    way = steps * sw.dt * float(np.mean(x[3]))
    err = np.linalg.norm(got - oracle_run(oracle, sw, steps)[0:3], axis=0).mean()
    print(f"mean position error {err:.2e} m over {way:.1f} m", flush=True)
    assert err < 0.5 * 0.49 * 2.0 ** -24 * way


@pytest.mark.parametrize("dt", [0.002, 0.02, 0.0599, 0.0601, 0.25])
def test_vehicles_with_large_stage_offsets(oracle, torch_dev, dt):
    """Cars and aircraft small and quick enough (up to 20 rad/s, actuators of
    20 ms) that a stage's angles lie past the series' 0.1 rad, beside ones
    far below it in the same waves, at time steps on both sides of the one
    from which every agent takes its stages' functions directly.  Against the
    reference after 3 steps: at 0.25 s the small cars' guidance, held through
    a step, is unstable (20 steps multiply 1e-7 rad by 1e4 in the reference
    itself, 3 by less than 10); the launches' bits after 20."""
    r = np.random.default_rng(int(1e5 * dt))
    types = [I.car_type(L=0.2, l_r=0.1, tau_delta=max(0.02, dt), v_cruise=2.0, rho=1.0), I.car_type(),
             I.wing_type(tau_V=max(0.1, dt), tau_phi=max(0.02, dt), tau_gamma=max(0.02, dt), V_cruise=4.0, rho=4.0),
             I.wing_type(lam=-1.0)]
    n, steps = 2000, 20
    labels = r.integers(0, 4, n).astype(np.uint8)
    s, wp = np.zeros((30, n)), np.zeros((1, 3, n))
    for t, ty in enumerate(types):
        idx = np.where(labels == t)[0]
        centre = np.stack([r.uniform(0, 100, idx.size), r.uniform(0, 100, idx.size), np.full(idx.size, 30.0 * (t > 1))])
        s[0:7, idx] = I.orbit_starts(r, ty, centre)
        s[5, idx] = r.uniform(-0.5, 0.5, idx.size)
        wp[0][:, idx] = centre
    sw = I.Swarm("offsets", 1, float(np.float32(dt)), steps, I.f32(s), types, I.globals_f32(), type_idx=labels,
                 wp=I.f32(wp))
    assert_kinds_parity(gpu_run(torch_dev, sw, 3), oracle_run(oracle, sw, 3), sw)
    got = gpu_run(torch_dev, sw, steps)
    assert np.array_equal(got, gpu_run(torch_dev, sw, steps, form="plain"))
    assert np.array_equal(got, gpu_run(torch_dev, sw, steps, ordered=True))
