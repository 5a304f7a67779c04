"""The hand-written adjoint (through the C ABI) against the FP64 reference.

Workload: the differentiable rollout -- closed loop, per-agent gains,
500 RK4 steps at dt = 2 ms, checkpoints every 50 steps, loss
sum ||p_T - target||^2 + 1e-4 * J_T.  Tolerance: per agent and per block
(30 initial-state rows; 9 gains) ||g_gpu - g_ref|| / ||g_ref|| <= 1e-3,
against (a) the reference's forward-mode dual-number gradient and (b) FP64
central finite differences (h = 1e-6) in the target-centred frame.
"""
import numpy as np
import pytest

from paper_2308_12698_amd import inputs as I

pytestmark = pytest.mark.gpu

TOL = 1e-3
H = 1e-6


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch, torch.device("cuda:0")


@pytest.fixture(scope="module")
def diff_run(torch_dev):
    """GPU forward with checkpoints + reverse sweep on the full 65,536-agent
    differentiable workload; returns inputs and gradients (numpy)."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config4()
    K = sw.extra["ckpt_every"]
    sim = Simulator(sw.types, sw.glob, mode=1, form="fused", steps_per_launch=100)
    x = torch.from_numpy(sw.state).to(dev)
    gains = torch.from_numpy(sw.gains).to(dev)
    wp = torch.from_numpy(sw.wp).to(dev)
    ckpt = torch.empty((sw.n_steps // K, 40, sw.n), device=dev)
    sim.step(x, sw.n_steps, sw.dt, gains=gains, wp=wp, ckpt=ckpt, ckpt_every=K, carry=torch.zeros_like(x[:10]))
    tgt = torch.from_numpy(sw.extra["target"]).to(dev)
    gfin = torch.zeros((30, sw.n), device=dev)
    gfin[0:3] = 2.0 * (x[0:3] - tgt)
    gfin[29] = sw.extra["cost_weight"]
    gx0, gg = sim.step_backward(ckpt, K, sw.n_steps, sw.dt, gfin, gains=gains, wp=wp)
    torch.cuda.synchronize()
    out = dict(sw=sw, sim=sim, final=x.cpu().numpy(), gx0=gx0.cpu().numpy(), gg=gg.cpu().numpy(),
               ckpt=ckpt, gains_t=gains, wp_t=wp, gfin=gfin)
    yield out
    sim.close()


def block_errors(got, ref):
    """got, ref: [n, 39] -> per-agent relative errors of (state, gains) blocks."""
    es = np.linalg.norm(got[:, :30] - ref[:, :30], axis=1) / np.linalg.norm(ref[:, :30], axis=1)
    eg = np.linalg.norm(got[:, 30:] - ref[:, 30:], axis=1) / np.linalg.norm(ref[:, 30:], axis=1)
    return es, eg


def sample(n, k=64, seed=4):
    return np.sort(np.random.default_rng(seed).choice(n, k, replace=False))


def test_adjoint_matches_dual_number_gradient(oracle, diff_run):
    """8,192 of the 65,536 agents against the reference's dual numbers
    (a few seconds of host time for 39-direction duals)."""
    sw = diff_run["sw"]
    idx = sample(sw.n, k=8192)
    sub = I.subset(sw, idx)
    fin, jac = oracle.jacobian(sub.state, sub.types, sub.glob, sub.dt, sub.n_steps, wp=sub.wp,
                               gains=sub.gains)
    seed = np.zeros((30, sub.n))
    seed[0:3] = 2.0 * (fin[0:3] - sub.extra["target"])
    seed[29] = sub.extra["cost_weight"]
    ref = np.einsum("ar,arc->ac", seed.T, jac)
    got = np.concatenate([diff_run["gx0"][:, idx].T, diff_run["gg"][:, idx].T], axis=1)
    es, eg = block_errors(got, ref)
    print(f"adjoint vs dual: state {es.max():.2e} gains {eg.max():.2e}", flush=True)
    assert es.max() <= TOL and eg.max() <= TOL


def test_adjoint_matches_central_differences(oracle, diff_run):
    sw = diff_run["sw"]
    idx = sample(sw.n, seed=9)
    sub = I.subset(sw, idx)
    tgt = sub.extra["target"].astype(np.float64)
    s0 = sub.state.astype(np.float64).copy()
    s0[0:3] -= tgt                                   # target-centred frame
    wp = sub.wp.astype(np.float64) - tgt[None]
    g0 = sub.gains.astype(np.float64)
    w = sub.extra["cost_weight"]

    def loss(s, g):
        f = oracle.rollout(s, sub.types, sub.glob, 1, sub.dt, sub.n_steps, wp=wp, gains=g)
        return np.sum(f[0:3] ** 2, axis=0) + w * f[29]

    fd = np.zeros((sub.n, 39))
    for c in range(39):
        sp, sm, gp, gm = s0.copy(), s0.copy(), g0.copy(), g0.copy()
        if c < 30:
            sp[c] += H; sm[c] -= H
        else:
            gp[c - 30] += H; gm[c - 30] -= H
        fd[:, c] = (loss(sp, gp) - loss(sm, gm)) / (2 * H)
    got = np.concatenate([diff_run["gx0"][:, idx].T, diff_run["gg"][:, idx].T], axis=1)
    es, eg = block_errors(got, fd)
    print(f"adjoint vs FD: state {es.max():.2e} gains {eg.max():.2e}", flush=True)
    assert es.max() <= TOL and eg.max() <= TOL


def test_adjoint_random_cotangent_all_rows(oracle, torch_dev):
    """Dot-product form: for random lambda_N on every physical row (controller
    memory and cost included), <lambda_0, dx_0> = <lambda_N, J dx_0> with the
    reference's Jacobian J, i.e. the GPU VJP equals J^T lambda_N."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config4(n=256, n_steps=120)
    K = 40
    sim = Simulator(sw.types, sw.glob, mode=1, steps_per_launch=30)
    x = torch.from_numpy(sw.state).to(dev)
    gains = torch.from_numpy(sw.gains).to(dev)
    wp = torch.from_numpy(sw.wp).to(dev)
    ckpt = torch.empty((3, 40, sw.n), device=dev)
    sim.step(x, 120, sw.dt, gains=gains, wp=wp, ckpt=ckpt, ckpt_every=K, carry=torch.zeros_like(x[:10]))
    lam = np.random.default_rng(3).normal(size=(30, sw.n)).astype(np.float32)
    gx0, gg = sim.step_backward(ckpt, K, 120, sw.dt, torch.from_numpy(lam).to(dev), gains=gains, wp=wp)
    torch.cuda.synchronize()
    sim.close()
    _, jac = oracle.jacobian(sw.state, sw.types, sw.glob, sw.dt, 120, wp=sw.wp, gains=sw.gains)
    ref = np.einsum("ar,arc->ac", lam.T.astype(np.float64), jac)
    got = np.concatenate([gx0.cpu().numpy().T, gg.cpu().numpy().T], axis=1)
    es, eg = block_errors(got, ref)
    assert es.max() <= TOL and eg.max() <= TOL
    dx = np.random.default_rng(4).normal(size=(sw.n, 39))
    lhs = np.sum(got * dx, axis=1)
    rhs = np.einsum("ar,arc,ac->a", lam.T.astype(np.float64), jac, dx)
    assert np.allclose(lhs, rhs, rtol=1e-3, atol=1e-3 * np.abs(rhs).max())


def test_checkpoint_interval_does_not_change_the_gradient(torch_dev):
    """Recomputation from checkpoints is exact: K = 1, 7 (a short last
    segment, an odd number of segments), 10, 50 and one segment of all steps
    give bitwise the same gradient."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config4(n=1000, n_steps=200)
    gains = torch.from_numpy(sw.gains).to(dev)
    wp = torch.from_numpy(sw.wp).to(dev)
    lam = torch.from_numpy(np.random.default_rng(1).normal(size=(30, sw.n)).astype(np.float32)).to(dev)
    outs = []
    for K in (10, 1, 7, 50, 200):
        sim = Simulator(sw.types, sw.glob, mode=1, steps_per_launch=64)
        x = torch.from_numpy(sw.state).to(dev)
        ckpt = torch.empty((-(-200 // K), 40, sw.n), device=dev)
        sim.step(x, 200, sw.dt, gains=gains, wp=wp, ckpt=ckpt, ckpt_every=K, carry=torch.zeros_like(x[:10]))
        gx0, gg = sim.step_backward(ckpt, K, 200, sw.dt, lam, gains=gains, wp=wp)
        torch.cuda.synchronize()
        outs.append((gx0.cpu().numpy(), gg.cpu().numpy()))
        sim.close()
    for o in outs[1:]:
        assert np.array_equal(o[0], outs[0][0]) and np.array_equal(o[1], outs[0][1])


def test_autotune_of_the_checkpointing_forward(torch_dev):
    """autotune(ckpt_every=K) times the variant that writes checkpoints, on
    scratch memory (the caller's state and carries are untouched), and the
    tuned shape then serves checkpointing calls: their checkpoints, final
    state and gradients equal those of an untuned run bit for bit."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config4(n=3000, n_steps=200)
    K = 50
    gains = torch.from_numpy(sw.gains).to(dev)
    wp = torch.from_numpy(sw.wp).to(dev)
    lam = torch.from_numpy(np.random.default_rng(2).normal(size=(30, sw.n)).astype(np.float32)).to(dev)
    outs = []
    for tune in (False, True):
        sim = Simulator(sw.types, sw.glob, mode=1)
        x = torch.from_numpy(sw.state).to(dev)
        carry = torch.zeros_like(x[:10])
        if tune:
            before = x.clone()
            shape = sim.autotune(x, sw.dt, 200, gains=gains, wp=wp, carry=carry, ckpt_every=K)
            torch.cuda.synchronize()
            assert torch.equal(x, before) and not carry.any()
            assert shape["block"] in (64, 128, 256, 512, 1024) and 1 <= shape["steps_per_launch"] <= 200
        ckpt = torch.empty((200 // K, 40, sw.n), device=dev)
        sim.step(x, 200, sw.dt, gains=gains, wp=wp, ckpt=ckpt, ckpt_every=K, carry=carry)
        gx0, gg = sim.step_backward(ckpt, K, 200, sw.dt, lam, gains=gains, wp=wp)
        torch.cuda.synchronize()
        outs.append([t.cpu().numpy() for t in (x, ckpt, gx0, gg)])
        sim.close()
    for a, b in zip(*outs):
        assert np.array_equal(a, b)


def test_autograd_function_matches_direct_call(diff_run, torch_dev):
    torch, dev = torch_dev
    from paper_2308_12698_amd.autograd import rollout
    sw, sim = diff_run["sw"], diff_run["sim"]
    x0 = torch.from_numpy(sw.state).to(dev).requires_grad_(True)
    gains = diff_run["gains_t"].clone().requires_grad_(True)
    xN = rollout(x0, gains, sim, diff_run["wp_t"], sw.dt, sw.n_steps, sw.extra["ckpt_every"])
    tgt = torch.from_numpy(sw.extra["target"]).to(dev)
    L = ((xN[0:3] - tgt) ** 2).sum() + sw.extra["cost_weight"] * xN[29].sum()
    L.backward()
    torch.cuda.synchronize()
    assert np.array_equal(xN.detach().cpu().numpy(), diff_run["final"])
    # the loss cotangent is formed by autograd here and by hand there
    assert np.allclose(x0.grad[:30].cpu().numpy(), diff_run["gx0"], rtol=1e-5, atol=1e-7)
    assert np.allclose(gains.grad.cpu().numpy(), diff_run["gg"], rtol=1e-5, atol=1e-7)
    assert x0.grad.shape == x0.shape


def test_adjoint_heterogeneous_budgets(oracle, torch_dev):
    """Agents past their budget pass the cotangent through unchanged and get
    zero gain gradient; the others match the reference."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.config4(n=300, n_steps=150)
    t_short = dict(sw.types[0]); t_short["budget"] = 70
    t_zero = dict(sw.types[0]); t_zero["budget"] = 0
    types = [sw.types[0], t_short, t_zero]
    ti = (np.arange(sw.n) % 3).astype(np.uint8)
    sim = Simulator(types, sw.glob, mode=1, steps_per_launch=64, debug=True)
    x = torch.from_numpy(sw.state).to(dev)
    gains = torch.from_numpy(sw.gains).to(dev)
    wp = torch.from_numpy(sw.wp).to(dev)
    tid = torch.from_numpy(ti).to(dev)
    ckpt = torch.empty((3, 40, sw.n), device=dev)
    sim.step(x, 150, sw.dt, gains=gains, wp=wp, type_idx=tid, ckpt=ckpt, ckpt_every=50, carry=torch.zeros_like(x[:10]))
    lam = np.random.default_rng(2).normal(size=(30, sw.n)).astype(np.float32)
    gx0, gg = sim.step_backward(ckpt, 50, 150, sw.dt, torch.from_numpy(lam).to(dev), gains=gains,
                                wp=wp, type_idx=tid)
    torch.cuda.synchronize()
    sim.close()
    gx0, gg = gx0.cpu().numpy(), gg.cpu().numpy()
    z = ti == 2
    assert np.array_equal(gx0[:, z], lam[:, z]) and np.all(gg[:, z] == 0)
    for t, steps in ((0, 150), (1, 70)):
        idx = np.where(ti == t)[0][:20]
        sub = I.subset(sw, idx)
        _, jac = oracle.jacobian(sub.state, sub.types, sub.glob, sub.dt, steps, wp=sub.wp, gains=sub.gains)
        ref = np.einsum("ar,arc->ac", lam[:, idx].T.astype(np.float64), jac)
        got = np.concatenate([gx0[:, idx].T, gg[:, idx].T], axis=1)
        es, eg = block_errors(got, ref)
        assert es.max() <= TOL and eg.max() <= TOL, (t, es.max(), eg.max())


def test_backward_rejects_invalid_arguments(diff_run, torch_dev):
    torch, dev = torch_dev
    from paper_2308_12698_amd import _lib as L
    from paper_2308_12698_amd.sim import Simulator
    sw = diff_run["sw"]
    with pytest.raises(ValueError):
        diff_run["sim"].step_backward(diff_run["ckpt"], 0, sw.n_steps, sw.dt, diff_run["gfin"],
                                      gains=diff_run["gains_t"], wp=diff_run["wp_t"])
    open_sim = Simulator(sw.types, sw.glob, mode=0)
    with pytest.raises(L.PotatoError) as e:
        open_sim.step_backward(diff_run["ckpt"], 50, sw.n_steps, sw.dt, diff_run["gfin"],
                               wp=diff_run["wp_t"])
    assert e.value.status == L.EUNSUPPORTED
    open_sim.close()


def test_autotune_rejects_checkpoints_it_cannot_write(diff_run, torch_dev):
    """Tuning the checkpointing forward takes the checks of potato_step with
    a checkpoint buffer: ckpt_every < 0, no carries, open loop."""
    torch, dev = torch_dev
    from paper_2308_12698_amd import _lib as L
    from paper_2308_12698_amd.sim import Simulator
    sw = diff_run["sw"]
    sim = Simulator(sw.types, sw.glob, mode=1)
    x = torch.from_numpy(sw.state).to(dev)
    carry = torch.zeros_like(x[:10])
    with pytest.raises(L.PotatoError) as e:
        sim.autotune(x, sw.dt, 50, gains=diff_run["gains_t"], wp=diff_run["wp_t"], carry=carry, ckpt_every=-1)
    assert e.value.status == L.EINVAL
    with pytest.raises(L.PotatoError) as e:
        sim.autotune(x, sw.dt, 50, gains=diff_run["gains_t"], wp=diff_run["wp_t"], ckpt_every=10)
    assert e.value.status == L.EINVAL and "carr" in str(e.value)
    sim.close()
    open_sim = Simulator(sw.types, sw.glob, mode=0)
    cmd = torch.zeros((4, sw.n), device=dev)
    with pytest.raises(L.PotatoError) as e:
        open_sim.autotune(x, sw.dt, 50, motor_cmd=cmd, carry=carry, ckpt_every=10)
    assert e.value.status == L.EUNSUPPORTED
    open_sim.close()


def test_adjoint_in_the_controller_limits(oracle, torch_dev):
    """Gradients through the saturations and clamps (inputs.limits_swarm:
    rotors at the speed limit and at 0, the vertical-acceleration floor,
    clamped integrals, tumbling agents), 300 steps, checkpoints every 50,
    every agent against the reference's dual numbers.  A clamp passes no
    derivative while it holds, so for the climbers every path from the gains
    to the final state is cut: their reference gain gradient is exactly 0,
    and there the GPU's must be 0 too."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    sw = I.limits_swarm(n_group=32, n_steps=300)
    K = 50
    sim = Simulator(sw.types, sw.glob, mode=1, form="fused", steps_per_launch=100)
    x = torch.from_numpy(sw.state).to(dev)
    gains = torch.from_numpy(sw.gains).to(dev)
    wp = torch.from_numpy(sw.wp).to(dev)
    ckpt = torch.empty((sw.n_steps // K, 40, sw.n), device=dev)
    sim.step(x, sw.n_steps, sw.dt, gains=gains, wp=wp, ckpt=ckpt, ckpt_every=K, carry=torch.zeros_like(x[:10]))
    seed = np.zeros((30, sw.n), dtype=np.float32)
    seed[0:3], seed[3:6], seed[29] = 1.0, 0.5, 1e-4
    gx0, gg = sim.step_backward(ckpt, K, sw.n_steps, sw.dt, torch.from_numpy(seed).to(dev),
                                gains=gains, wp=wp)
    torch.cuda.synchronize()
    got = np.concatenate([gx0.cpu().numpy().T, gg.cpu().numpy().T], axis=1)
    sim.close()
    _, jac = oracle.jacobian(sw.state, sw.types, sw.glob, sw.dt, sw.n_steps, wp=sw.wp, gains=sw.gains)
    ref = np.einsum("ar,arc->ac", seed.T.astype(np.float64), jac)
    g = sw.n // 4
    for k, name in enumerate(sw.extra["groups"]):
        sl = slice(k * g, (k + 1) * g)
        for blk, cols in (("state", slice(0, 30)), ("gains", slice(30, 39))):
            r = np.linalg.norm(ref[sl, cols], axis=1)
            d = np.linalg.norm(got[sl, cols] - ref[sl, cols], axis=1)
            cut = r == 0.0
            e = np.where(cut, 0.0, d / np.where(cut, 1.0, r))
            print(f"{name} {blk}: worst {e.max():.2e}, {int(cut.sum())} exactly zero "
                  f"(GPU there <= {d[cut].max() if cut.any() else 0.0:.1e})", flush=True)
            assert e.max() <= TOL
            assert not cut.any() or d[cut].max() == 0.0


@pytest.mark.parametrize("het", [False, True], ids=["homogeneous", "heterogeneous"])
def test_pipelined_adjoint_is_bitwise_the_one_wave_adjoint(torch_dev, het):
    """Swarms too small to give every SIMD two waves take the pipelined
    reverse sweep (one recomputing and one reversing wave per 64 agents),
    larger ones one agent per thread.  An agent's gradient must not depend
    on which: 4,096 agents alone (pipelined) against the same agents at the
    front of a 262,144-agent swarm (one per thread), bit for bit; with step
    budgets ending inside segments, the type order and dead agents in the
    heterogeneous case."""
    torch, dev = torch_dev
    import ctypes as C
    from paper_2308_12698_amd import _lib as L
    from paper_2308_12698_amd.sim import Simulator
    K, n_steps = 50, 150
    small = I.config4(n=4096, n_steps=n_steps)
    types = [small.types[0]]
    ti_small = alive_small = None
    if het:
        alive_small = (np.random.default_rng(9).random(small.n) > 0.1).astype(np.uint8)
        types = [dict(t, budget=b) for t, b in zip(I.hetero_types(), (37, 150, 75, 120, 149, 50, 99, 1))]
        ti_small = np.random.default_rng(7).integers(0, len(types), small.n).astype(np.uint8)
    reps = 64
    runs = []
    for n in (small.n, small.n * reps):
        sim = Simulator(types, small.glob, mode=1, form="fused", steps_per_launch=50)
        tile = lambda a: np.ascontiguousarray(np.tile(a, (1,) * (a.ndim - 1) + (n // small.n,)))
        x = torch.from_numpy(tile(small.state)).to(dev)
        gains = torch.from_numpy(tile(small.gains)).to(dev)
        wp = torch.from_numpy(tile(small.wp)).to(dev)
        ti = perm = alive = None
        if het:
            ti = torch.from_numpy(tile(ti_small)).to(dev)
            perm = sim.order_by_type(ti)
            alive = torch.from_numpy(tile(alive_small)).to(dev)
        ckpt = torch.empty((n_steps // K, 40, n), device=dev)
        sim.step(x, n_steps, small.dt, gains=gains, wp=wp, ckpt=ckpt, ckpt_every=K, type_idx=ti, perm=perm,
                 alive=alive, carry=torch.zeros_like(x[:10]))
        seed = torch.from_numpy(tile(np.random.default_rng(8).normal(size=(30, small.n)).astype(np.float32))).to(dev)
        pp = L.Params(C.c_void_p(ti.data_ptr()) if het else None, C.c_void_p(perm.data_ptr()) if het else None,
                      C.c_void_p(gains.data_ptr()), n, None)
        ws = int(sim._lib.potato_backward_workspace_bytes(sim._h, C.byref(pp), n, K))
        gx0, gg = sim.step_backward(ckpt, K, n_steps, small.dt, seed, gains=gains, wp=wp, type_idx=ti, perm=perm,
                                    alive=alive)
        torch.cuda.synchronize()
        runs.append((ws, gx0[:, :small.n].cpu().numpy(), gg[:, :small.n].cpu().numpy()))
        sim.close()
    tape_per_thread = K * 31 * 4          # 31 tape rows per step (state, held command, branch bits)
    assert runs[0][0] == tape_per_thread * 128 * (small.n // 64)      # pipelined: 64 blocks of 2 waves
    assert runs[1][0] % (tape_per_thread * 256) == 0                   # one agent per thread, 256-thread blocks
    assert np.isfinite(runs[0][1]).all() and np.abs(runs[0][2]).max() > 0
    assert np.array_equal(runs[0][1], runs[1][1]) and np.array_equal(runs[0][2], runs[1][2])
    if het:
        # dead agents: the cotangent passes through unchanged, no gain gradient
        dead = alive_small == 0
        seed0 = np.random.default_rng(8).normal(size=(30, small.n)).astype(np.float32)
        assert np.array_equal(runs[0][1][:, dead], seed0[:, dead]) and not runs[0][2][:, dead].any()


def test_backward_contract_17_rows_and_optional_memory(torch_dev, diff_run):
    """Through the C ABI: grad_x0 is the 17 rows of the rigid body and rotors
    ([17][ld]) and grad_mem, when given, the 13 rows of controller memory and
    cost ([13][ld]); buffers of exactly those rows with guard rows after them
    come back with every guard element untouched, and the values equal the
    binding's 30-row result."""
    import ctypes as C
    torch, dev = torch_dev
    from paper_2308_12698_amd import _lib as L
    sw, sim = diff_run["sw"], diff_run["sim"]
    n, K, guard, sentinel = sw.n, sw.extra["ckpt_every"], 4, -7777.0
    pp = L.Params(None, None, C.c_void_p(diff_run["gains_t"].data_ptr()), n, None)
    wp = diff_run["wp_t"]
    cm = L.Cmds(None, C.c_void_p(wp.data_ptr()), wp.shape[0], 0, wp.shape[2], 0)
    nbytes = int(sim._lib.potato_backward_workspace_bytes(sim._h, C.byref(pp), n, K))
    ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    for with_mem in (False, True):
        gx = torch.full((17 + guard, n), sentinel, device=dev)
        gm = torch.full((13 + guard, n), sentinel, device=dev) if with_mem else None
        gg = torch.zeros((9, n), device=dev)
        rc = sim._lib.potato_step_backward(sim._h, C.byref(pp), C.byref(cm), float(sw.dt), n, sw.n_steps,
                                           C.c_void_p(diff_run["ckpt"].data_ptr()), K, n,
                                           C.c_void_p(diff_run["gfin"].data_ptr()), C.c_void_p(gx.data_ptr()),
                                           None if gm is None else C.c_void_p(gm.data_ptr()),
                                           C.c_void_p(gg.data_ptr()), C.c_void_p(ws.data_ptr()), nbytes, None)
        L.check(rc)
        torch.cuda.synchronize()
        assert torch.all(gx[17:] == sentinel)
        assert np.array_equal(gx[:17].cpu().numpy(), diff_run["gx0"][:17])
        assert np.array_equal(gg.cpu().numpy(), diff_run["gg"])
        if with_mem:
            assert torch.all(gm[13:] == sentinel)
            assert np.array_equal(gm[:13].cpu().numpy(), diff_run["gx0"][17:30])


@pytest.mark.parametrize("n_steps", [15, 16, 17, 60])
def test_integrals_off_the_tape_at_clamps(torch_dev, n_steps):
    """The reverse sweep takes the controller's integrals from the tape only
    at every 16th step and where an agent is at a clamp.  Agents that start
    at, near and away from the three clamps, with waypoints and rates that
    drive them in and out of them: an agent's gradient does not depend on the
    checkpoint interval, on which agents share its wave, or on the kernel
    (a swarm small enough for the pipelined one, and 70,016 agents), bit for
    bit.  Most agents meet a clamp."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    n = 256
    rng = np.random.default_rng(n_steps)
    glob = I.globals_f32(ipos_max=0.5, iatt_max=0.05, irate_max=0.1)
    s = I.hover_state(rng.uniform(0.0, 20.0, (3, n))).astype(np.float64)
    s[10:13] = rng.normal(0.0, 1.0, (3, n))
    for rows, top in ((slice(17, 20), 0.5), (slice(20, 23), 0.05), (slice(23, 26), 0.1)):
        near = rng.uniform(0.97, 1.0, (3, n)) * rng.choice([-1.0, 1.0], (3, n))
        s[rows] = top * np.where(rng.random((3, n)) < 0.5, near, rng.uniform(-0.5, 0.5, (3, n)))
    s[17:26] = np.clip(s[17:26], -np.repeat([0.5, 0.05, 0.1], 3)[:, None], np.repeat([0.5, 0.05, 0.1], 3)[:, None])
    wp = s[0:3] + rng.uniform(-3.0, 3.0, (3, n))
    gains = np.asarray(I.DEFAULT_GAINS)[:, None] * rng.uniform(0.8, 1.2, (9, n))
    lam = rng.normal(size=(30, n))
    shuffle = rng.permutation(n)

    def gradient(K, pick, reps=1):
        up = lambda a: torch.from_numpy(np.ascontiguousarray(I.f32(np.tile(a[:, pick], (1, reps))))).to(dev)
        sim = Simulator([I.base_type()], glob, mode=1)
        x, m = up(s), n * reps
        w, g = up(wp)[None].contiguous(), up(gains)
        ckpt = torch.empty((-(-n_steps // K), 40, m), device=dev)
        sim.step(x, n_steps, 2e-3, gains=g, wp=w, ckpt=ckpt, ckpt_every=K, carry=torch.zeros_like(x[:10]))
        gx, gg = sim.step_backward(ckpt, K, n_steps, 2e-3, up(lam), gains=g, wp=w)
        torch.cuda.synchronize()
        sim.close()
        both = torch.cat([gx, gg])[:, :n].cpu().numpy()
        out = np.empty_like(both)
        out[:, pick] = both
        return out, x[17:26, :n].cpu().numpy()

    ref, end = gradient(50, np.arange(n))
    assert np.isfinite(ref).all()
    limit = I.f32(np.repeat([0.5, 0.05, 0.1], 3))[:, None]
    if n_steps == 60:
        assert (np.abs(end) == limit).any(axis=0).mean() > 0.3
    for K, pick, reps in ((1, np.arange(n), 1), (7, shuffle, 1), (16, np.arange(n), 1), (50, shuffle, 1),
                          (50, np.arange(n), 274), (7, shuffle, 274)):
        assert np.array_equal(gradient(K, pick, reps)[0], ref), (K, reps)


@pytest.mark.parametrize("n", [49152, 65536, 131137])
@pytest.mark.parametrize("types", [1, 8])
def test_streamed_tape_gives_the_same_gradient(torch_dev, n, types):
    """Tapes of more than 192 MiB are read with streaming loads: 50 steps
    per segment, pipelined (49,152 and 65,536 agents) and one agent per
    thread in more than one round (131,137 agents), against 7 steps per
    segment, whose tapes are a seventh of that.  Gradients bit for bit, types
    with different budgets, dead agents."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    gen = torch.Generator(device=dev)
    gen.manual_seed(n)
    rand = lambda *shape: torch.rand(shape, device=dev, generator=gen)
    table = [I.base_type()] if types == 1 else [dict(t, budget=b) for t, b in
                                                zip(I.hetero_types(), (37, 50, 75, 120, 149, 53, 99, 1))]
    ti = None if types == 1 else torch.randint(0, types, (n,), device=dev, generator=gen, dtype=torch.uint8)
    gains = (torch.tensor(I.DEFAULT_GAINS, device=dev)[:, None] * (rand(9, n) * 0.4 + 0.8)).contiguous()
    alive = (rand(n) > 0.1).to(torch.uint8)
    start = torch.zeros((30, n), device=dev)
    start[0:3] = rand(3, n) * 50.0
    start[6] = 1.0
    start[10:13] = rand(3, n) - 0.5
    wp = (start[0:3] + rand(3, n) * 8.0 - 4.0)[None].contiguous()
    seed = rand(30, n) - 0.5
    sim = Simulator(table, I.globals_f32(), mode=1)
    out = []
    for K in (7, 50):
        x = start.clone()
        ckpt = torch.empty((-(-56 // K), 40, n), device=dev)
        sim.step(x, 56, 1e-3, gains=gains, wp=wp, ckpt=ckpt, ckpt_every=K, type_idx=ti, alive=alive,
                 carry=torch.zeros_like(x[:10]))
        out.append(torch.cat(sim.step_backward(ckpt, K, 56, 1e-3, seed, gains=gains, wp=wp, type_idx=ti, alive=alive)))
    torch.cuda.synchronize()
    sim.close()
    assert torch.isfinite(out[0]).all() and out[0][30:].abs().max() > 0
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("n", [250, 70016])
@pytest.mark.parametrize("types", [1, 8])
@pytest.mark.parametrize("first", [1, 7, 23])
def test_a_call_in_two_parts_has_the_bits_of_one(torch_dev, n, types, first):
    """The reverse of step k reads the forward's integrals before it, bit for
    bit, wherever in a call the step is: a rollout of 60 steps in one call,
    and in calls of `first` and the rest with the second's cotangents given
    to the first, give the same cotangents of state and memory (steps,
    waypoint epochs and budgets counted across the calls; integrals through
    zero, near and at their clamps, far larger and far smaller than their
    increments).  Pipelined sweep and one agent per thread."""
    torch, dev = torch_dev
    from paper_2308_12698_amd.sim import Simulator
    rng = np.random.default_rng(first + types)
    m, steps, every = 250, 60, 20
    table = [I.base_type()] if types == 1 else [dict(t, budget=b) for t, b in
                                                zip(I.hetero_types(), (60, 59, 40, 24, 23, 7, 6, 1000))]
    glob = I.globals_f32(ipos_max=0.5, iatt_max=0.05, irate_max=0.3)
    s = I.hover_state(rng.uniform(0.0, 20.0, (3, m))).astype(np.float64)
    s[10:13] = rng.normal(0.0, 0.5, (3, m))
    s[17:26] = rng.uniform(-1.0, 1.0, (9, m)) * np.repeat([0.5, 0.05, 0.3], 3)[:, None] * 10.0 ** rng.uniform(-6, 0, (9, m))
    wp = s[0:3] + rng.uniform(-2.0, 2.0, (2, 3, m))
    gains = np.asarray(I.DEFAULT_GAINS)[:, None] * rng.uniform(0.8, 1.2, (9, m))
    reps = n // m + 1
    up = lambda a: torch.from_numpy(np.ascontiguousarray(I.f32(np.tile(a, reps)[..., :n]))).to(dev)
    ti = None if types == 1 else torch.from_numpy(np.tile(rng.integers(0, types, m).astype(np.uint8), reps)[:n]).to(dev)
    W, G, lam = up(wp), up(gains), up(rng.normal(size=(30, m)))
    sim = Simulator(table, glob, mode=1)

    def rollout(parts):
        x, ca, legs, k = up(s), torch.zeros((10, n), device=dev), [], 0
        for count in parts:
            ck = torch.empty((-(-count // every), 40, n), device=dev)
            sim.step(x, count, 1e-3, type_idx=ti, gains=G, wp=W, resample_every=11, step0=k, ckpt=ck, ckpt_every=every,
                     carry=ca)
            legs.append((ck, count, k))
            k += count
        g = lam
        for ck, count, k0 in reversed(legs):
            g, _ = sim.step_backward(ck, every, count, 1e-3, g, type_idx=ti, gains=G, wp=W, resample_every=11, step0=k0)
        torch.cuda.synchronize()
        return x.cpu().numpy(), g.cpu().numpy()

    x1, g1 = rollout((steps,))
    x2, g2 = rollout((first, steps - first))
    sim.close()
    assert np.array_equal(x1, x2) and np.isfinite(g1).all()
    assert np.array_equal(g1, g2), np.abs(g1 - g2).max()
