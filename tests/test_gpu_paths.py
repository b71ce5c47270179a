"""GPU tests of single kernel branches at the sizes where they can go wrong,
against the FP64 CPU oracle.

Tolerances (fixed before the first run): FP64 sums of at most a few hundred terms
with cancellation to O(1) leave relative errors of 1e-15 to 1e-13, and the few
optimizer steps from perturbed starts do not amplify them; 1e-10 leaves three orders
of margin."""

import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

TOL = 1e-10


@pytest.fixture(scope="module")
def dpf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_28203_amd as m
    m.lib()
    return m


def cu(x, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(x)).to("cuda", dtype)


def random_grid(rng, n, m, hub=0):
    """Random tree plus chords in an arbitrary numbering, with a hub bus of about
    ``hub`` further branches (one matrix row much longer than the others)."""
    f, t = synth.tree_chord_grid(rng, n, m)
    if hub:
        c = int(rng.integers(0, n))
        others = rng.choice(np.setdiff1d(np.arange(n), [c]), size=hub, replace=False)
        f = np.concatenate([f, np.full(hub, c, np.int32)])
        t = np.concatenate([t, others.astype(np.int32)])
    nb = len(f)
    bt = np.zeros(n, np.int8)
    kinds = rng.permutation(n)
    bt[kinds[0]] = 2
    bt[kinds[1:1 + max(1, n // 7)]] = 1
    va = rng.uniform(-0.1, 0.1, n)
    va[kinds[0]] = 0.0
    return synth.Grid(n, f.astype(np.int32), t.astype(np.int32), rng.uniform(0.01, 0.1, nb), rng.uniform(0.05, 0.3, nb),
                      rng.uniform(0.0, 0.05, nb), bt, rng.uniform(0.97, 1.03, n), va)


@pytest.mark.parametrize("n,m,hub", [(2, 1, 0), (64, 100, 40), (65, 98, 40), (256, 380, 20), (257, 400, 12),
                                     (512, 700, 0), (513, 900, 9), (1100, 1600, 30), (1537, 2200, 17),
                                     (2048, 3000, 5), (130, 5000, 0)])
def test_register_solves_at_their_size_edges(dpf, n, m, hub):
    """The register-resident kernels on sorted rows: one and several rows per thread,
    rows longer than the columns kept in registers and than the last sort key, a
    matrix that does not fit the workgroup's LDS (130 buses, 5000 branches), outages,
    and optimizer state in and out; angles beyond pi/4 in one case."""
    rng = np.random.default_rng(41000 + n)
    g = random_grid(rng, n, m, hub)
    B, steps = 3, 6
    S0 = oracle.injections(oracle.ybus_of(g), g.vm, g.va)
    S = S0[None] * rng.uniform(0.97, 1.03, (B, 1))
    vm0 = g.vm[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type == 0)
    va0 = g.va[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type != 2)
    va0[2] += 2.5 * (g.bus_type != 2)
    nbr = synth.non_bridge_branches(n, g.f, g.t)
    outage = np.array([-1, nbr[len(nbr) // 2] if len(nbr) else -1, -1], np.int32)
    state = torch.zeros(4, B, n, dtype=torch.float64, device="cuda")
    vm, va = cu(vm0), cu(va0)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    out = dpf.solve(Yg, g.bus_type, cu(S, torch.complex128), vm, va, outage=cu(outage, torch.int32), adam_state=state,
                    sched_state=dpf.fresh_sched_state(B, 1e-3),
                    opts=dpf.Options(lr=1e-3, tol=0.0, max_iter=steps))
    assert out["iters"].tolist() == [steps] * B
    for c in range(B):
        ref = oracle.solve_adam(oracle.ybus_of(g, skip=int(outage[c])), g.bus_type, S[c], vm0[c], va0[c],
                                oracle.AdamOptions(lr=1e-3, tol=0.0, max_iter=steps))
        assert np.abs(vm[c].cpu().numpy() - ref["vm"]).max() < TOL, c
        assert np.abs(va[c].cpu().numpy() - ref["va"]).max() < TOL, c
        assert abs(out["max_mis"][c].item() - ref["mu"]) <= TOL * max(1.0, ref["mu"]), c
    # the moments of coordinates that are not learnable come back as they went in
    fixed = cu(g.bus_type != 0, torch.bool)
    assert (state[0][:, fixed] == 0).all() and (state[2][:, fixed] == 0).all()


@pytest.mark.parametrize("n,m,hub", [(2049, 3000, 30), (3072, 4300, 0), (3073, 4400, 0), (3413, 4800, 8), (4096, 5600, 0)])
def test_resident_solves_above_the_register_kernels(dpf, n, m, hub):
    """The default kernels of 2049 to 4096 buses with more items than fill half of the
    device (sizes at the edges of rows per thread and of the third LDS array), with an
    outage, optimizer state and angles beyond pi/4."""
    rng = np.random.default_rng(42000 + n)
    g = random_grid(rng, n, m, hub)
    B, steps, checked = 160, 4, (0, 1, 2, 159)
    S = oracle.injections(oracle.ybus_of(g), g.vm, g.va) * 0.98
    vm0 = g.vm[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type == 0)
    va0 = g.va[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type != 2)
    va0[2] += 2.5 * (g.bus_type != 2)
    nbr = synth.non_bridge_branches(n, g.f, g.t)
    outage = np.full(B, -1, np.int32)
    outage[1] = nbr[len(nbr) // 2]
    outage[159] = nbr[0]
    state = torch.zeros(4, B, n, dtype=torch.float64, device="cuda")
    vm, va = cu(vm0), cu(va0)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    v = dpf.variants()[dpf.variant_for(n, B)]
    assert v["kind"] == "register" and v["threads"] * v["buses_per_thread"] >= n
    out = dpf.solve(Yg, g.bus_type, cu(S, torch.complex128), vm, va, outage=cu(outage, torch.int32), adam_state=state,
                    sched_state=dpf.fresh_sched_state(B, 1e-3), opts=dpf.Options(lr=1e-3, tol=0.0, max_iter=steps))
    assert out["iters"].tolist() == [steps] * B
    for c in checked:
        ref = oracle.solve_adam(oracle.ybus_of(g, skip=int(outage[c])), g.bus_type, S, vm0[c], va0[c],
                                oracle.AdamOptions(lr=1e-3, tol=0.0, max_iter=steps))
        assert np.abs(vm[c].cpu().numpy() - ref["vm"]).max() < TOL, c
        assert np.abs(va[c].cpu().numpy() - ref["va"]).max() < TOL, c
    fixed = cu(g.bus_type != 0, torch.bool)
    assert (state[0][:, fixed] == 0).all() and (state[2][:, fixed] == 0).all()


@pytest.mark.parametrize("n,m,B", [(2, 1, 2), (64, 100, 3), (65, 99, 2), (256, 380, 2), (257, 390, 2), (1024, 1500, 2),
                                   (1025, 1500, 2), (2048, 3000, 2), (2049, 3000, 3), (2049, 3000, 64),
                                   (5121, 7300, 64), (10176, 14500, 64), (10300, 14700, 64)])
def test_evaluation_by_case_and_by_bus(dpf, n, m, B):
    """dpf_mismatch_grad at the edges of its kernels (rows per thread of the
    one-workgroup-per-case form, its largest grid, one bus-per-thread form beyond it
    and for few cases of large grids), with a hub row, an outage, per-case injections
    and angles beyond pi/4; and without outputs that are not asked for."""
    rng = np.random.default_rng(43000 + n + B)
    g = random_grid(rng, n, m, min(70, n // 3))
    S0 = oracle.injections(oracle.ybus_of(g), g.vm, g.va)
    S = S0[None] * rng.uniform(0.9, 1.1, (B, n))
    vm = g.vm[None] + rng.normal(0, 1e-2, (B, n))
    va = g.va[None] + rng.normal(0, 1e-2, (B, n))
    va[1] += 2.5
    nbr = synth.non_bridge_branches(n, g.f, g.t)
    outage = np.full(B, -1, np.int32)
    if len(nbr):
        outage[1] = nbr[len(nbr) // 2]
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    args = (Yg, g.bus_type, cu(S, torch.complex128), cu(vm), cu(va))
    r = dpf.mismatch_grad(*args, outage=cu(outage, torch.int32))
    for c in sorted({0, 1, B - 1}):
        Yo = oracle.ybus_of(g, skip=int(outage[c]))
        loss, mu, gv, ga = oracle.loss_grad(Yo, g.bus_type, vm[c], va[c], S[c])
        dS = oracle.injections(Yo, vm[c], va[c]) - S[c]
        assert abs(r["loss"][c].item() - loss) <= TOL * loss
        assert abs(r["max_mis"][c].item() - mu) <= TOL * mu
        for x, ref in ((r["dS"], dS), (r["g_vm"], gv), (r["g_va"], ga)):
            assert np.abs(x[c].cpu().numpy() - ref).max() <= TOL * max(np.abs(ref).max(), 1e-300), c
    few = dpf.mismatch_grad(*args, outage=cu(outage, torch.int32), want_dS=False, want_grad=False)
    assert torch.equal(few["loss"], r["loss"]) and torch.equal(few["max_mis"], r["max_mis"])


@pytest.mark.parametrize("n,m", [(2049, 3000), (5080, 7300)])
def test_branch_gradients_by_case_and_by_bus(dpf, n, m):
    """dpf_param_grad of the same case alone (one thread per bus) and in a batch of 64
    (one workgroup per case) agrees; the branch that is out gets 0."""
    rng = np.random.default_rng(44000 + n)
    g = random_grid(rng, n, m, 20)
    S = oracle.injections(oracle.ybus_of(g), g.vm, g.va) * 0.97
    vm = cu(np.tile(g.vm + rng.normal(0, 1e-2, n), (64, 1)))
    va = cu(np.tile(g.va + rng.normal(0, 1e-2, n), (64, 1)))
    out = cu(np.full(64, synth.non_bridge_branches(n, g.f, g.t)[0]), torch.int32)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    one = dpf.param_grad(Yg, g.bus_type, cu(S, torch.complex128), vm[:1], va[:1], outage=out[:1])
    many = dpf.param_grad(Yg, g.bus_type, cu(S, torch.complex128), vm, va, outage=out)
    for k in ("loss", "max_mis", "g_r", "g_x", "g_b", "g_s"):
        a, b = one[k][0].cpu().numpy(), many[k].cpu().numpy()
        for c in (0, 63):
            assert np.abs(a - b[c]).max() <= TOL * max(np.abs(a).max(), 1e-300), (k, c)
    assert (many["g_r"][:, out[0].item()] == 0).all() and (one["g_x"][:, out[0].item()] == 0).all()


@pytest.mark.parametrize("n,m,hub", [(2, 1, 0), (64, 90, 40), (65, 90, 9), (513, 760, 30), (1537, 2300, 12),
                                     (3072, 4400, 0), (3073, 4400, 20), (4097, 5900, 10), (8193, 11800, 0)])
def test_dc_start_at_its_size_edges(dpf, n, m, hub):
    """dpf_dc_init at the edges of its kernels (rows per thread, rows longer than the
    entries kept in registers, the largest register form and the form beyond it), with
    a non-zero slack angle and an outage, against the oracle's direct solve."""
    rng = np.random.default_rng(45000 + n)
    g = random_grid(rng, n, m, hub)
    S = rng.normal(0, 0.1, (3, n)) + 0j
    nbr = synth.non_bridge_branches(n, g.f, g.t)
    outage = np.array([-1, nbr[0] if len(nbr) else -1, -1], np.int32)
    va0 = np.zeros((3, n))
    va0[:, g.slack] = 0.25
    va = cu(va0)
    Yg = dpf.build_dc_grid(n, g.f, g.t, g.x)
    r = dpf.dc_init(Yg, g.bus_type, cu(S, torch.complex128), va, outage=cu(outage, torch.int32), tol=1e-13)
    assert (r["residual"] <= 1e-13).all()
    for c in range(3):
        ref = oracle.dc_power_flow(g, g.bus_type, S[c], va_slack=0.25, skip=int(outage[c]))
        assert np.abs(va[c].cpu().numpy() - ref).max() <= 1e-9 * max(1.0, np.abs(ref).max()), c


@pytest.mark.parametrize("n,hub,twins", [(1, 0, 0), (2, 0, 3), (128, 15, 4), (129, 16, 9), (3000, 900, 200),
                                         (32768, 40, 500), (32769, 17, 500), (300000, 300, 2000)])
def test_ybus_build_at_its_size_edges(dpf, n, hub, twins):
    """dpf_build_ybus at the edges of its kernels (rows sorted in LDS or in place, one
    workgroup or several for the slots, the totals added up or scanned, the static
    array or memory of its own), with a hub row and parallel branches in both
    directions: pattern exact, values to the rounding of their sums (1e-15 relative to the
    row's largest entry, which the branch-order sums keep)."""
    rng = np.random.default_rng(46000 + n)
    k = np.arange(1, n)
    f = np.concatenate([k - 1 - rng.integers(0, np.minimum(k, 7)), np.zeros(hub, np.int64)]).astype(np.int32)
    t = np.concatenate([k, 1 + rng.choice(max(1, n - 1), size=hub, replace=False)]).astype(np.int32)
    if n > 1 and twins:
        pick = rng.integers(0, len(f), twins)
        f, t = np.concatenate([f, t[pick]]), np.concatenate([t, f[pick]])
    m = len(f)
    r, x, b = rng.uniform(0.01, 0.1, m), rng.uniform(0.05, 0.3, m), rng.uniform(0, 0.05, m)
    y, ysh = 1.0 / (r + 1j * x), 0.5j * b
    d = np.arange(n, dtype=np.int64)
    f64, t64 = f.astype(np.int64), t.astype(np.int64)
    key = np.concatenate([d * n + d, f64 * n + f64, t64 * n + t64, f64 * n + t64, t64 * n + f64])
    u, at = np.unique(key, return_inverse=True)
    v = np.concatenate([np.zeros(n), y + ysh, y + ysh, -y, -y])
    ref = np.bincount(at, v.real, len(u)) + 1j * np.bincount(at, v.imag, len(u))
    Y = dpf.build_ybus(n, f, t, r, x, b)
    ptr = np.searchsorted(u // n, np.arange(n + 1))
    assert Y.nnz == len(u) and Y.max_row_nnz == np.diff(ptr).max()
    assert np.array_equal(Y.row_ptr.cpu().numpy(), ptr) and np.array_equal(Y.col_idx.cpu().numpy(), u % n)
    scale = np.maximum.reduceat(np.abs(ref), ptr[:-1])[u // n]
    assert (np.abs(Y.val.cpu().numpy() - ref) <= 1e-15 * np.maximum(scale, np.abs(ref)) * np.sqrt(1 + hub)).all()
    if n > 1:  # too small a capacity: the needed size is reported, no entry is written
        import ctypes
        col = torch.full((Y.nnz,), -7, dtype=torch.int32, device="cuda")
        val = torch.full((Y.nnz,), 5.0, dtype=torch.complex128, device="cuda")
        row = torch.empty(n + 1, dtype=torch.int32, device="cuda")
        nnz, mx = ctypes.c_int32(0), ctypes.c_int32(0)
        rc = dpf.lib().dpf_build_ybus(n, m, *(ctypes.c_void_p(z.data_ptr()) for z in (Y.f, Y.t, Y.r, Y.x, Y.b)),
                                      Y.nnz - 1, *(ctypes.c_void_p(z.data_ptr()) for z in (row, col, val)),
                                      ctypes.byref(nnz), ctypes.byref(mx),
                                      ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == dpf.binding.DPF_ECAP and nnz.value == Y.nnz
        assert (col == -7).all() and (val == 5.0).all()


def test_ybus_builds_from_several_threads(dpf):
    """Overlapping builds on one device (the static array is used by one at a time, the
    allocating call falls back to memory of its own) all give the grid's own matrix."""
    import threading
    grids = [random_grid(np.random.default_rng(47000 + k), 500 + 300 * k, 800 + 450 * k) for k in range(4)]
    want = [dpf.build_ybus(g.n_bus, g.f, g.t, g.r, g.x, g.b) for g in grids]
    bad = []

    def work(k):
        g = grids[k]
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(20):
                Y = dpf.build_ybus(g.n_bus, g.f, g.t, g.r, g.x, g.b, noalloc=(i + k) % 2 == 0)
                torch.cuda.current_stream().synchronize()
                if not (torch.equal(Y.col_idx, want[k].col_idx) and torch.equal(Y.val, want[k].val)):
                    bad.append((k, i))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert not bad


@pytest.mark.parametrize("n,m,numbered", [(2049, 3000, False), (2500, 3900, True), (6000, 8800, True), (6000, 8800, False),
                                          (10300, 14700, True)])
def test_few_large_items_on_persistent_teams(dpf, n, m, numbered):
    """Few large items on the persistent teams: members of at most one row per thread
    with their matrix and halo in LDS (small-bandwidth numberings), members whose columns
    lie outside their window or whose halo exceeds its list (arbitrary numberings), an
    outage, and optimizer state in and out: follows the oracle, and two calls that
    continue each other equal one bit for bit."""
    rng = np.random.default_rng(48000 + n + numbered)
    if numbered:
        base = synth.config1(B=1, seed=48100 + n, n_bus=n, n_branch=m, n_pv=n // 6)["grid"]
        perm = dpf.rcm_order(n, base.f, base.t, group=256)[0]
        inv = np.empty(n, np.int64)
        inv[perm] = np.arange(n)
        g = synth.Grid(n, inv[base.f].astype(np.int32), inv[base.t].astype(np.int32), base.r, base.x, base.b,
                       base.bus_type[perm], base.vm[perm], base.va[perm])
    else:
        g = random_grid(rng, n, m, 30)
    B, steps = 2, 6
    assert dpf.variants()[dpf.variant_for(n, B)]["kind"] == "wide"
    S = oracle.injections(oracle.ybus_of(g), g.vm, g.va) * 0.98
    vm0 = g.vm[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type == 0)
    va0 = g.va[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type != 2)
    nbr = synth.non_bridge_branches(n, g.f, g.t)
    outage = np.array([-1, nbr[len(nbr) // 3]], np.int32)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)

    def solve(parts):
        vm, va = cu(vm0), cu(va0)
        state, sched = torch.zeros(4, B, n, dtype=torch.float64, device="cuda"), dpf.fresh_sched_state(B, 1e-3)
        for k in parts:
            out = dpf.solve(Yg, g.bus_type, cu(S, torch.complex128), vm, va, outage=cu(outage, torch.int32),
                            adam_state=state, sched_state=sched, opts=dpf.Options(lr=1e-3, tol=0.0, max_iter=k))
            assert out["iters"].tolist() == [k] * B
        return vm, va, state, sched

    vm, va, state, sched = solve([steps])
    for c in range(B):
        ref = oracle.solve_adam(oracle.ybus_of(g, skip=int(outage[c])), g.bus_type, S, vm0[c], va0[c],
                                oracle.AdamOptions(lr=1e-3, tol=0.0, max_iter=steps))
        assert np.abs(vm[c].cpu().numpy() - ref["vm"]).max() < TOL, c
        assert np.abs(va[c].cpu().numpy() - ref["va"]).max() < TOL, c
    for x, y in zip((vm, va, state, sched), solve([2, steps - 2])):
        assert torch.equal(x, y)


@pytest.mark.parametrize("n,n_pv", [(10208, 300), (10100, 1700), (9300, 3700), (4097, 0)])
def test_paired_kernel_with_and_without_room_for_pv_values(dpf, n, n_pv):
    """The paired-state kernel keeps one value per PV row in LDS where it fits behind the
    exchange vector (the largest sub-grid and many PV rows leave no room: the scratch
    takes them): equal to the banded kernel bit for bit, and follows the oracle."""
    rng = np.random.default_rng(49000 + n)
    k = np.arange(1, n)
    f = np.concatenate([k - 1 - rng.integers(0, np.minimum(k, 60)), k[:n // 2]])
    t = np.concatenate([k, np.minimum(k[:n // 2] + rng.integers(2, 80, n // 2), n - 1)])
    f, t = f[f != t].astype(np.int32), t[f != t].astype(np.int32)
    nb = len(f)
    bt = np.zeros(n, np.int8)
    kinds = rng.permutation(n)
    bt[kinds[0]] = 2
    bt[kinds[1:1 + n_pv]] = 1
    va = rng.uniform(-0.1, 0.1, n)
    va[kinds[0]] = 0.0
    g = synth.Grid(n, f, t, rng.uniform(0.01, 0.1, nb), rng.uniform(0.05, 0.3, nb), rng.uniform(0, 0.05, nb), bt,
                   rng.uniform(0.97, 1.03, n), va)
    S = oracle.injections(oracle.ybus_of(g), g.vm, g.va) * 0.98
    vm0, va0 = g.vm[None] * np.ones((3, 1)), g.va[None] + rng.normal(0, 1e-2, (3, n)) * (bt != 2)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    got = {}
    for kind in ("banded-stream", "banded-pair"):
        index = next(v["index"] for v in dpf.variants() if v["kind"] == kind and v["buses_per_thread"] == 4)
        vm, va_ = cu(vm0), cu(va0)
        dpf.solve(Yg, g.bus_type, cu(S, torch.complex128), vm, va_, route=dpf.Route(variant=index),
                  opts=dpf.Options(lr=1e-3, tol=0.0, max_iter=5))
        got[kind] = vm, va_
    assert all(torch.equal(a, b) for a, b in zip(got["banded-stream"], got["banded-pair"]))
    ref = oracle.solve_adam(oracle.ybus_of(g), g.bus_type, S, vm0[1], va0[1],
                            oracle.AdamOptions(lr=1e-3, tol=0.0, max_iter=5))
    assert np.abs(got["banded-pair"][0][1].cpu().numpy() - ref["vm"]).max() < TOL
    assert np.abs(got["banded-pair"][1][1].cpu().numpy() - ref["va"]).max() < TOL


def collection(grids):
    """Grids side by side as the sub-grids of one call: (offsets, branch arrays, bus kinds)."""
    off = np.cumsum([0] + [g.n_bus for g in grids])
    f, t = (np.concatenate([getattr(g, k) + o for g, o in zip(grids, off)]) for k in "ft")
    r, x, b, bt = (np.concatenate([getattr(g, k) for g in grids]) for k in ("r", "x", "b", "bus_type"))
    return off.tolist(), (f, t, r, x, b), bt


def check_mixed_call(dpf, seed, grids, B, steps, team_cap, kind, J):
    """Every item of a call whose sub-grids above ``team_cap`` run on the host-driven
    multi-workgroup path beside a named banded kernel follows the oracle."""
    rng = np.random.default_rng(seed)
    off, branches, bt = collection(grids)
    n = off[-1]
    S = np.concatenate([oracle.injections(oracle.ybus_of(g), g.vm, g.va) for g in grids]) * 0.98
    vm0 = np.concatenate([g.vm for g in grids])[None] + rng.normal(0, 1e-2, (B, n)) * (bt == 0)
    va0 = np.concatenate([g.va for g in grids])[None] + rng.normal(0, 1e-2, (B, n)) * (bt != 2)
    index = next(v["index"] for v in dpf.variants() if v["kind"] == kind and v["buses_per_thread"] == J)
    vm, va = cu(vm0), cu(va0)
    state = torch.zeros(4, B, n, dtype=torch.float64, device="cuda")
    Yg = dpf.build_ybus(n, *branches)
    out = dpf.solve(Yg, bt, cu(S, torch.complex128), vm, va, sub_offset=off, adam_state=state,
                    opts=dpf.Options(lr=1e-3, tol=0.0, max_iter=steps),
                    route=dpf.Route(variant=index, team_cap=team_cap, wide_host=1))
    assert out["iters"].flatten().tolist() == [steps] * (B * len(grids))
    for k, g in enumerate(grids):
        sl = slice(off[k], off[k + 1])
        for c in sorted({0, B - 1}):
            ref = oracle.solve_adam(oracle.ybus_of(g), g.bus_type, S[sl], vm0[c, sl], va0[c, sl],
                                    oracle.AdamOptions(lr=1e-3, tol=0.0, max_iter=steps))
            assert np.abs(vm[c, sl].cpu().numpy() - ref["vm"]).max() < TOL, (k, c)
            assert np.abs(va[c, sl].cpu().numpy() - ref["va"]).max() < TOL, (k, c)
    # every learnable coordinate of every item left its moments
    assert (state[0][:, cu(bt == 0, torch.bool)] != 0).all() and (state[1][:, cu(bt != 2, torch.bool)] != 0).all()


@pytest.mark.parametrize("J", [2, 4])
def test_paired_kernel_beside_the_multi_workgroup_path(dpf, J):
    """The paired kernel's state pairs belong to its own items: the larger sub-grids that
    the multi-workgroup path solves at the same time keep their scratch and their
    results, whichever of the two ends first."""
    rng = np.random.default_rng(50000 + J)
    grids = [random_grid(rng, n, int(1.5 * n)) for n in (900, 400, 700, 60, 300)]
    check_mixed_call(dpf, 50010 + J, grids, 3, 40, 500, "banded-pair", J)


def local_grid(rng, n, n_pv):
    """Random tree plus chords between near buses, in a numbering of bandwidth below 80."""
    k = np.arange(1, n)
    f = np.concatenate([k - 1 - rng.integers(0, np.minimum(k, 60)), k[:n // 2]])
    t = np.concatenate([k, np.minimum(k[:n // 2] + rng.integers(2, 80, n // 2), n - 1)])
    f, t = f[f != t].astype(np.int32), t[f != t].astype(np.int32)
    nb = len(f)
    bt = np.zeros(n, np.int8)
    kinds = rng.permutation(n)
    bt[kinds[0]] = 2
    bt[kinds[1:1 + n_pv]] = 1
    va = rng.uniform(-0.1, 0.1, n)
    va[kinds[0]] = 0.0
    return synth.Grid(n, f, t, rng.uniform(0.01, 0.1, nb), rng.uniform(0.05, 0.3, nb), rng.uniform(0, 0.05, nb), bt,
                      rng.uniform(0.97, 1.03, n), va)


@pytest.mark.parametrize("kind,J,sizes,cap,B,steps", [
    ("banded-stream", 2, ((600, 90), (400, 60), (450, 0), (800, 100)), 500, 3, 60),
    ("banded-stream", 4, ((600, 90), (400, 60)), 500, 2, 60),
    ("banded-pair", 4, ((9800, 1500), (9300, 3700)), 9500, 2, 6)])
def test_banded_items_keep_their_values_apart_from_the_multi_workgroup_path(dpf, kind, J, sizes, cap, B, steps):
    """What the banded kernels keep between their sweeps (the paired one where its LDS has
    no room: 9300 buses with 3700 PV rows) lies in the items' own scratch, beside larger
    sub-grids, listed first and in between, that the multi-workgroup path solves at the
    same time."""
    rng = np.random.default_rng(51000 + J)
    check_mixed_call(dpf, 51010 + J, [local_grid(rng, *s) for s in sizes], B, steps, cap, kind, J)


@pytest.mark.parametrize("path", ["default", "streaming", "banded-stream", "banded-pair", "split", "teams", "wide"])
def test_pv_bus_at_zero_magnitude_stays_finite(dpf, path):
    """A PV bus held at |V| = 0 has an angle that moves nothing: its gradient is zero (no
    0/0), and the other buses follow the oracle on every path."""
    rng = np.random.default_rng(52000)
    n, B, steps = 700, 3, 6
    g = local_grid(rng, n, 90)
    pv = np.flatnonzero(g.bus_type == 1)[40]
    S = oracle.injections(oracle.ybus_of(g), g.vm, g.va) * 0.98
    vm0 = g.vm[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type == 0)
    va0 = g.va[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type != 2)
    vm0[:, pv] = 0.0
    route = {"default": None, "teams": dpf.Route(team_cap=300), "wide": dpf.Route(team_cap=300, wide_host=1)}.get(path)
    if path not in ("default", "teams", "wide"):
        kind = "banded-pair" if path == "split" else path
        route = dpf.Route(variant=next(v["index"] for v in dpf.variants() if v["kind"] == kind))
    if path == "split":  # handed over after 32 iterations
        route.tail_handoff, route.tail_team, steps = B, 8, 36
    vm, va = cu(vm0), cu(va0)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    out = dpf.solve(Yg, g.bus_type, cu(S, torch.complex128), vm, va, route=route,
                    opts=dpf.Options(lr=1e-4, tol=0.0, max_iter=steps))
    assert out["iters"].tolist() == [steps] * B and out["status"].tolist() == [1] * B
    assert (va[:, pv].cpu().numpy() == va0[:, pv]).all()
    ref = oracle.solve_adam(oracle.ybus_of(g), g.bus_type, S, vm0[1], va0[1],
                            oracle.AdamOptions(lr=1e-4, tol=0.0, max_iter=steps))
    assert np.abs(vm[1].cpu().numpy() - ref["vm"]).max() < TOL
    assert np.abs(va[1].cpu().numpy() - ref["va"]).max() < TOL


@pytest.mark.parametrize("top,sizes", [(2048, (65, 64, 512, 513, 1024, 2, 1100)), (1500, (2, 512, 700, 63, 300)),
                                       (900, (129, 512, 40)), (300, (257, 3, 100, 256, 30))])
def test_many_unlike_sub_grids_on_the_register_kernels(dpf, top, sizes):
    """Calls of many sub-grids well below the largest skip the rows a wave has none of: every
    item, from two buses to all rows of every thread, follows the oracle, with optimizer
    state in and out."""
    rng = np.random.default_rng(53000 + top)
    sizes = (top,) + sizes
    B, steps = 514 // len(sizes) + 1, 5  # more items than two per CU of 256
    grids = [random_grid(rng, n, int(1.5 * n) if n > 9 else n - 1) for n in sizes]
    off, branches, bt = collection(grids)
    n = off[-1]
    S = np.concatenate([oracle.injections(oracle.ybus_of(g), g.vm, g.va) for g in grids]) * 0.98
    vm0 = np.concatenate([g.vm for g in grids])[None] + rng.normal(0, 1e-2, (B, n)) * (bt == 0)
    va0 = np.concatenate([g.va for g in grids])[None] + rng.normal(0, 1e-2, (B, n)) * (bt != 2)
    va0[1] += 2.5 * (bt != 2)
    vm, va = cu(vm0), cu(va0)
    state = torch.zeros(4, B, n, dtype=torch.float64, device="cuda")
    sched = dpf.fresh_sched_state(B * len(sizes), 1e-3)
    Yg = dpf.build_ybus(n, *branches)
    for part in (2, steps - 2):
        out = dpf.solve(Yg, bt, cu(S, torch.complex128), vm, va, sub_offset=off, adam_state=state, sched_state=sched,
                        opts=dpf.Options(lr=1e-3, tol=0.0, max_iter=part))
    assert (out["iters"] == steps - 2).all()
    for k, g in enumerate(grids):
        sl = slice(off[k], off[k + 1])
        for c in (0, 1, B - 1):
            ref = oracle.solve_adam(oracle.ybus_of(g), g.bus_type, S[sl], vm0[c, sl], va0[c, sl],
                                    oracle.AdamOptions(lr=1e-3, tol=0.0, max_iter=steps))
            assert np.abs(vm[c, sl].cpu().numpy() - ref["vm"]).max() < TOL, (k, c)
            assert np.abs(va[c, sl].cpu().numpy() - ref["va"]).max() < TOL, (k, c)


def run_both_ways(dpf, g, S, vm0, va0, opts, route, parts):
    """One call and the same iterations in several calls that continue each other through
    the caller's optimizer and schedule state: equal bit for bit; returns the one call's
    (vm, va, schedule, outputs)."""
    B, n = vm0.shape
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    got = []
    for split in ([sum(parts)], parts):
        vm, va = cu(vm0), cu(va0)
        state, sched = torch.zeros(4, B, n, dtype=torch.float64, device="cuda"), dpf.fresh_sched_state(B, opts["lr"])
        for k in split:
            out = dpf.solve(Yg, g.bus_type, cu(S, torch.complex128), vm, va, adam_state=state, sched_state=sched,
                            opts=dpf.Options(**opts, tol=0.0, max_iter=k), route=route)
            assert out["iters"].tolist() == [k] * B
        got.append((vm, va, sched, state, out["max_mis"], out["loss"]))
    assert all(torch.equal(a, b) for a, b in zip(*got))
    return got[0]


@pytest.mark.parametrize("kind,threads,J,n", [("register", 512, 6, 2300), ("register", 512, 8, 3500),
                                              ("streaming", 1024, 0, 3000)])
@pytest.mark.parametrize("opt", ["adam-plateau", "adam-step", "sgd-step", "rmsprop-plateau", "rmsprop"])
def test_named_kernels_above_the_register_sizes(dpf, kind, threads, J, n, opt):
    """The resident kernels and the streaming kernel, named in the route: every optimizer
    and schedule against the oracle, resumed from non-zero moments and schedule state, and
    the stop test at a tolerance the solve reaches."""
    rng = np.random.default_rng(54000 + n)
    g = random_grid(rng, n, int(1.4 * n), 12)
    B = 3
    S = oracle.injections(oracle.ybus_of(g), g.vm, g.va)
    vm0 = g.vm[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type == 0)
    va0 = g.va[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type != 2)
    o = {"adam": dict(lr=1e-3), "sgd": dict(lr=1e-3, beta1=0.9, optimizer=dpf.OPT_SGD),
         "rmsprop": dict(lr=1e-3, beta2=0.99, optimizer=dpf.OPT_RMSPROP)}[opt.split("-")[0]]
    if "plateau" in opt:
        o.update(sched=dpf.SCHED_PLATEAU, factor=0.5, patience=2, threshold=0.3, cooldown=1)
    if "step" in opt:
        o.update(sched=dpf.SCHED_STEP, factor=0.7, patience=3)
    route = dpf.Route(variant=next(v["index"] for v in dpf.variants() if v["kind"] == kind and v["threads"] == threads
                                   and v["buses_per_thread"] == J))
    vm, va, sched, _, mu, _ = run_both_ways(dpf, g, S, vm0, va0, o, route, [5, 4, 5])
    Yo = oracle.ybus_of(g)
    for c in (0, B - 1):
        ref = oracle.solve_adam(Yo, g.bus_type, S, vm0[c], va0[c], oracle.AdamOptions(tol=0.0, max_iter=14, **o))
        assert np.abs(vm[c].cpu().numpy() - ref["vm"]).max() < TOL, c
        assert np.abs(va[c].cpu().numpy() - ref["va"]).max() < TOL, c
        assert sched[c, 1].item() == pytest.approx(ref["lr"], rel=1e-14), c
        assert abs(mu[c].item() - ref["mu"]) <= TOL * ref["mu"], c
    # the first of the steps at which max|r| falls below a bound in the widest gap of its way
    mus = [oracle.solve_adam(Yo, g.bus_type, S, vm0[0], va0[0], oracle.AdamOptions(tol=0.0, max_iter=k, **o))["mu"]
           for k in range(15)]
    low = np.minimum.accumulate(mus)
    k = 1 + int(np.argmax(low[:-1] / low[1:]))
    tol = np.sqrt(low[k - 1] * low[k])
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    vm, va = cu(vm0[:1]), cu(va0[:1])
    out = dpf.solve(Yg, g.bus_type, cu(S, torch.complex128), vm, va, opts=dpf.Options(**o, tol=tol, max_iter=14),
                    route=route)
    ref = oracle.solve_adam(Yo, g.bus_type, S, vm0[0], va0[0], oracle.AdamOptions(tol=tol, max_iter=14, **o))
    assert (out["status"].item(), out["iters"].item()) == (0, k) == (ref["status"], ref["iters"])
    assert np.abs(vm[0].cpu().numpy() - ref["vm"]).max() < TOL and np.abs(va[0].cpu().numpy() - ref["va"]).max() < TOL


@pytest.mark.parametrize("kind", ["banded-stream", "banded-pair"])
@pytest.mark.parametrize("n", [3000, 3500])
def test_wide_band_of_a_named_banded_kernel_runs_the_resident_one(dpf, kind, n):
    """One grid of 2049 to 4096 buses whose bandwidth exceeds the named banded kernel's
    block (a numbering as in its file) runs on a resident kernel of the same call, a*I in
    LDS (3000 buses) or in the scratch the banded kernels lay out (3500), with and without
    the caller's optimizer state."""
    rng = np.random.default_rng(55000 + n)
    g = random_grid(rng, n, int(1.4 * n))
    assert np.abs(g.f - g.t).max() > 2048
    B = 3
    S = oracle.injections(oracle.ybus_of(g), g.vm, g.va)
    vm0 = g.vm[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type == 0)
    va0 = g.va[None] + rng.normal(0, 1e-2, (B, n)) * (g.bus_type != 2)
    route = dpf.Route(variant=next(v["index"] for v in dpf.variants() if v["kind"] == kind and v["buses_per_thread"] == 2))
    vm, va, *_ = run_both_ways(dpf, g, S, vm0, va0, dict(lr=1e-3), route, [4, 5])
    ref = oracle.solve_adam(oracle.ybus_of(g), g.bus_type, S, vm0[2], va0[2],
                            oracle.AdamOptions(lr=1e-3, tol=0.0, max_iter=9))
    assert np.abs(vm[2].cpu().numpy() - ref["vm"]).max() < TOL and np.abs(va[2].cpu().numpy() - ref["va"]).max() < TOL
    vm2, va2 = cu(vm0), cu(va0)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    dpf.solve(Yg, g.bus_type, cu(S, torch.complex128), vm2, va2, opts=dpf.Options(lr=1e-3, tol=0.0, max_iter=9),
              route=route)
    assert torch.equal(vm2, vm) and torch.equal(va2, va)


@pytest.mark.parametrize("kind", ["banded-stream", "banded-pair", "split"])
def test_injections_of_the_librarys_own_evaluation_leave_rounding_residuals(dpf, kind):
    """The paired, banded and split kernels form V conj(I) - S with S inside the chain of
    multiply-adds.  Started where S was evaluated by the library itself, a bus's residual is
    then the rounding of the product, as for injections from anywhere else, and not exactly
    zero at every bus (which changes the optimizer's path)."""
    rng = np.random.default_rng(56000)
    n = 900
    g = local_grid(rng, n, 120)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    vm0, va0 = cu(g.vm[None]), cu(g.va[None])
    zero = torch.zeros(n, dtype=torch.complex128, device="cuda")
    S = dpf.mismatch_grad(Yg, g.bus_type, zero, vm0, va0, want_grad=False)["dS"][0].contiguous()
    variant = next(v["index"] for v in dpf.variants() if v["kind"] == ("banded-pair" if kind == "split" else kind))
    route = dpf.Route(variant=variant)
    mu = dpf.solve(Yg, g.bus_type, S, vm0.clone(), va0.clone(), route=route,
                   opts=dpf.Options(lr=0.0, tol=0.0, max_iter=0))["max_mis"].item()
    if kind == "split":  # lr 0 keeps the start; handed over after 32 iterations
        route.tail_handoff, route.tail_team = 1, 4
        mu = dpf.solve(Yg, g.bus_type, S, vm0.clone(), va0.clone(), route=route,
                       opts=dpf.Options(lr=0.0, tol=0.0, max_iter=40))["max_mis"].item()
    # a product of at most |S| + its share of the row sum rounds by some units of 2^-53
    assert 0.0 < mu <= 64 * 2.0 ** -53 * S.abs().max().item()


def test_strided_and_lazily_conjugated_inputs_are_read_as_their_values(dpf):
    """Bus kinds and outages given as a column of a wider tensor, and injections as a lazy
    conjugate, give what contiguous copies of them give."""
    rng = np.random.default_rng(57000)
    n, B = 200, 4
    g = random_grid(rng, n, 320)
    Yg = dpf.build_ybus(n, g.f, g.t, g.r, g.x, g.b)
    S = cu(oracle.injections(oracle.ybus_of(g), g.vm, g.va) * 0.98, torch.complex128)
    bt = cu(np.stack([g.bus_type, np.roll(g.bus_type, 5)], 1), torch.int8)[:, 0]
    nbr = synth.non_bridge_branches(n, g.f, g.t)
    outage = cu(np.stack([rng.choice(nbr, B), np.full(B, -1)], 1), torch.int32)[:, 0]
    lazy = S.resolve_conj().conj().clone().conj()  # equal to S, its storage conjugated
    assert lazy.is_conj() and not bt.is_contiguous() and not outage.is_contiguous()
    vm, va = cu(np.tile(g.vm, (B, 1))), cu(np.tile(g.va, (B, 1)))

    def run(bt, s, out):
        v, a, d = vm.clone(), va.clone(), torch.zeros_like(va)
        opts = dpf.Options(lr=1e-3, tol=0.0, max_iter=5)
        o = dpf.solve(Yg, bt, s, v, a, outage=out, opts=opts)
        e = dpf.mismatch_grad(Yg, bt, s, vm, va, outage=out)
        p = dpf.param_grad(Yg, bt, s, vm, va, outage=out)
        dpf.dc_init(dpf.build_dc_grid(n, g.f, g.t, g.x), bt, s, d, outage=out)
        t = dpf.solve_series(Yg, bt, s[None].expand(3, n), vm[0], va[0], opts=opts, window=2)
        return [v, a, d, o["loss"], *(e[k] for k in sorted(e)), *(p[k] for k in sorted(p)), t["vm"], t["va"]]

    for x, y in zip(run(bt.clone(memory_format=torch.contiguous_format), S, outage.clone(memory_format=torch.contiguous_format)),
                    run(bt, lazy, outage)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("path", ["default", "streaming", "banded-pair", "wide", "teams", "host", "few-large-host"])
@pytest.mark.parametrize("tol", [0.0, 1e-6])
def test_empty_sub_grids_report_like_any_item(dpf, path, tol):
    """A sub-grid without buses has nothing to learn: every path reports it with a mismatch
    and loss of 0, converged at once, or after every iteration where the tolerance is 0."""
    rng = np.random.default_rng(58000)
    sizes = (2500, 40) if path == "few-large-host" else (300, 40)
    grids = [random_grid(rng, n, int(1.4 * n)) for n in sizes]
    off, branches, bt = collection(grids)
    off = [off[0], off[0], off[1], off[1], off[2], off[2]]
    B, steps, n = 2, 4, off[-1]
    S = np.concatenate([oracle.injections(oracle.ybus_of(g), g.vm, g.va) for g in grids])
    vm0 = np.concatenate([g.vm for g in grids])[None] + rng.normal(0, 1e-2, (B, n)) * (bt == 0)
    va0 = np.tile(np.concatenate([g.va for g in grids]), (B, 1))
    kinds = {v["kind"]: v["index"] for v in dpf.variants()}
    route = {"default": None, "teams": dpf.Route(team_cap=200), "host": dpf.Route(team_cap=200, wide_host=1),
             "few-large-host": dpf.Route(wide_host=1)}.get(path) or dpf.Route(variant=kinds.get(path, -1))
    outs = {k: torch.full((B * 5,), -7, dtype=d, device="cuda") for k, d in
            (("iters", torch.int32), ("status", torch.int32), ("max_mis", torch.float64), ("loss", torch.float64))}
    vm, va = cu(vm0), cu(va0)
    Yg = dpf.build_ybus(n, *branches)
    dpf.solve(Yg, bt, cu(S, torch.complex128), vm, va, sub_offset=off, route=route, outputs=outs,
              opts=dpf.Options(lr=1e-3, tol=tol, max_iter=steps))
    got = {k: outs[k].reshape(B, 5).cpu().numpy() for k in ("iters", "status", "max_mis", "loss")}
    full = [1, 3]
    assert (got["iters"][:, full] == steps).all() and (got["status"][:, full] == 1).all()
    empty = [0, 2, 4]
    assert (got["iters"][:, empty] == (0 if tol > 0 else steps)).all()
    assert (got["status"][:, empty] == (0 if tol > 0 else 1)).all()
    assert (got["max_mis"][:, empty] == 0).all() and (got["loss"][:, empty] == 0).all()
    for k, g in enumerate(grids):
        sl = slice(off[2 * k + 1], off[2 * k + 2])
        ref = oracle.solve_adam(oracle.ybus_of(g), g.bus_type, S[sl], vm0[1, sl], va0[1, sl],
                                oracle.AdamOptions(lr=1e-3, tol=tol, max_iter=steps))
        assert np.abs(vm[1, sl].cpu().numpy() - ref["vm"]).max() < TOL
        assert np.abs(va[1, sl].cpu().numpy() - ref["va"]).max() < TOL
