"""Serving (continuous batching over many systems): each request's result is
the same alone and in a mix, and the server completes a Poisson stream."""
import numpy as np
import pytest

from paper_1909_04667_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _system(spec, precision):
    from paper_1909_04667_amd import binding as B
    from paper_1909_04667_amd import serve as S
    params, stages = S.system_params(spec, precision)
    p = W.system_particles(spec)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=_dev())
    ctx = B.Context(params)
    xyz = (t(p.x), t(p.y), t(p.z))
    ctx.build_tree(*xyz)
    return ctx, xyz, p


def test_batch_alone_equals_mix_equals_single():
    from paper_1909_04667_amd import binding as B
    specs = [W.SystemSpec(0, "plummer", 3000, 1), W.SystemSpec(1, "hernquist", 20000, 2),
             W.SystemSpec(2, "periodic", 16 ** 3, 3), W.SystemSpec(3, "plummer", 70000, 4)]
    precs = ["fp64", "fp32", "fp64", "fp32"]
    systems = [_system(s, pr) for s, pr in zip(specs, precs)]
    rng = np.random.default_rng(0)
    idx = []
    for (ctx, _, p), f in zip(systems, (1.0, 0.3, 0.05, 0.5)):
        sub = rng.choice(p.n, max(1, int(f * p.n)), replace=False).astype(np.int32)
        idx.append(torch.as_tensor(sub, device=_dev()))
    # single-system path
    single = [ctx.compute_forces(ix, "bh")[0].cpu() for (ctx, _, _), ix in zip(systems, idx)]
    # each alone in a batch
    alone = []
    for (ctx, _, _), ix in zip(systems, idx):
        b = B.Batch()
        acc = b.add(ctx, ix, "bh")
        b.launch()
        torch.cuda.synchronize()
        alone.append(acc.cpu())
        b.close()
    # all together in one batch
    b = B.Batch()
    accs = [b.add(ctx, ix, "bh") for (ctx, _, _), ix in zip(systems, idx)]
    b.launch()
    torch.cuda.synchronize()
    for k in range(len(systems)):
        assert torch.equal(alone[k], accs[k].cpu()), k
        assert torch.equal(single[k], accs[k].cpu()), k
    # relative pass in a mix, fed the first pass's |a|
    an = [ctx.accel_norm(ix, a) for (ctx, _, _), ix, a in zip(systems, idx, accs)]
    b2 = B.Batch()
    rel = [b2.add(ctx, ix, "rel", a_old_norm=a) for (ctx, _, _), ix, a in zip(systems, idx, an)]
    b2.launch()
    torch.cuda.synchronize()
    for k, ((ctx, _, _), ix) in enumerate(zip(systems, idx)):
        ref, _ = ctx.compute_forces(ix, "rel", a_old_norm=an[k])
        assert torch.equal(ref.cpu(), rel[k].cpu()), k
    for ctx, _, _ in systems:
        ctx.check()


def test_batch_rejects_same_context_twice():
    from paper_1909_04667_amd import binding as B
    ctx, _, p = _system(W.SystemSpec(0, "plummer", 500, 1), "fp32")
    ix = torch.arange(10, dtype=torch.int32, device=_dev())
    b = B.Batch()
    b.add(ctx, ix, "bh")
    with pytest.raises(B.TreePMError):
        b.add(ctx, ix, "bh")
    b.launch()
    torch.cuda.synchronize()


def _marked_before(n=20000):
    """A context above 8192 particles whose marks hold the value 2 for every
    particle, and the full set's interaction counts."""
    from paper_1909_04667_amd import binding as B
    p = W.uniform_cube(n, 59)
    ctx = B.Context(precision="fp32", eps=0.01, theta=1.5)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=_dev())
    xyz = (t(p.x), t(p.y), t(p.z))
    ctx.build_tree(*xyz)
    idx = torch.arange(n, dtype=torch.int32, device=_dev())
    full = torch.empty(n, dtype=torch.int32, device=_dev())
    for _ in range(2):
        ctx.compute_forces(idx, "bh", n_interactions=full)
    return ctx, xyz, full


def _check_small_set(ctx, full, seed, k=700):
    g = torch.Generator(device=_dev()).manual_seed(seed)
    ids = torch.randperm(full.numel(), generator=g, device=_dev())[:k].to(torch.int32)
    got = torch.full((k,), -1, dtype=torch.int32, device=_dev())
    ctx.compute_forces(ids, "bh", n_interactions=got)
    ctx.check()
    assert torch.equal(got, full[ids.long()])


@pytest.mark.parametrize("calls", [0, 253, 254, 255])
def test_empty_batch_request_keeps_the_marks(calls):
    """An empty batch request queues no clear of the active set's marks: the
    clear that it would have been due (the first call after a build, the call
    after the last of a byte's 255 values) is left to the next call."""
    from paper_1909_04667_amd import binding as B
    ctx, xyz, full = _marked_before()
    none = torch.empty(0, dtype=torch.int32, device=_dev())
    one = torch.zeros(1, dtype=torch.int32, device=_dev())
    every = torch.arange(full.numel(), dtype=torch.int32, device=_dev())
    ctx.build_tree(*xyz)
    for k in range(calls):  # the second one marks every particle with 2
        ctx.compute_forces(every if k == 1 else one, "bh")
    b = B.Batch()
    for _ in range(3):
        b.add(ctx, none, "bh")
        b.launch()
    for k in range(4):
        _check_small_set(ctx, full, k)
    b.close()


def test_failed_submission_keeps_the_marks():
    """A submission that fails (the mesh does not fit the context's arena)
    leaves the clear that it was due to the next call."""
    from paper_1909_04667_amd import binding as B
    n = 20000
    p = W.uniform_cube(n, 61, side=100.0)
    kw = dict(precision="fp32", eps=0.05, theta=1.5, periodic=True, box_size=100.0, pm_grid=256,
              asmth=20.0, rcut=2.0)
    held = B.bytes_needed(B.make_params(precision="fp32", eps=0.05), n)
    ctx = B.Context(arena_bytes=held, **kw)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=_dev())
    xyz = (t(p.x), t(p.y), t(p.z))
    ctx.build_tree(*xyz)
    idx = torch.arange(n, dtype=torch.int32, device=_dev())
    full = torch.empty(n, dtype=torch.int32, device=_dev())
    for _ in range(2):
        ctx.compute_forces(idx, "bh", n_interactions=full)
    ctx.build_tree(*xyz)
    lp = B.ResidentServer("fp32")
    with pytest.raises(B.TreePMError) as ei:
        lp.submit_step(ctx, idx[:1].contiguous())
    assert ei.value.code == B.TPM_ENOMEM
    for k in range(3):
        _check_small_set(ctx, full, k)
    lp.close()


def test_resident_marks_through_their_wrap():
    """More requests than a mark byte has values, on a tree above 8192
    particles: every request selects exactly its own set."""
    from paper_1909_04667_amd import binding as B
    ctx, _, full = _marked_before()
    lp = B.ResidentServer("fp32")
    g = torch.Generator(device=_dev()).manual_seed(3)
    n = full.numel()
    for call in range(300):
        k = (1, 33, 700, n)[call % 4]
        ids = torch.randperm(n, generator=g, device=_dev())[:k].to(torch.int32)
        got = torch.full((k,), -1, dtype=torch.int32, device=_dev())
        torch.cuda.synchronize()
        tk, _ = lp.submit(ctx, ids, "bh", n_interactions=got)
        lp.wait(tk)
        assert torch.equal(got, full[ids.long()]), call
    lp.close()
    ctx.check()


def test_resident_alone_equals_mix_equals_single():
    """Requests for four systems of both precisions submitted together to
    the running kernels (and one at a time): bit-identical to the
    single-system path, BH and relative pass, with interaction counts."""
    from paper_1909_04667_amd import binding as B
    specs = [W.SystemSpec(0, "plummer", 3000, 1), W.SystemSpec(1, "hernquist", 20000, 2),
             W.SystemSpec(2, "periodic", 16 ** 3, 3), W.SystemSpec(3, "plummer", 70000, 4),
             W.SystemSpec(4, "hernquist", 5000, 5), W.SystemSpec(5, "periodic", 20 ** 3, 6)]
    precs = ["fp64", "fp32", "fp64", "fp32", "fp32", "fp32"]
    systems = [_system(s, pr) for s, pr in zip(specs, precs)]
    rng = np.random.default_rng(0)
    idx = []
    for (ctx, _, p), f in zip(systems, (1.0, 0.3, 0.05, 0.5, 0.002, 1.0)):
        sub = rng.choice(p.n, max(1, int(f * p.n)), replace=False).astype(np.int32)
        sub = np.concatenate([sub, sub[:2]])  # duplicates
        idx.append(torch.as_tensor(sub, device=_dev()))
    single, nsingle = [], []
    for (ctx, _, _), ix in zip(systems, idx):
        n = torch.empty(ix.numel(), dtype=torch.int32, device=_dev())
        a, _ = ctx.compute_forces(ix, "bh", n_interactions=n)
        single.append(a.cpu())
        nsingle.append(n.cpu())
    torch.cuda.synchronize()
    loops = {p: B.ResidentServer(p) for p in ("fp32", "fp64")}
    # one at a time
    for k, ((ctx, _, _), ix) in enumerate(zip(systems, idx)):
        lp = loops[precs[k]]
        n = torch.zeros(ix.numel(), dtype=torch.int32, device=_dev())
        t, acc = lp.submit(ctx, ix, "bh", n_interactions=n)
        lp.wait(t)
        assert torch.equal(acc.cpu(), single[k]), k
        assert torch.equal(n.cpu(), nsingle[k]), k
    # all together
    sub = []
    for k, ((ctx, _, _), ix) in enumerate(zip(systems, idx)):
        n = torch.zeros(ix.numel(), dtype=torch.int32, device=_dev())
        t, acc = loops[precs[k]].submit(ctx, ix, "bh", n_interactions=n)
        sub.append((t, acc, n))
    for k, (t, acc, n) in enumerate(sub):
        loops[precs[k]].wait(t)
        assert torch.equal(acc.cpu(), single[k]), k
        assert torch.equal(n.cpu(), nsingle[k]), k
    # relative pass in a mix, fed the first pass's |a|
    an = [ctx.accel_norm(ix, a.to(_dev())) for (ctx, _, _), ix, a in zip(systems, idx, single)]
    torch.cuda.synchronize()
    rel = [loops[precs[k]].submit(ctx, ix, "rel", a_old_norm=an[k])
           for k, ((ctx, _, _), ix) in enumerate(zip(systems, idx))]
    for k, ((ctx, _, _), ix) in enumerate(zip(systems, idx)):
        loops[precs[k]].wait(rel[k][0])
        ref, _ = ctx.compute_forces(ix, "rel", a_old_norm=an[k])
        assert torch.equal(ref.cpu(), rel[k][1].cpu()), k
    for ctx, _, _ in systems:
        ctx.check()
    for lp in loops.values():
        lp.close()


def test_resident_step_equals_single_system_sequence():
    """One step request (geometric pass, mesh force, |a|, relative pass) run
    inside the resident kernel equals the four single-system calls in
    sequence, bit for bit: periodic boxes and isolated systems with and
    without a mesh, both precisions, several at once."""
    from paper_1909_04667_amd import binding as B
    cases = [(W.zeldovich_box(16, 100.0, 31), dict(periodic=True, box_size=100.0, pm_grid=32,
                                                   eps=100.0 / 800), 1.0),
             (W.lognormal_box(16, 100.0, 32), dict(periodic=True, box_size=100.0, pm_grid=64,
                                                   eps=100.0 / 800), 0.3),
             (W.hernquist(1 << 14, 33), dict(eps=0.005), 0.5),
             (W.hernquist(1 << 13, 34), dict(eps=0.005, pm_grid=32), 1.0)]
    for prec in ("fp64", "fp32"):
        lp = B.ResidentServer(prec)
        subs, refs = [], []
        for p, kw, f in cases:
            ctx = B.Context(precision=prec, **kw)
            t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=_dev())
            ctx.build_tree(t(p.x), t(p.y), t(p.z))
            rng = np.random.default_rng(5)
            ids = rng.choice(p.n, max(1, int(f * p.n)), replace=False).astype(np.int32)
            ix = torch.as_tensor(ids, device=_dev())
            a, _ = ctx.compute_forces(ix, "bh")
            apm = ctx.pm_long_range(ix)[0] if kw.get("pm_grid") else None
            an = ctx.accel_norm(ix, a, apm)
            n_ref = torch.empty(ids.size, dtype=torch.int32, device=_dev())
            ar, _ = ctx.compute_forces(ix, "rel", a_old_norm=an, n_interactions=n_ref)
            refs.append((ar.cpu(), None if apm is None else apm.cpu(), n_ref.cpu()))
            torch.cuda.synchronize()
            n = torch.zeros(ids.size, dtype=torch.int32, device=_dev())
            subs.append((ctx, n) + lp.submit_step(ctx, ix, n_interactions=n))
        for (ctx, n, tk, acc, acc_pm), (ar, apm, n_ref) in zip(subs, refs):
            lp.wait(tk)
            ctx.check()
            assert torch.equal(acc.cpu(), ar), prec
            assert (apm is None) == (acc_pm is None)
            if apm is not None:
                assert torch.equal(acc_pm.cpu(), apm), prec
            assert torch.equal(n.cpu(), n_ref), prec
        lp.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("mesh", [0, 16])
def test_resident_adds_the_same_shares(prec, mesh):
    """The resident kernel walks all shares of its targets in one pass, the
    single-system launch each share on its own: the same sums bit for bit, in
    a dense set (shared cursor) and a sparse one (lanes), with a leaf parent
    of 700 particles, larger than the blocks the shares are dealt."""
    from paper_1909_04667_amd import binding as B
    p = W.uniform_cube(30000, 47, side=100.0)
    for v in (p.x, p.y, p.z):
        v[50:750] = 31.0
    kw = dict(periodic=True, box_size=100.0, pm_grid=mesh, rcut=2.0) if mesh else {}
    ctx = B.Context(precision=prec, eps=0.05, alpha=0.02, **kw)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=_dev())
    ctx.build_tree(t(p.x), t(p.y), t(p.z))
    lp = B.ResidentServer(prec)
    an = t(np.full(p.n, 1e-3))
    for k, opening in ((30000, "rel"), (6000, "rel"), (30000, "bh"), (6000, "bh")):
        ids = np.sort(np.random.default_rng(3).choice(p.n, k, replace=False)).astype(np.int32)
        ix = torch.as_tensor(ids, device=_dev())
        n_ref = torch.empty(k, dtype=torch.int32, device=_dev())
        ref, _ = ctx.compute_forces(ix, opening, a_old_norm=an, n_interactions=n_ref)
        torch.cuda.synchronize()
        n = torch.zeros(k, dtype=torch.int32, device=_dev())
        tk, acc = lp.submit(ctx, ix, opening, a_old_norm=an, n_interactions=n)
        lp.wait(tk)
        ctx.check()
        assert torch.equal(acc.cpu(), ref.cpu()), (k, opening)
        assert torch.equal(n.cpu(), n_ref.cpu()), (k, opening)
    lp.close()


@pytest.mark.parametrize("prec", ["fp32", "fp64"])
@pytest.mark.parametrize("n", [65537, 196609, 262145])
def test_shares_in_batch_and_resident(prec, n):
    """Beyond each size where the number of shares changes: batch and resident
    kernel add the shares of the single-system launch, bit for bit -- all
    targets (shared cursor) and a spread-out fifth (lanes)."""
    from paper_1909_04667_amd import binding as B
    p = W.uniform_cube(n, 47, side=100.0)
    for v in (p.x, p.y, p.z):
        v[50:750] = 31.0
    ctx = B.Context(precision=prec, eps=0.05, alpha=0.02, theta=1.0)
    t = lambda a: torch.as_tensor(a, dtype=torch.float64, device=_dev())
    ctx.build_tree(t(p.x), t(p.y), t(p.z))
    lp, batch = B.ResidentServer(prec), B.Batch()
    an = t(np.full(n, 1e-3))
    for k in (n, n // 5):
        ids = np.sort(np.random.default_rng(3).choice(n, k, replace=False)).astype(np.int32)
        ix = torch.as_tensor(ids, device=_dev())
        for opening in ("rel", "bh"):
            c = [torch.empty(k, dtype=torch.int32, device=_dev()) for _ in range(3)]
            ref, _ = ctx.compute_forces(ix, opening, a_old_norm=an, n_interactions=c[0])
            got = batch.add(ctx, ix, opening, a_old_norm=an, n_interactions=c[1])
            batch.launch()
            torch.cuda.synchronize()
            assert torch.equal(got, ref) and torch.equal(c[0], c[1]), (k, opening)
            tk, acc = lp.submit(ctx, ix, opening, a_old_norm=an, n_interactions=c[2])
            lp.wait(tk)
            assert torch.equal(acc, ref) and torch.equal(c[0], c[2]), (k, opening)
    ctx.check()
    lp.close()
    batch.close()


def _threshold_lattice(side=64):
    """2 side^3 particles of a periodic lattice with a basis of two, on
    coordinates without rounding: with every cube opened all particles have
    one |a| up to the rounding of its sums.  alpha puts the relative criterion
    for the cube two sites along x exactly at that |a|, so that last bits of
    |a| decide."""
    s = 1.0 / side
    q = (np.arange(side) + 0.25) * s
    g = np.stack(np.meshgrid(q, q, q, indexing="ij")).reshape(3, -1)
    x = np.concatenate([g, g + np.array([[0.375 * s], [0.0], [0.0]])], axis=1)
    kw = dict(periodic=True, box_size=1.0, pm_grid=side, asmth=1.0, rcut=2.5, theta=0.0,
              eps=0.01 * s, precision="fp64")
    d = (2.0 + 0.1875) * s  # from the first of a basis to the centre of the next but one
    return x, kw, (2.0 / x.shape[1]) * s * s / d ** 4


def test_resident_step_geometric_pass_between_2p18_and_2p19():
    """An FP64 step of 2^19 targets: its geometric pass is summed as
    tpm_compute_forces sums it (undivided at this size, where the relative
    pass is divided), to the last bit of |a| -- opening decisions hang on it
    here -- so the step equals the four calls bit for bit."""
    from paper_1909_04667_amd import binding as B
    x, kw, num = _threshold_lattice()
    n = x.shape[1]
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=_dev())
    xyz = [t(v) for v in x]
    ix = torch.arange(n, dtype=torch.int32, device=_dev())
    ctx = B.Context(**kw)
    ctx.build_tree(*xyz)
    an = ctx.accel_norm(ix, ctx.compute_forces(ix, "bh")[0], ctx.pm_long_range(ix)[0])
    ctx.close()
    ctx = B.Context(alpha=num / float(an[: n // 2].median()), **kw)
    ctx.build_tree(*xyz)
    count = lambda: torch.empty(n, dtype=torch.int32, device=_dev())
    c_ref, c_off, c_step = count(), count(), count()
    pm, _ = ctx.pm_long_range(ix)
    an = ctx.accel_norm(ix, ctx.compute_forces(ix, "bh")[0], pm)
    ref, _ = ctx.compute_forces(ix, "rel", a_old_norm=an, n_interactions=c_ref)
    # the last bit of |a| does decide here
    off = torch.nextafter(an, torch.full_like(an, float("inf")))
    ctx.compute_forces(ix, "rel", a_old_norm=off, n_interactions=c_off)
    assert int((c_ref != c_off).sum()) > 100
    lp = B.ResidentServer("fp64")
    torch.cuda.synchronize()
    tk, acc, acc_pm = lp.submit_step(ctx, ix, n_interactions=c_step)
    lp.wait(tk)
    lp.close()
    ctx.check()
    assert torch.equal(c_step, c_ref)
    assert torch.equal(acc, ref) and torch.equal(acc_pm, pm)


def test_resident_requests_join_the_running_kernel():
    """A large request keeps the kernel busy; requests submitted meanwhile
    are taken up by the same launch, and a context rebuilt meanwhile is
    served correctly (the kernel is drained and launched again first)."""
    from paper_1909_04667_amd import binding as B
    big, _, pb = _system(W.SystemSpec(0, "hernquist", 1 << 19, 7), "fp32")
    small = [_system(W.SystemSpec(k, "plummer", 2000 + 500 * k, 8 + k), "fp32")
             for k in range(1, 5)]
    lp = B.ResidentServer("fp32", idle_ms=200.0)
    ib = torch.arange(pb.n, dtype=torch.int32, device=_dev())
    t0 = lp.info()["launches"]
    tb, ab = lp.submit(big, ib, "bh")
    subs = []
    for ctx, _, p in small:
        ix = torch.arange(p.n, dtype=torch.int32, device=_dev())
        subs.append((ctx, ix) + lp.submit(ctx, ix, "bh"))
    for ctx, ix, t, acc in subs:
        lp.wait(t)
        ref, _ = ctx.compute_forces(ix, "bh")
        assert torch.equal(acc.cpu(), ref.cpu())
    lp.wait(tb)
    assert lp.info()["launches"] - t0 == 1  # all joined the first launch
    ref, _ = big.compute_forces(ib, "bh")
    assert torch.equal(ab.cpu(), ref.cpu())
    # rebuild one small system on moved positions while the kernel runs
    ctx, xyz, p = small[0]
    moved = [v * 1.5 for v in xyz]
    ctx.build_tree(*moved)
    ix = torch.arange(p.n, dtype=torch.int32, device=_dev())
    t, acc = lp.submit(ctx, ix, "bh")
    lp.wait(t)
    ref, _ = ctx.compute_forces(ix, "bh")
    assert torch.equal(acc.cpu(), ref.cpu())
    lp.close()


def test_server_admission_budget_evicts_waits_rejects():
    """A memory budget that holds about two of the systems at a time: the
    stream is served with evictions and waiting, a system that can never fit
    is rejected, and every served result equals the single-system path."""
    from paper_1909_04667_amd import binding as B
    from paper_1909_04667_amd import serve as S
    pool = [W.SystemSpec(0, "plummer", 20000, 21), W.SystemSpec(1, "hernquist", 24000, 22),
            W.SystemSpec(2, "plummer", 16000, 23), W.SystemSpec(3, "hernquist", 1 << 20, 24)]
    need = [B.bytes_needed(S.system_params(sp, "fp32")[0], sp.n) for sp in pool]
    budget = int(max(need[:3]) * 2.2)
    assert need[3] > budget
    reqs = [W.Request(i, 0.0005 * i, i % 4 if i % 7 else 3, 0.3, "fp32", 100 + i)
            for i in range(40)]
    srv = S.Server(pool, budget_bytes=budget)
    stats, jobs = srv.run(reqs)
    s = stats.summary()
    n_rej = sum(1 for r in reqs if r.sid == 3)
    assert s["rejected"] == n_rej and s["requests"] == len(reqs) - n_rej
    assert s["evictions"] > 0 and s["waited_for_memory"] > 0
    assert srv.used <= budget
    for j in jobs:
        if j.rejected:
            continue
        ctx, _, _ = _system(pool[j.req.sid], "fp32")
        a, _ = ctx.compute_forces(j.idx, "bh")
        an = ctx.accel_norm(j.idx, a)
        if pool[j.req.sid].kind == "hernquist":
            a, _ = ctx.compute_forces(j.idx, "rel", a_old_norm=an)
        assert torch.equal(S.total_force(j).cpu(), a.cpu())
        ctx.close()
    srv.close()


def test_server_stream_small():
    from paper_1909_04667_amd import serve as S
    pool = W.system_pool(6, seed=11, log2n=(10, 15))
    reqs = W.request_stream(40, rate=2000.0, n_systems=6, seed=11)
    srv = S.Server(pool, budget_bytes=8 << 30)
    stats, jobs = srv.run(reqs)
    s = stats.summary()
    assert s["requests"] == 40
    assert np.isfinite(s["p99_ms"]) and s["p50_ms"] > 0
    # every served result equals a fresh single-system computation
    for j in jobs[:8]:
        spec = pool[j.req.sid]
        ctx, _, _ = _system(spec, j.req.precision)
        params, stages = S.system_params(spec, j.req.precision)
        a, _ = ctx.compute_forces(j.idx, "bh")
        if spec.kind == "periodic":
            apm, _ = ctx.pm_long_range(j.idx)
        else:
            apm = None
        if len(stages) > 1:
            an = ctx.accel_norm(j.idx, a, apm)
            a, _ = ctx.compute_forces(j.idx, "rel", a_old_norm=an)
        tot = a if apm is None else a + apm
        assert torch.equal(S.total_force(j).cpu(), tot.cpu())
    srv.close()
