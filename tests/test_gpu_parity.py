"""GPU parity: the HIP path through the C ABI against the FP64 CPU oracle.

Bars (Sec. 3.1-3.4 of the paper define what is computed):
  * keys, sort order, tree topology (level, first, count, skip, particle):
    bit-exact;
  * FP64 monopole moments: bit-exact (both sides follow one written operation
    order with explicit fma);
  * FP64 forces: relative error <= 1e-10 per target (floor 1e-3 rms |a|), and
    identical interaction counts (the same opening decisions);
  * FP32 forces: p99 of |a32 - a64| / |a64| <= 1e-3;
  * PM (FP64): deposited density within 1e-13 of max(rho_cell, mean rho)
    (two-plane fixed point against plain FP64 sums), potential mesh within
    1e-12 of its rms, forces at the targets within 1e-10 per target;
  * sampled targets at the full workload sizes.
"""
import math

import numpy as np
import pytest

import oracle as O
from paper_1909_04667_amd import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _t(a, dtype=torch.float64):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=dtype, device=_dev())


def _indiv_eps(n, eps, seed):
    """Individual softening lengths around eps (log-normal spread)."""
    return eps * np.exp(np.random.default_rng(seed).normal(0.0, 0.7, n))


def _ctx(**kw):
    from paper_1909_04667_amd import binding as B
    kw.pop("indiv_eps", None)
    return B.Context(**kw)


def _build(ctx, p, eps=None):
    x, y, z = _t(p.x), _t(p.y), _t(p.z)
    m = None if p.mass is None else _t(p.mass)
    ctx.build_tree(x, y, z, m, eps=None if eps is None else _t(eps))
    return x, y, z, m


def _case_eps(p, kw):
    """The individual softenings a force case asks for (or None)."""
    seed = kw.get("indiv_eps")
    return None if seed is None else _indiv_eps(p.n, kw["eps"], seed)


def rel_err(a, ref, floor_frac=1e-3):
    na = np.linalg.norm(ref, axis=0)
    rms = math.sqrt(float(np.mean(na * na))) if na.size else 1.0
    return np.linalg.norm(a - ref, axis=0) / np.maximum(na, floor_frac * rms)


def _tree_equal(g, T):
    o = T.export()
    for k in ("level", "first", "count", "skip", "pidx"):
        assert np.array_equal(g[k], o[k]), k
    assert np.array_equal(g["mass"], o["mass"]), "moments: mass"
    assert np.array_equal(g["com"], o["com"]), "moments: centre of mass"
    nodes = o["level"] >= 0
    assert np.array_equal(g["cen"][:, nodes], o["cen"][:, nodes]), "node centres"
    assert np.array_equal(g["frame"], T.frame)
    _, _, key = T.positions()
    perm = O.sort(key)
    assert np.array_equal(g["perm"], perm)
    assert np.array_equal(g["key"], key[perm])


def _dup_cloud(n, seed):
    rng = np.random.default_rng(seed)
    x, y, z = rng.normal(0, 1.0, (3, n))
    x[5:9], y[5:9], z[5:9] = x[4], y[4], z[4]          # exact duplicates
    x[20] = x[19] + 1e-13
    y[20], z[20] = y[19], z[19]
    return W.Particles(x, y, z)


CASES = {
    "plummer4096": lambda: (W.plummer(4096, 1), {}),
    "dups3000": lambda: (_dup_cloud(3000, 2), {}),
    "hernquist65536": lambda: (W.hernquist(1 << 16, 2), {}),
    "shifted": lambda: (W.plummer(5000, 3), dict(shift=(0.3, 0.7, 0.1))),
    "masses": lambda: (W.Particles(*np.random.default_rng(4).uniform(-1, 1, (3, 777)),
                                   mass=np.random.default_rng(5).uniform(0.1, 2, 777)), {}),
    "zeldovich16": lambda: (W.zeldovich_box(16, 100.0, 3),
                            dict(periodic=True, box_size=100.0, pm_grid=32)),
    "zeldovich16_shift": lambda: (W.zeldovich_box(16, 100.0, 6),
                                  dict(periodic=True, box_size=100.0, pm_grid=32,
                                       shift=(0.5, 0.25, 0.9))),
    "n1": lambda: (W.Particles(np.array([0.3]), np.array([0.1]), np.array([-0.2])), {}),
    "n2": lambda: (W.Particles(np.array([0.0, 1.0]), np.zeros(2), np.zeros(2)), {}),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_tree_bit_exact(case):
    p, kw = CASES[case]()
    ctx = _ctx(eps=0.01, **kw)
    _build(ctx, p)
    g = ctx.export_tree()
    T = O.Tree(p.x, p.y, p.z, mass=p.mass, periodic=kw.get("periodic", False),
               box=kw.get("box_size", 0.0), shift=kw.get("shift", (0.0, 0.0, 0.0)))
    assert g["level"].size == T.E
    _tree_equal(g, T)


def _pairs(n, seed, gap):
    """n / 2 pairs of particles `gap` apart: a chain of nodes above every pair."""
    rng = np.random.default_rng(seed)
    x, y, z = rng.uniform(-1.0, 1.0, (3, n))
    h = n // 2
    for v in (x, y, z):
        v[h:2 * h] = v[:h] + gap * rng.uniform(-1.0, 1.0, h)
    return W.Particles(x, y, z)


@pytest.mark.parametrize("n,gap", [(63, 0.0), (64, 1e-3), (65, 1e-5), (1023, 1e-4), (1024, 1.0),
                                   (1025, 1e-6), (4095, 1e-6), (8000, 1e-6), (8191, 1.0),
                                   (8192, 1.0), (8193, 1.0), (8193, 1e-6), (10240, 0.0),
                                   (20001, 1e-6), (20480, 1e-3)])
def test_tree_bit_exact_at_the_builds_edges(n, gap):
    """Trees around the sizes where the build changes its kernels: one workgroup
    up to 8192 particles (with more entries than its LDS holds at 8000 and
    1e-6), 256 particles per block beyond (with more entries than a block's
    LDS, 640, where the pairs' chains are long), last blocks full and ragged;
    with masses and individual softening, whose records take the same path;
    the FP32 records by the forces they give."""
    p = _pairs(n, n, gap)
    p.mass = np.random.default_rng(n).uniform(0.5, 2.0, n)
    T = O.Tree(p.x, p.y, p.z, mass=p.mass)
    eps = np.random.default_rng(n + 1).uniform(0.01, 0.05, n)
    res = {}
    idx = _t(np.arange(n), torch.int32)
    for prec, e in (("fp64", None), ("fp64", eps), ("fp32", None)):
        ctx = _ctx(precision=prec, eps=0.03)
        _build(ctx, p, e)
        _tree_equal(ctx.export_tree(), T)
        acc, _ = ctx.compute_forces(idx, "bh")
        ctx.check()
        res[prec, e is None] = acc.double().cpu().numpy()
    err = rel_err(res["fp32", True], res["fp64", True])
    assert np.percentile(err, 99) <= 1e-3, np.percentile(err, [50, 99, 100])


@pytest.mark.parametrize("n", [8193, 10240, 10241, 65536 + 63, 1 << 18, (1 << 18) + 1, 1 << 20,
                               (1 << 20) + 1])
def test_sort_bit_exact_at_the_tiles_edges(n):
    """Keys and stable sort order in tiles of 2048 keys (up to 2^18), 4096 (up to
    2^20) and 8192: full and ragged last tiles, both sides of each change, a
    sixteenth of the particles on one position."""
    rng = np.random.default_rng(n)
    x, y, z = rng.uniform(-50.0, 50.0, (3, n))
    dup = rng.choice(n, n // 16, replace=False)
    x[dup], y[dup], z[dup] = 1.25, -3.5, 7.0
    ctx = _ctx(eps=0.01)
    _build(ctx, W.Particles(x, y, z))
    g = ctx.export_tree()
    _, _, key = O.positions(x, y, z, False, O.frame(x, y, z))
    perm = O.sort(key)
    assert np.array_equal(g["perm"], perm)
    assert np.array_equal(g["key"], key[perm])


def test_sort_many_tiles_bit_exact():
    """Keys and stable sort order at 2^21 + 12345 particles (516 tiles of the
    radix sort), with 6000 copies of one position spread over the whole index
    range so that equal keys cross many tiles: identical to the oracle."""
    n = (1 << 21) + 12345
    rng = np.random.default_rng(21)
    x, y, z = rng.uniform(-50.0, 50.0, (3, n))
    dup = rng.choice(n, 6000, replace=False)
    x[dup], y[dup], z[dup] = 1.25, -3.5, 7.0
    p = W.Particles(x, y, z)
    ctx = _ctx(eps=0.01)
    _build(ctx, p)
    g = ctx.export_tree()
    fr = O.frame(x, y, z)
    assert np.array_equal(g["frame"], fr)
    _, _, key = O.positions(x, y, z, False, fr)
    perm = O.sort(key)
    assert np.array_equal(g["perm"], perm)
    assert np.array_equal(g["key"], key[perm])


def _oracle_params(ctx_kw, opening, eps, theta=0.5, alpha=0.0025, pot=False, frame=None):
    periodic = ctx_kw.get("periodic", False)
    box = ctx_kw.get("box_size", 0.0)
    ng = ctx_kw.get("pm_grid", 0)
    if ng and not periodic:  # isolated mesh over the root cube of the build
        _, rs = O.isolated_scale(frame[3], ng, ctx_kw.get("asmth", 1.25))
    else:
        rs = ctx_kw.get("asmth", 1.25) * box / ng if ng else 0.0
    return O.make_params(periodic=periodic, box=box, eps=eps, opening=opening, theta=theta,
                         alpha=alpha, treepm=ng > 0, rs=rs,
                         rcut=ctx_kw.get("rcut", 4.5) * rs if ng else 0.0, want_pot=pot)


def _pile_box(seed):
    """Zel'dovich box with 150 particles moved onto one point: a cell whose
    150 particles are the children of one cube (more than a wavefront)."""
    p = W.zeldovich_box(16, 100.0, seed)
    x, y, z = p.x.copy(), p.y.copy(), p.z.copy()
    x[:150], y[:150], z[:150] = 37.5, 12.25, 81.0
    return W.Particles(x, y, z)


FORCE_CASES = {
    "plummer_bh": (lambda: W.plummer(4096, 1), dict(eps=0.01, theta=0.5), "bh"),
    "plummer_rel": (lambda: W.plummer(4096, 1), dict(eps=0.01, theta=0.5), "rel"),
    "hernquist_bh": (lambda: W.hernquist(1 << 14, 2), dict(eps=0.005, theta=0.7), "bh"),
    "dups": (lambda: _dup_cloud(2500, 7), dict(eps=0.02, theta=0.6), "bh"),
    "masses_rel": (lambda: W.Particles(*np.random.default_rng(8).uniform(-1, 1, (3, 3000)),
                                       mass=np.random.default_rng(9).uniform(0.1, 2, 3000)),
                   dict(eps=0.01), "rel"),
    "box_bh": (lambda: W.zeldovich_box(16, 100.0, 3),
               dict(eps=100.0 / 800, periodic=True, box_size=100.0, pm_grid=32), "bh"),
    "box_rel_shift": (lambda: W.zeldovich_box(16, 100.0, 4),
                      dict(eps=100.0 / 800, periodic=True, box_size=100.0, pm_grid=32,
                           shift=(0.2, 0.6, 0.95)), "rel"),
    "box_clustered": (lambda: W.lognormal_box(16, 100.0, 5),
                      dict(eps=100.0 / 800, periodic=True, box_size=100.0, pm_grid=64), "bh"),
    "iso_plummer_bh": (lambda: W.plummer(4096, 1), dict(eps=0.01, pm_grid=32), "bh"),
    "iso_hernquist_rel": (lambda: W.hernquist(1 << 13, 4),
                          dict(eps=0.005, pm_grid=64, shift=(0.3, 0.1, 0.8)), "rel"),
    "mixed_plummer_bh": (lambda: W.plummer(4096, 11), dict(eps=0.01, indiv_eps=1), "bh"),
    "mixed_hernquist_rel": (lambda: W.hernquist(1 << 13, 12),
                            dict(eps=0.005, theta=0.6, indiv_eps=2), "rel"),
    "mixed_box_rel": (lambda: W.lognormal_box(16, 100.0, 13),
                      dict(eps=100.0 / 800, periodic=True, box_size=100.0, pm_grid=32,
                           indiv_eps=3), "rel"),
    # r_cut = 35 against a half box of 50: groups wider than 15 walk without
    # the leaf-run prefilter (all of them here, some of them when clustered)
    "box_wide_cutoff": (lambda: W.zeldovich_box(16, 100.0, 14),
                        dict(eps=100.0 / 800, periodic=True, box_size=100.0, pm_grid=16), "bh"),
    "box_clustered_wide_cutoff": (lambda: W.lognormal_box(16, 100.0, 15),
                                  dict(eps=100.0 / 800, periodic=True, box_size=100.0,
                                       pm_grid=16), "rel"),
    "box_pile_bh": (lambda: _pile_box(16),
                    dict(eps=100.0 / 800, periodic=True, box_size=100.0, pm_grid=32), "bh"),
    "box_pile_rel": (lambda: _pile_box(17),
                     dict(eps=100.0 / 800, periodic=True, box_size=100.0, pm_grid=32), "rel"),
}


def _oracle_anorm(p, kw, T):
    P = _oracle_params(kw, "bh", kw["eps"], kw.get("theta", 0.5), frame=T.frame)
    a, _, _ = T.walk(P)
    return np.linalg.norm(a, axis=0)


@pytest.mark.parametrize("case", sorted(FORCE_CASES))
def test_fp64_forces_match_oracle(case):
    mk, kw, opening = FORCE_CASES[case]
    p = mk()
    eps = _case_eps(p, kw)
    ctx = _ctx(want_potential=True, **kw)
    _build(ctx, p, eps)
    T = O.Tree(p.x, p.y, p.z, mass=p.mass, periodic=kw.get("periodic", False),
               box=kw.get("box_size", 0.0), shift=kw.get("shift", (0.0, 0.0, 0.0)), eps=eps)
    an = _oracle_anorm(p, kw, T) if opening == "rel" else None
    # all particles active, in a shuffled caller order with a ragged tail
    order = np.random.default_rng(11).permutation(p.n)[: p.n - 13 if p.n > 100 else p.n]
    idx = _t(order, torch.int32)
    nint = torch.empty(order.size, dtype=torch.int32, device=_dev())
    acc, pot = ctx.compute_forces(idx, opening, a_old_norm=None if an is None else _t(an),
                                  n_interactions=nint)
    ctx.check()
    P = _oracle_params(kw, opening, kw["eps"], kw.get("theta", 0.5), pot=True, frame=T.frame)
    ao, po, no = T.walk(P, targets=order, anorm=an)
    ag = acc.cpu().numpy()
    err = rel_err(ag, ao)
    assert err.max() <= 1e-10, (err.max(), int(err.argmax()))
    assert np.array_equal(nint.cpu().numpy().astype(np.int64), no)
    assert np.abs(pot.cpu().numpy() - po).max() <= 1e-10 * np.abs(po).max()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", sorted(FORCE_CASES))
def test_walk_variants_identical(case, prec, monkeypatch):
    """The shared-cursor walk and the independent-lane walk visit each
    target's entries in the same depth-first order with the same arithmetic:
    accelerations, potentials and interaction counts are bit-identical, on
    the full set and on a sparse subset (ragged last wavefront).  The walk
    with one wavefront per target (64 ranges of the depth-first sequence)
    makes the same interactions, summed in another order."""
    mk, kw, opening = FORCE_CASES[case]
    p = mk()
    eps = _case_eps(p, kw)
    an = None
    if opening == "rel":
        c0 = _ctx(precision="fp64", **kw)
        _build(c0, p, eps)
        a0, _ = c0.compute_forces(_t(np.arange(p.n), torch.int32), "bh")
        an = torch.linalg.norm(a0, dim=0).contiguous()
    sets = [np.arange(p.n), np.random.default_rng(17).choice(p.n, max(1, p.n // 7 + 5),
                                                             replace=False)]
    out = {}
    for mode in ("1", "2", "3"):
        monkeypatch.setenv("TPM_WALK_MODE", mode)
        ctx = _ctx(precision=prec, want_potential=True, **kw)
        _build(ctx, p, eps)
        res = []
        for ids in sets:
            idx = _t(ids, torch.int32)
            nint = torch.empty(ids.size, dtype=torch.int32, device=_dev())
            acc, pot = ctx.compute_forces(idx, opening, a_old_norm=an, n_interactions=nint)
            ctx.check()
            res.append((acc.cpu(), pot.cpu(), nint.cpu()))
        out[mode] = res
    for k in range(len(sets)):
        for a, b in zip(out["1"][k], out["2"][k]):
            assert torch.equal(a, b), (case, prec, k)
        # one wavefront per target: the same interactions (identical counts),
        # partial sums of 64 ranges added in another order
        acc1, pot1, n1 = out["1"][k]
        acc3, pot3, n3 = out["3"][k]
        assert torch.equal(n1, n3), (case, prec, k)
        u = 2.0 ** (-24 if prec == "fp32" else -53)
        mag = acc1.double().norm(dim=0)
        scale = mag.clamp_min(float(mag.square().mean().sqrt()))  # no small-|a| blow-up
        err = (acc3.double() - acc1.double()).norm(dim=0) / scale
        # rounding of two summation orders of at most n_int terms
        assert float(err.max()) <= 64 * u * float(n1.max()), (case, prec, k, float(err.max()))


@pytest.mark.parametrize("case", ["plummer_bh", "plummer_rel", "box_bh", "box_clustered",
                                  "hernquist_bh", "mixed_hernquist_rel", "mixed_box_rel",
                                  "iso_plummer_bh"])
def test_fp32_against_fp64(case):
    mk, kw, opening = FORCE_CASES[case]
    p = mk()
    eps = _case_eps(p, kw)
    res = {}
    an = None
    for prec in ("fp64", "fp32"):
        ctx = _ctx(precision=prec, **kw)
        _build(ctx, p, eps)
        idx = _t(np.arange(p.n), torch.int32)
        if opening == "rel" and an is None:
            c64 = _ctx(precision="fp64", **kw)
            _build(c64, p, eps)
            a0, _ = c64.compute_forces(idx, "bh")
            an = torch.linalg.norm(a0, dim=0).contiguous()
        acc, _ = ctx.compute_forces(idx, opening, a_old_norm=an)
        ctx.check()
        res[prec] = acc.double().cpu().numpy()
    e = rel_err(res["fp32"], res["fp64"])
    assert np.percentile(e, 99) <= 1e-3, np.percentile(e, [50, 99, 100])


def test_active_subsets_and_duplicates():
    """A subset's forces are the full set's at the same targets: bit for bit
    where both take the same walk variant (the lane walk is bit-identical to
    the shared cursor), to rounding where the subset takes one wavefront per
    target (at most 4096 targets in a tree of this size: the same
    interactions summed in another order; interaction counts identical)."""
    p = W.plummer(6000, 12)
    ctx = _ctx(eps=0.01, want_potential=True)
    _build(ctx, p)
    nfull = torch.empty(p.n, dtype=torch.int32, device=_dev())
    full, fpot = ctx.compute_forces(_t(np.arange(p.n), torch.int32), "bh", n_interactions=nfull)
    full = full.cpu().numpy()
    nfull = nfull.cpu().numpy()
    rms = float(np.sqrt(np.mean(np.sum(full * full, axis=0))))
    rng = np.random.default_rng(3)
    for frac in (0.001, 0.05, 0.5, 0.9):
        sub = rng.choice(p.n, max(1, int(frac * p.n)), replace=False)
        sub = np.concatenate([sub, sub[:3]])  # duplicates
        nint = torch.empty(sub.size, dtype=torch.int32, device=_dev())
        acc, _ = ctx.compute_forces(_t(sub, torch.int32), "bh", n_interactions=nint)
        acc = acc.cpu().numpy()
        assert np.array_equal(nint.cpu().numpy(), nfull[sub])
        if sub.size > 4096:
            assert np.array_equal(acc, full[:, sub])
        else:
            assert np.abs(acc - full[:, sub]).max() <= 1e-13 * rms
    # empty active set is a no-op
    acc, _ = ctx.compute_forces(_t(np.zeros(0), torch.int32), "bh")
    assert acc.shape == (3, 0)
    ctx.check()


@pytest.mark.parametrize("n", [8192, 8193, 8192 + 31, 3 * 8192 - 1, 40001])
def test_active_slots_over_many_calls(n):
    """The marks of the active set are bytes that count calls: more calls than a
    byte holds, each with another set (none, one, ragged runs, all), select
    exactly that set -- counts as the full set's at the same targets, in the
    caller's order."""
    p = W.uniform_cube(n, 53)
    ctx = _ctx(precision="fp32", eps=0.01, theta=1.5)
    _build(ctx, p)
    full = torch.empty(n, dtype=torch.int32, device=_dev())
    ctx.compute_forces(_t(np.arange(n), torch.int32), "bh", n_interactions=full)
    g = torch.Generator(device=_dev()).manual_seed(7)
    for call in range(530):
        k = (1, 2, 33, 700, n)[call % 5]
        ids = torch.randperm(n, generator=g, device=_dev())[:k].to(torch.int32)
        got = torch.full((k,), -1, dtype=torch.int32, device=_dev())
        ctx.compute_forces(ids, "bh", n_interactions=got)
        assert torch.equal(got, full[ids.long()]), call
    ctx.check()


@pytest.mark.parametrize("n", [1, 512, 8192])
@pytest.mark.parametrize("m", [16384, 16385, 70001])
def test_active_lists_of_many_duplicates(n, m):
    """Lists longer than the tree, around the length where the selection of
    small trees changes its kernels: every entry gets its particle's result
    and count, out-of-range entries NaN, and the flag is set."""
    from paper_1909_04667_amd import binding as B
    p = W.uniform_cube(n, 67)
    ctx = _ctx(precision="fp32", eps=0.01, theta=1.0)
    _build(ctx, p)
    nfull = torch.empty(n, dtype=torch.int32, device=_dev())
    full, _ = ctx.compute_forces(_t(np.arange(n), torch.int32), "bh", n_interactions=nfull)
    ids = torch.randint(0, n, (m,), dtype=torch.int32, device=_dev(),
                        generator=torch.Generator(device=_dev()).manual_seed(m))
    for bad in (False, True):
        if bad:
            ids[m // 2], ids[m - 1] = n, -1
        got = torch.zeros(m, dtype=torch.int32, device=_dev())
        acc, _ = ctx.compute_forces(ids, "bh", n_interactions=got)
        ok = (ids >= 0) & (ids < n)
        sel = ids[ok].long()
        assert torch.equal(got[ok], nfull[sel])
        assert bool(torch.isnan(acc[:, ~ok]).all())
        assert torch.equal(acc[:, ok], full[:, sel])
    with pytest.raises(B.TreePMError) as ei:
        ctx.check()
    assert ei.value.code == B.TPM_EINDEX


@pytest.mark.parametrize("n", [4097, 65536, 65537, 196609, 262145, 524288, 524289])
@pytest.mark.parametrize("mesh", [0, 16])
def test_shares_of_a_walk(n, mesh, monkeypatch):
    """Walks of small sets are divided into shares, eight to one at these
    sizes: the shared cursor and the lanes add the same shares (bit for bit),
    and no interaction is lost or done twice (counts of the undivided walk,
    one wavefront per target).  700 particles share a place, so that a leaf
    parent is larger than the blocks the shares are dealt."""
    p = W.uniform_cube(n, 43, side=100.0)
    for v in (p.x, p.y, p.z):
        v[50:750] = 31.0
    kw = dict(precision="fp32", eps=0.05, alpha=0.02, want_potential=True)
    if mesh:
        kw.update(periodic=True, box_size=100.0, pm_grid=mesh, rcut=2.0)
    out = []
    for mode in ("1", "2", "3"):
        monkeypatch.setenv("TPM_WALK_MODE", mode)
        ctx = _ctx(**kw)
        _build(ctx, p)
        nint = torch.full((n,), -1, dtype=torch.int32, device=_dev())
        acc, pot = ctx.compute_forces(_t(np.arange(n), torch.int32), "rel", n_interactions=nint,
                                      a_old_norm=_t(np.full(n, 1e-3)))
        ctx.check()
        out.append((acc, pot, nint))
    for a, b in zip(out[0], out[1]):
        assert torch.equal(a, b)
    assert torch.equal(out[0][2], out[2][2])
    mag = out[0][0].double().norm(dim=0)
    scale = mag.clamp_min(float(mag.square().mean().sqrt()))
    err = (out[2][0].double() - out[0][0].double()).norm(dim=0) / scale
    # rounding of two summation orders of at most n_int terms
    assert float(err.max()) <= 64 * 2.0 ** -24 * float(out[0][2].max())


@pytest.mark.parametrize("n", [20000, 196608, 196609, 262144, 262145, 524288, 524289])
@pytest.mark.parametrize("mesh", [0, 16])
def test_shares_of_a_walk_fp64(n, mesh, monkeypatch):
    """The same in FP64, around the sizes where its number of shares changes
    (the relative pass is divided in two up to 524288, the geometric one up to
    262144), with potentials: a group's shares are added in one workgroup, a
    target's in neighbouring lanes."""
    p = W.uniform_cube(n, 43, side=100.0)
    for v in (p.x, p.y, p.z):
        v[50:750] = 31.0
    kw = dict(precision="fp64", eps=0.05, alpha=0.02, theta=1.0, want_potential=True)
    if mesh:
        kw.update(periodic=True, box_size=100.0, pm_grid=mesh, rcut=0.5)
    for opening in ("bh", "rel"):
        out = []
        for mode in ("1", "2", "3"):
            monkeypatch.setenv("TPM_WALK_MODE", mode)
            ctx = _ctx(**kw)
            _build(ctx, p)
            nint = torch.full((n,), -1, dtype=torch.int32, device=_dev())
            acc, pot = ctx.compute_forces(_t(np.arange(n), torch.int32), opening,
                                          n_interactions=nint, a_old_norm=_t(np.full(n, 1e-3)))
            ctx.check()
            out.append((acc, pot, nint))
        for a, b in zip(out[0], out[1]):
            assert torch.equal(a, b)
        assert torch.equal(out[0][2], out[2][2])
        for k in (0, 1):
            a, b = (out[q][k].reshape(-1, n) for q in (0, 2))
            mag = a.norm(dim=0)
            scale = mag.clamp_min(float(mag.square().mean().sqrt()))
            # rounding of two summation orders of at most n_int terms
            bound = 64 * 2.0 ** -53 * float(out[0][2].max())
            assert float(((a - b).norm(dim=0) / scale).max()) <= bound


@pytest.mark.parametrize("n", [4097, 16383, 16384, 16385])
@pytest.mark.parametrize("periodic", [False, True])
def test_wavefront_per_target_with_a_cutoff(n, periodic, monkeypatch):
    """FP64 with a mesh takes one wavefront per target up to 16384 targets: the
    interactions of the shared cursor, summed in another order; the walk that
    runs by default is that one up to there, and not beyond."""
    p = W.uniform_cube(n, 47, side=100.0)
    for v in (p.x, p.y, p.z):
        v[50:750] = 31.0
    kw = dict(precision="fp64", eps=0.05, alpha=0.02, want_potential=True, pm_grid=16, rcut=2.0,
              periodic=periodic)
    if periodic:
        kw["box_size"] = 100.0
    for opening in ("bh", "rel"):
        out = []
        for mode in ("0", "1", "3"):
            monkeypatch.setenv("TPM_WALK_MODE", mode)
            ctx = _ctx(**kw)
            _build(ctx, p)
            nint = torch.full((n,), -1, dtype=torch.int32, device=_dev())
            acc, pot = ctx.compute_forces(_t(np.arange(n), torch.int32), opening,
                                          n_interactions=nint,
                                          a_old_norm=_t(np.full(n, 1e-3)))
            ctx.check()
            out.append((acc, pot, nint))
        for a, b in zip(out[0], out[2 if n <= 16384 else 1]):
            assert torch.equal(a, b)
        assert torch.equal(out[1][2], out[2][2])
        mag = out[1][0].norm(dim=0)
        scale = mag.clamp_min(float(mag.square().mean().sqrt()))
        err = (out[2][0] - out[1][0]).norm(dim=0) / scale
        # rounding of two summation orders of at most n_int terms
        assert float(err.max()) <= 64 * 2.0 ** -53 * float(out[1][2].max())


@pytest.mark.parametrize("n", [255 * 64, 64 * 256 + 1, 8192 * 256 - 63, 8305 * 256 - 1])
def test_block_order_covers_every_group(n, monkeypatch):
    """The blocks of a walk are dealt to the dies in runs of a length that
    follows from their number: every group of 64 targets is walked once,
    whatever number of blocks the runs leave over.  The shared cursor against
    the independent lanes (another launch geometry), bit for bit."""
    p = W.uniform_cube(n, 41)
    out = []
    for mode in ("1", "2"):
        monkeypatch.setenv("TPM_WALK_MODE", mode)
        ctx = _ctx(precision="fp32", eps=0.01, theta=1.5)
        _build(ctx, p)
        nint = torch.full((n,), -1, dtype=torch.int32, device=_dev())
        acc = torch.full((3, n), float("nan"), dtype=torch.float32, device=_dev())
        ctx.compute_forces(_t(np.arange(n), torch.int32), "bh", acc=acc, n_interactions=nint)
        ctx.check()
        out.append((acc, nint))
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_sparse_sets_group_or_lanes_identical(prec):
    """Sparse active sets with a cutoff take the shared cursor or independent
    lanes as a census of their groups' extents decides on the device: the two
    give the same results, so every subset equals the full set at its targets
    bit for bit -- a compact set (a slab), a spread-out one (random) and
    their union."""
    p = W.zeldovich_box(40, box=100.0, seed=23)  # 64000 particles
    kw = dict(precision=prec, periodic=True, box_size=100.0, pm_grid=64, eps=0.05)
    ctx = _ctx(**kw)
    _build(ctx, p)
    nfull = torch.empty(p.n, dtype=torch.int32, device=_dev())
    full, _ = ctx.compute_forces(_t(np.arange(p.n), torch.int32), "bh", n_interactions=nfull)
    full, nfull = full.cpu(), nfull.cpu()
    slab = np.argsort(p.x, kind="stable")[:6000]
    rand = np.random.default_rng(29).choice(p.n, 6000, replace=False)
    both = np.union1d(slab, rand)
    for sub in (slab, rand, both):
        assert 4096 < sub.size and 4 * sub.size < p.n  # the per-group choice
        nint = torch.empty(sub.size, dtype=torch.int32, device=_dev())
        acc, _ = ctx.compute_forces(_t(sub, torch.int32), "bh", n_interactions=nint)
        ctx.check()
        assert torch.equal(nint.cpu(), nfull[sub])
        assert torch.equal(acc.cpu(), full[:, sub])


@pytest.mark.parametrize("k", [4097, 33333, 33334, 49152, 49153, 98304, 98305])
@pytest.mark.parametrize("prec,mesh", [("fp64", 0), ("fp64", 32), ("fp32", 32)])
def test_sparse_sets_of_an_isolated_system(prec, mesh, k, monkeypatch):
    """Sparse sets of an isolated system: shared cursor or lanes by the census
    (spread sets and compact ones), lanes in the FP64 geometric pass with a
    mesh beyond 49152 targets, four, two shares or one there.  Whatever is
    taken, the shared cursor and the lanes give it bit for bit, and no
    interaction is lost (counts of one wavefront per target)."""
    p = W.hernquist(400000, 31)
    n = p.n
    r = p.x ** 2 + p.y ** 2 + p.z ** 2
    near = np.sort(np.argsort(r, kind="stable")[:k])
    rand = np.sort(np.random.default_rng(k).choice(n, k, replace=False))
    kw = dict(precision=prec, eps=0.02, theta=0.8)
    if mesh:
        kw.update(pm_grid=mesh, rcut=1.5)
    ctxs = []
    for mode in ("0", "1", "2", "3"):
        monkeypatch.setenv("TPM_WALK_MODE", mode)
        ctxs.append(_ctx(**kw))
        _build(ctxs[-1], p)
    an = _t(np.full(n, 1.0))
    for sub in (near, rand):
        for opening in ("bh", "rel"):
            out = []
            for ctx in ctxs:
                nint = torch.empty(k, dtype=torch.int32, device=_dev())
                acc, _ = ctx.compute_forces(_t(sub, torch.int32), opening, a_old_norm=an,
                                            n_interactions=nint)
                ctx.check()
                out.append((acc, nint))
            for acc, nint in out[1:3]:
                assert torch.equal(acc, out[0][0])
            for acc, nint in out[1:]:
                assert torch.equal(nint, out[0][1])


def test_out_of_range_index_reported():
    from paper_1909_04667_amd import binding as B
    p = W.plummer(500, 13)
    ctx = _ctx(eps=0.01)
    _build(ctx, p)
    acc, _ = ctx.compute_forces(_t(np.array([3, 500, -1, 7]), torch.int32), "bh")
    a = acc.cpu().numpy()
    assert np.all(np.isnan(a[:, 1])) and np.all(np.isnan(a[:, 2]))
    assert np.all(np.isfinite(a[:, 0])) and np.all(np.isfinite(a[:, 3]))
    with pytest.raises(B.TreePMError) as ei:
        ctx.check()
    assert ei.value.code == B.TPM_EINDEX
    ctx.check()  # the flag is cleared


def test_single_particle_and_determinism():
    p = W.Particles(np.array([0.3]), np.array([0.1]), np.array([-0.2]))
    ctx = _ctx(eps=0.01)
    _build(ctx, p)
    acc, _ = ctx.compute_forces(_t(np.array([0]), torch.int32), "bh")
    assert np.array_equal(acc.cpu().numpy(), np.zeros((3, 1)))
    q = W.hernquist(20000, 21)
    outs = []
    for _ in range(2):
        c = _ctx(eps=0.005)
        _build(c, q)
        a, _ = c.compute_forces(_t(np.arange(q.n), torch.int32), "bh")
        outs.append(a.cpu().numpy())
    assert np.array_equal(outs[0], outs[1])


def fp32_mesh_bounds(ng3, h, a_ref, pot_ref):
    """Absolute error bounds of the FP32 mesh, from the FFT error model: the
    unit roundoff u = 2^-24 grows with the log2(ng^3) butterfly levels of the
    forward and inverse transforms, so the potential carries errors of order
    u log2(ng^3) rms(Phi); the four-point difference turns them into force
    errors of order u log2(ng^3) rms(Phi) / h, i.e. u log2(ng^3) kappa
    rms|a| with kappa = rms(Phi) / (h rms|a|) (the reference's potential and
    force at the targets); the float storage of the density and potential
    adds a term of order u kappa rms|a| that does not grow with the mesh.
    Bounds: force u (2 log2(ng^3) + 32) kappa rms|a|, potential
    8 u log2(ng^3) rms(Phi).  Measured: force errors up to 0.75 u log2(ng^3)
    kappa rms|a| on near-uniform and clustered boxes with meshes of 16^3 to
    256^3, and 34 u kappa rms|a| on the 8^3 mesh."""
    u = 2.0 ** -24
    lg = math.log2(ng3)
    rms_a = math.sqrt(float(np.mean(np.sum(a_ref * a_ref, axis=0))))
    rms_p = math.sqrt(float(np.mean(pot_ref * pot_ref)))
    kappa = rms_p / (h * rms_a)
    return u * (2.0 * lg + 32.0) * kappa * rms_a, 8.0 * u * lg * rms_p


def _check_fp32_mesh(a, pot, a_ref, pot_ref, ng3, h):
    fb, pb = fp32_mesh_bounds(ng3, h, a_ref, pot_ref)
    da = np.linalg.norm(a - a_ref, axis=0).max()
    assert da <= fb, (ng3, da, fb)
    if pot is not None:
        dp = np.abs(pot - pot_ref).max()
        assert dp <= pb, (ng3, dp, pb)


def _mesh_check(ctx, p, box, ng, rs, prec, tol_rho=1e-13):
    """Deposited density cell by cell and the potential mesh against the
    oracle's FP64 deposit and mesh solve."""
    rho_g, phi_g = ctx.export_mesh()
    rho_o = O.cic_deposit(p.x, p.y, p.z, p.mass, box, ng)
    rbar = rho_o.mean()
    d = np.abs(rho_g - rho_o) / np.maximum(rho_o, rbar)
    if prec == "fp64":
        assert d.max() <= tol_rho, (ng, d.max())
    else:  # one 64-bit word: 2^-62 of the total mass per contribution
        assert d.max() <= 1e-9, (ng, d.max())
    phi_o, _, _, _ = O.pm_mesh(rho_o, box, 1.0, rs)
    rms = math.sqrt(float(np.mean(phi_o * phi_o)))
    dphi = np.abs(phi_g - phi_o).max() / rms
    if prec == "fp64":
        assert dphi <= 1e-12, (ng, dphi)
    else:  # the potential bound of fp32_mesh_bounds
        assert dphi <= 8.0 * 2.0 ** -24 * math.log2(ng ** 3), (ng, dphi)
    return d.max(), dphi


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_pm_mesh_matches_oracle(prec):
    """The deposited density and the potential of the mesh solve, cell by
    cell, on a near-uniform and a clustered box."""
    for p, ng in ((W.zeldovich_box(32, 100.0, 3), 64), (W.lognormal_box(32, 100.0, 5), 128),
                  (W.zeldovich_box(16, 100.0, 7), 32)):
        ctx = _ctx(eps=0.1, periodic=True, box_size=100.0, pm_grid=ng, precision=prec)
        _build(ctx, p)
        _mesh_check(ctx, p, 100.0, ng, 1.25 * 100.0 / ng, prec)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_pm_matches_oracle(prec):
    p = W.zeldovich_box(16, 100.0, 3)
    # every line decomposition of the FFT up to 128 (8 = 4 x 2 ... 128 = 16 x 8)
    for ng, asmth in ((8, 0.5), (16, 1.25), (32, 1.25), (64, 1.25), (128, 1.25)):
        ctx = _ctx(eps=0.1, periodic=True, box_size=100.0, pm_grid=ng, precision=prec,
                   want_potential=True, asmth=asmth)
        _build(ctx, p)
        order = np.random.default_rng(1).permutation(p.n)
        acc, pot = ctx.pm_long_range(_t(order, torch.int32))
        ctx.check()
        ao, po = O.pm(p.x, p.y, p.z, None, 100.0, ng, 1.0, asmth * 100.0 / ng, targets=order)
        ag, pg = acc.double().cpu().numpy(), pot.double().cpu().numpy()
        if prec == "fp64":
            e = rel_err(ag, ao)
            assert e.max() <= 1e-10, (ng, e.max())
            assert np.percentile(e, 99) <= 1e-12, (ng, np.percentile(e, 99))
            assert np.abs(pg - po).max() <= 1e-12 * np.abs(po).max()
        else:
            _check_fp32_mesh(ag, pg, ao, po, ng ** 3, 100.0 / ng)


def test_pm_momentum_on_gpu():
    p = W.lognormal_box(32, 100.0, 8)
    ctx = _ctx(eps=0.1, periodic=True, box_size=100.0, pm_grid=64)
    _build(ctx, p)
    acc, _ = ctx.pm_long_range(_t(np.arange(p.n), torch.int32))
    a = acc.cpu().numpy()
    m = 1.0 / p.n
    assert np.abs((m * a).sum(axis=1)).max() / (m * np.linalg.norm(a, axis=0)).sum() < 1e-10


# ---- full workload sizes, sampled targets -----------------------------------

@pytest.mark.slow
def test_full_hernquist_2p20_sampled():
    """Workload 2 at N = 2^20: topology bit-exact, BH then relative forces
    bit-compatible on 2048 sampled targets, FP32 within 1e-3, tree within 1 %."""
    p = W.hernquist(1 << 20, 2)
    kw = dict(eps=0.005, theta=0.5, alpha=0.0025)
    T = O.Tree(p.x, p.y, p.z)
    ctx = _ctx(**kw)
    _build(ctx, p)
    g = ctx.export_tree()
    _tree_equal(g, T)
    idx_all = _t(np.arange(p.n), torch.int32)
    a_bh, _ = ctx.compute_forces(idx_all, "bh")
    an = torch.linalg.norm(a_bh, dim=0).contiguous()
    a_rel, _ = ctx.compute_forces(idx_all, "rel", a_old_norm=an)
    samp = np.sort(np.random.default_rng(0).choice(p.n, 2048, replace=False))
    P = _oracle_params({}, "bh", 0.005)
    ao, _, _ = T.walk(P, targets=samp)
    assert rel_err(a_bh.cpu().numpy()[:, samp], ao).max() <= 1e-10
    # relative pass on the sampled targets, both sides fed the oracle's |a|
    an_o = np.zeros(p.n)
    an_o[samp] = np.linalg.norm(ao, axis=0)
    a_rs, _ = ctx.compute_forces(_t(samp, torch.int32), "rel", a_old_norm=_t(an_o))
    Pr = _oracle_params({}, "rel", 0.005)
    ar, _, _ = T.walk(Pr, targets=samp, anorm=an_o)
    assert rel_err(a_rs.cpu().numpy(), ar).max() <= 1e-10
    ad, _ = O.direct(p.x, p.y, p.z, None, P, targets=samp)
    assert np.percentile(rel_err(a_rel.cpu().numpy()[:, samp], ad), 99) <= 0.01
    c32 = _ctx(precision="fp32", **kw)
    _build(c32, p)
    a32, _ = c32.compute_forces(idx_all, "rel", a_old_norm=an)
    e = rel_err(a32.double().cpu().numpy(), a_rel.cpu().numpy())
    assert np.percentile(e, 99) <= 1e-3


def _progress(msg):
    """A line per finished stage of the long full-size tests (visible with -s)."""
    import sys
    print(f"  [{msg}]", file=sys.stderr, flush=True)


def _truncated_direct(p, kw, targets):
    """The exact short-range reference: nearest-image pair sum with the
    spline softening, the short-range factor and the cutoff."""
    P = _oracle_params(kw, "bh", kw["eps"])
    ad, _ = O.direct(p.x, p.y, p.z, None, P, targets=targets)
    return ad


@pytest.mark.slow
@pytest.mark.timeout(600)
def test_full_zeldovich_128_pm256_sampled():
    """Workload 3 at full size (128^3 particles, 256^3 mesh), FP64: tree and
    moments bit-exact; deposited density and potential cell by cell; the
    geometric pass, the mesh force and the relative pass (both sides fed the
    oracle's |a| of geometric + mesh force) at 1024 sampled targets within
    1e-10 with identical interaction counts; the relative pass's short-range
    force within p99 1 % of the exact truncated pair sum on 256 of them."""
    p = W.zeldovich_box(128, 100.0, 3)
    kw = dict(eps=100.0 / 6400, periodic=True, box_size=100.0, pm_grid=256)
    rs = 1.25 * 100.0 / 256
    ctx = _ctx(**kw)
    _build(ctx, p)
    T = O.Tree(p.x, p.y, p.z, periodic=True, box=100.0)
    _tree_equal(ctx.export_tree(), T)
    _progress("tree and moments bit-exact")
    _mesh_check(ctx, p, 100.0, 256, rs, "fp64")
    _progress("mesh density and potential")
    samp = np.sort(np.random.default_rng(1).choice(p.n, 1024, replace=False))
    idx = _t(samp, torch.int32)
    nint = torch.empty(samp.size, dtype=torch.int32, device=_dev())
    acc, _ = ctx.compute_forces(idx, "bh", n_interactions=nint)
    ao, _, no = T.walk(_oracle_params(kw, "bh", kw["eps"]), targets=samp)
    assert rel_err(acc.cpu().numpy(), ao).max() <= 1e-10
    assert np.array_equal(nint.cpu().numpy().astype(np.int64), no)
    apm, _ = ctx.pm_long_range(idx)
    apo, _ = O.pm(p.x, p.y, p.z, None, 100.0, 256, 1.0, rs, targets=samp, want_pot=False)
    assert rel_err(apm.cpu().numpy(), apo).max() <= 1e-10
    an = np.zeros(p.n)
    an[samp] = np.linalg.norm(ao + apo, axis=0)
    ag, _ = ctx.compute_forces(idx, "rel", a_old_norm=_t(an), n_interactions=nint)
    ctx.check()
    ar, _, nr = T.walk(_oracle_params(kw, "rel", kw["eps"]), targets=samp, anorm=an)
    assert rel_err(ag.cpu().numpy(), ar).max() <= 1e-10
    assert np.array_equal(nint.cpu().numpy().astype(np.int64), nr)
    ad = _truncated_direct(p, kw, samp[:256])
    assert np.percentile(rel_err(ar[:, :256], ad), 99) <= 0.01


@pytest.mark.slow
@pytest.mark.timeout(600)
def test_full_zeldovich_fp32_against_fp64_full_step():
    """Workload 3 at full size: the whole step (build, mesh, geometric pass,
    |a|, relative pass) in FP32 and in FP64 on all 2,097,152 targets, each
    with its own |a|: the FP32 total force (tree + mesh) within p99 1e-3 of
    the FP64 one, and the FP32 mesh force within the FP32 mesh bound."""
    p = W.zeldovich_box(128, 100.0, 3)
    kw = dict(eps=100.0 / 6400, periodic=True, box_size=100.0, pm_grid=256)
    ao, po = O.pm(p.x, p.y, p.z, None, 100.0, 256, 1.0, 1.25 * 100.0 / 256)
    _progress("oracle mesh force")
    res = {}
    for prec in ("fp64", "fp32"):
        ctx = _ctx(precision=prec, **kw)
        _build(ctx, p)
        idx = _t(np.arange(p.n), torch.int32)
        apm, ppm = ctx.pm_long_range(idx, want_pot=True)
        abh, _ = ctx.compute_forces(idx, "bh")
        an = ctx.accel_norm(idx, abh, apm)
        arel, _ = ctx.compute_forces(idx, "rel", a_old_norm=an)
        ctx.check()
        res[prec] = ((arel.double() + apm.double()).cpu().numpy(), apm.double().cpu().numpy(),
                     ppm.double().cpu().numpy())
        ctx.close()
        _progress(f"{prec} full step")
    e = rel_err(res["fp32"][0], res["fp64"][0])
    assert np.percentile(e, 99) <= 1e-3, np.percentile(e, [50, 99, 100])
    assert rel_err(res["fp64"][1], ao).max() <= 1e-10
    _check_fp32_mesh(res["fp32"][1], res["fp32"][2], ao, po, 256 ** 3, 100.0 / 256)


@pytest.mark.parametrize("frac", [0.001, 0.01, 0.1])
def test_clustered_time_bin_subsets(frac):
    """Workload 4 at 32^3: the tree is built once and reused for nested
    time-bin active sets; relative pass fed the oracle's own |a|."""
    p = W.lognormal_box(32, 100.0, 4)
    sets, _ = W.time_bin_active_sets(p.meta["rho"])
    sub = sets[frac]
    kw = dict(eps=100.0 / (50 * 32), periodic=True, box_size=100.0, pm_grid=64)
    T = O.Tree(p.x, p.y, p.z, periodic=True, box=100.0)
    Pb = _oracle_params(kw, "bh", kw["eps"])
    ab, _, _ = T.walk(Pb, targets=sub)
    apm, _ = O.pm(p.x, p.y, p.z, None, 100.0, 64, 1.0, 1.25 * 100.0 / 64, targets=sub)
    an = np.zeros(p.n)
    an[sub] = np.linalg.norm(ab + apm, axis=0)
    Pr = _oracle_params(kw, "rel", kw["eps"])
    ar, _, nr = T.walk(Pr, targets=sub, anorm=an)
    for prec in ("fp64", "fp32"):
        ctx = _ctx(precision=prec, **kw)
        _build(ctx, p)
        idx = _t(sub, torch.int32)
        nint = torch.empty(sub.size, dtype=torch.int32, device=_dev())
        acc, _ = ctx.compute_forces(idx, "rel", a_old_norm=_t(an), n_interactions=nint)
        g_pm, _ = ctx.pm_long_range(idx)
        ctx.check()
        e = rel_err(acc.double().cpu().numpy(), ar)
        if prec == "fp64":
            assert e.max() <= 1e-10
            assert np.array_equal(nint.cpu().numpy().astype(np.int64), nr)
            assert rel_err(g_pm.cpu().numpy(), apm).max() <= 1e-10
        else:
            assert np.percentile(e, 99) <= 1e-3


@pytest.mark.slow
@pytest.mark.timeout(900)
def test_full_lognormal_256():
    """Workload 4 at full size (256^3 clustered particles, 256^3 mesh):
    complete topology and FP64 moments bit-exact; deposited density and
    potential cell by cell; on the 0.1 % time-bin set (16,777 targets) the
    geometric pass, the mesh force and the relative pass fed the oracle's |a|
    within 1e-10 with identical interaction counts; FP32 (tree + mesh, same
    |a|) within p99 1e-3 of FP64; the relative pass within p99 1 % of the
    exact truncated pair sum on 128 targets."""
    p = W.lognormal_box(256, 100.0, 4)
    sets, _ = W.time_bin_active_sets(p.meta["rho"])
    sub = sets[0.001]
    kw = dict(eps=100.0 / (50 * 256), periodic=True, box_size=100.0, pm_grid=256)
    rs = 1.25 * 100.0 / 256
    ctx = _ctx(**kw)
    _build(ctx, p)
    T = O.Tree(p.x, p.y, p.z, periodic=True, box=100.0)
    _tree_equal(ctx.export_tree(), T)
    _progress("tree and moments bit-exact")
    _mesh_check(ctx, p, 100.0, 256, rs, "fp64")
    _progress("mesh density and potential")
    idx = _t(sub, torch.int32)
    nint = torch.empty(sub.size, dtype=torch.int32, device=_dev())
    gb, _ = ctx.compute_forces(idx, "bh", n_interactions=nint)
    ab, _, nb = T.walk(_oracle_params(kw, "bh", kw["eps"]), targets=sub)
    assert rel_err(gb.cpu().numpy(), ab).max() <= 1e-10
    assert np.array_equal(nint.cpu().numpy().astype(np.int64), nb)
    gpm, _ = ctx.pm_long_range(idx)
    apo, _ = O.pm(p.x, p.y, p.z, None, 100.0, 256, 1.0, rs, targets=sub, want_pot=False)
    assert rel_err(gpm.cpu().numpy(), apo).max() <= 1e-10
    an = np.zeros(p.n)
    an[sub] = np.linalg.norm(ab + apo, axis=0)
    gr, _ = ctx.compute_forces(idx, "rel", a_old_norm=_t(an), n_interactions=nint)
    ctx.check()
    ar, _, nr = T.walk(_oracle_params(kw, "rel", kw["eps"]), targets=sub, anorm=an)
    assert rel_err(gr.cpu().numpy(), ar).max() <= 1e-10
    assert np.array_equal(nint.cpu().numpy().astype(np.int64), nr)
    ctx.close()
    _progress("FP64 passes of the 0.1 % set")
    c32 = _ctx(precision="fp32", **kw)
    _build(c32, p)
    g32, _ = c32.compute_forces(idx, "rel", a_old_norm=_t(an))
    p32, _ = c32.pm_long_range(idx)
    c32.check()
    e = rel_err((g32.double() + p32.double()).cpu().numpy(), ar + apo)
    assert np.percentile(e, 99) <= 1e-3, np.percentile(e, [50, 99, 100])
    c32.close()
    ad = _truncated_direct(p, kw, sub[:128])
    assert np.percentile(rel_err(ar[:, :128], ad), 99) <= 0.01


def test_pm_512_converges_to_ewald_long_range():
    """The 512^3 mesh (32 x 16 line decomposition) and the 256^3 mesh at the
    same split scale against the oracle's Ewald long-range part (Ewald force
    minus the exact short-range pair sum): the finer mesh is closer."""
    p = W.zeldovich_box(32, 100.0, 9)
    rs = 1.25 * 100.0 / 256
    samp = np.sort(np.random.default_rng(4).choice(p.n, 256, replace=False))
    full = O.ewald(p.x, p.y, p.z, None, 100.0, 1.0, 1e-3, 8.0, samp)
    P = O.make_params(periodic=True, box=100.0, eps=1e-3, treepm=True, rs=rs, rcut=12 * rs)
    short, _ = O.direct(p.x, p.y, p.z, None, P, targets=samp)
    lr = full - short
    err = {}
    for ng in (256, 512):
        ctx = _ctx(eps=0.1, periodic=True, box_size=100.0, pm_grid=ng, asmth=rs * ng / 100.0)
        _build(ctx, p)
        a, _ = ctx.pm_long_range(_t(samp.astype(np.int32), torch.int32))
        ctx.check()
        err[ng] = np.percentile(rel_err(a.cpu().numpy(), lr), 50)
    assert err[512] < 0.01 and err[512] < 0.5 * err[256], err


# ---- isolated systems: zero-padded mesh (Sec. 3.3) ---------------------------

ISO_CASES = {
    "plummer_32": (lambda: W.plummer(4096, 1), dict(eps=0.01, pm_grid=32)),
    "masses_16_shift": (lambda: W.Particles(*np.random.default_rng(8).uniform(-1, 1, (3, 3000)),
                                            mass=np.random.default_rng(9).uniform(0.1, 2, 3000)),
                        dict(eps=0.01, pm_grid=16, shift=(0.4, 0.9, 0.05))),
    "hernquist_64": (lambda: W.hernquist(1 << 14, 2), dict(eps=0.005, pm_grid=64)),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("case", sorted(ISO_CASES))
def test_isolated_pm_matches_oracle(case, prec):
    mk, kw = ISO_CASES[case]
    p = mk()
    ctx = _ctx(precision=prec, want_potential=True, **kw)
    _build(ctx, p)
    fr = ctx.export_tree()["frame"]
    order = np.random.default_rng(5).permutation(p.n)
    acc, pot = ctx.pm_long_range(_t(order, torch.int32))
    ctx.check()
    ao, po = O.pm_isolated(p.x, p.y, p.z, p.mass, fr, kw["pm_grid"], 1.0, 1.25,
                           targets=order)
    e = rel_err(acc.double().cpu().numpy(), ao)
    ep = np.abs(pot.double().cpu().numpy() - po) / np.abs(po).max()
    if prec == "fp64":
        assert e.max() <= 1e-10, e.max()
        assert ep.max() <= 1e-12, ep.max()
    else:
        h, _ = O.isolated_scale(fr[3], kw["pm_grid"], 1.25)
        _check_fp32_mesh(acc.double().cpu().numpy(), pot.double().cpu().numpy(), ao, po,
                         (2 * kw["pm_grid"]) ** 3, h)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_isolated_treepm_total_follows_direct(prec):
    """Tree (short range, theta = 0.5) plus mesh against the direct Newtonian
    sum; and the mesh conserves momentum on the GPU too."""
    p = W.plummer(8192, 3)
    ctx = _ctx(precision=prec, eps=0.01, pm_grid=64)
    _build(ctx, p)
    idx = _t(np.arange(p.n), torch.int32)
    at, _ = ctx.compute_forces(idx, "bh")
    apm, _ = ctx.pm_long_range(idx)
    ctx.check()
    tot = (at + apm).double().cpu().numpy()
    ref, _ = O.direct(p.x, p.y, p.z, None, O.make_params(eps=0.01))
    e = rel_err(tot, ref)
    assert np.percentile(e, 50) <= 0.005 and np.percentile(e, 99) <= 0.03, \
        np.percentile(e, [50, 99])
    a_pm = apm.double().cpu().numpy()
    mom = np.abs(a_pm.sum(axis=1)).max() / np.linalg.norm(a_pm, axis=0).sum()
    assert mom <= (1e-12 if prec == "fp64" else 1e-5), mom


@pytest.mark.slow
def test_isolated_hernquist_2p20_sampled():
    """Full-size isolated TreePM (2^20 particles, 128-cell mesh padded to
    256^3): mesh and relative-criterion tree walk at sampled targets."""
    p = W.hernquist(1 << 20, 2)
    kw = dict(eps=0.005, pm_grid=128)
    ctx = _ctx(precision="fp64", **kw)
    _build(ctx, p)
    fr = ctx.export_tree()["frame"]
    samp = np.sort(np.random.default_rng(1).choice(p.n, 2048, replace=False))
    idx = _t(samp, torch.int32)
    apm, _ = ctx.pm_long_range(idx)
    ao, _ = O.pm_isolated(p.x, p.y, p.z, None, fr, 128, 1.0, 1.25, targets=samp,
                          want_pot=False)
    assert rel_err(apm.cpu().numpy(), ao).max() <= 1e-10
    T = O.Tree(p.x, p.y, p.z)
    P = _oracle_params(kw, "bh", 0.005, frame=T.frame)
    a_bh, _, _ = T.walk(P, targets=samp)
    an = np.zeros(p.n)
    an[samp] = np.linalg.norm(a_bh + ao, axis=0)
    nint = torch.empty(samp.size, dtype=torch.int32, device=_dev())
    ag, _ = ctx.compute_forces(idx, "rel", a_old_norm=_t(an), n_interactions=nint)
    ctx.check()
    Pr = _oracle_params(kw, "rel", 0.005, frame=T.frame)
    ar, _, nr = T.walk(Pr, targets=samp, anorm=an)
    assert rel_err(ag.cpu().numpy(), ar).max() <= 1e-10
    assert np.array_equal(nint.cpu().numpy().astype(np.int64), nr)


def test_individual_softening_rejects_bad_values():
    from paper_1909_04667_amd import binding as B
    p = W.plummer(1000, 14)
    ctx = _ctx(eps=0.01)
    for bad in (0.0, -1.0, float("nan"), float("inf")):
        e = np.full(p.n, 0.01)
        e[517] = bad
        with pytest.raises(B.TreePMError) as ei:
            _build(ctx, p, e)
        assert ei.value.code == B.TPM_EINVAL
    # the context recovers: a good build and a walk succeed afterwards
    _build(ctx, p, np.full(p.n, 0.01))
    a, _ = ctx.compute_forces(_t(np.arange(p.n), torch.int32), "bh")
    ctx.check()
    ref, _ = ctx.compute_forces(_t(np.arange(p.n), torch.int32), "bh")
    assert torch.equal(a, ref)


def test_equal_individual_softening_is_uniform_on_gpu():
    """Equal individual softenings take the mixed code path and must give
    the uniform path's results: bit for bit in FP64 (the same operations on
    the same support), to FP32 rounding in FP32 (there the uniform path's
    1/h and h^2 are rounded from double, the mixed path's formed in float)."""
    p = W.hernquist(1 << 13, 15)
    idx = None
    for prec in ("fp64", "fp32"):
        out = []
        for eps in (None, np.full(p.n, 0.005)):
            ctx = _ctx(precision=prec, eps=0.005, want_potential=True)
            _build(ctx, p, eps)
            idx = _t(np.arange(p.n), torch.int32)
            a, pot = ctx.compute_forces(idx, "bh")
            ctx.check()
            out.append((a.cpu(), pot.cpu()))
        if prec == "fp64":
            assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
        else:
            e = rel_err(out[1][0].double().numpy(), out[0][0].double().numpy())
            assert e.max() <= 1e-5, e.max()
