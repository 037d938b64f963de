"""The forward walk at the launch sizes where it changes shape: the number of
wavefronts that share a ray group (16 down to 1 as the launch grows), far
boxes through the groups' local expansions (65,536 rays and more), ragged last
groups, groups whose rays all sit at one point, and long lists under wide ray
groups.  Against the FP64
oracle tree: decision counts exactly, values to FP32 rounding (the bound of
every tree test)."""
import numpy as np
import pytest

import synth
from gpu_helpers import assert_matches_oracle_tree, build, dev, say, shoot

pytestmark = pytest.mark.gpu


def lens_of(n, seed):
    lens = synth.gaussian_blobs(n, seed, s_lo=0.003, s_hi=0.2)
    lens.s[synth.rng(seed + 1).random(n) < 0.2] = 0.0
    return lens


@pytest.mark.parametrize("nr", [1, 64, 65, 4097, 32_769, 65_535, 65_536, 131_073, 262_145, 524_225, 524_289])
def test_walk_launch_sizes_match_oracle_tree(ora, nr):
    lens = lens_of(3000, 601)
    theta, leaf, order = 0.4, 8, 7
    say(f"[gpu] walk of {nr} rays")
    tree = build(lens, theta, leaf, order)
    g0 = synth.rng(603 + nr)
    # scattered rays, a dense patch (every box far from most of its groups), and 200 rays at one point
    rx, ry = g0.uniform(-0.6, 0.6, nr), g0.uniform(-0.6, 0.6, nr)
    k = nr // 2
    rx[:k], ry[:k] = 0.11 + 0.01 * g0.random(k), -0.07 + 0.01 * g0.random(k)
    if nr > 4000:
        rx[k:k + 200], ry[k:k + 200] = 0.3, 0.2
    T = ora.Tree(lens.x, lens.y, lens.m, lens.s, lens.q, theta, leaf, order)
    idx = np.union1d(synth.sample_rays(rx, ry, 3000, 605), np.arange(k, min(nr, k + 70)))
    idx = np.union1d(idx, np.arange(max(0, nr - 70), nr))
    ref, rc = T.shoot(rx[idx], ry[idx], counts=True)
    got = shoot(tree, rx, ry)[idx]
    assert_matches_oracle_tree(got, ref)
    withc, cnt = shoot(tree, rx, ry, counts=True)
    np.testing.assert_array_equal(cnt[idx], rc[:, [0, 1, 2, 4]])
    assert_matches_oracle_tree(withc[idx], ref)
    ao = shoot(tree, rx, ry, alpha_only=True)[idx]
    np.testing.assert_array_equal(ao, got[:, :2])
    import paper_1312_1128_amd as g
    import torch

    o = g.shoot_potential(tree, dev(rx), dev(ry))
    torch.cuda.synchronize()
    psi, ref_psi = o["psi"].double().cpu().numpy()[idx], T.shoot_psi(rx[idx], ry[idx])
    assert np.abs(psi - ref_psi).max() <= 2e-6 * np.abs(ref_psi).max()


@pytest.mark.parametrize("order", range(13))
def test_far_expansion_at_every_order(ora, order):
    """70,000 rays in a small patch outside and inside the lens: most accepted
    boxes go through the local expansion, at each multipole order, for Gaussians
    and halos."""
    lens = lens_of(1500, 611)
    g0 = synth.rng(613)
    rx, ry = 0.2 + 0.02 * g0.random(70_000), 0.1 + 0.02 * g0.random(70_000)
    rx[:20_000] += 0.9
    idx = np.arange(0, rx.size, 41)
    say(f"[gpu] far expansion at order {order}")
    T = ora.Tree(lens.x, lens.y, lens.m, lens.s, lens.q, 0.5, 4, order)
    got = shoot(build(lens, 0.5, 4, order), rx, ry)[idx]
    assert_matches_oracle_tree(got, T.shoot(rx[idx], ry[idx]))
    import paper_1312_1128_amd as g

    halos, c = synth.nfw_halo_field(800, 615)
    tree = g.Tree().build(dev(halos.x), dev(halos.y), dev(halos.m), dev(halos.s), theta=0.5, q=c, leaf_size=4,
                          order=order, nfw=True)
    T = ora.Tree(halos.x, halos.y, halos.m, halos.s, c, 0.5, 4, order, nfw=True)
    assert_matches_oracle_tree(shoot(tree, rx, ry)[idx], T.shoot(rx[idx], ry[idx]))


def test_wide_groups_over_a_dense_core(ora):
    """A few thousand scattered rays over a halo whose core is far denser than
    the rays: lists of thousands of particles per group, each holding few rays."""
    lens = synth.nfw_halo(40_000, 621)
    rx, ry = synth.uniform_points(3001, 622)
    say("[gpu] wide groups over a dense core")
    tree = build(lens, 0.4, 8, 6)
    T = ora.Tree(lens.x, lens.y, lens.m, lens.s, lens.q, 0.4, 8, 6)
    ref, rc = T.shoot(rx, ry, counts=True)
    got, cnt = shoot(tree, rx, ry, counts=True)
    np.testing.assert_array_equal(cnt, rc[:, [0, 1, 2, 4]])
    assert_matches_oracle_tree(got, ref)


@pytest.mark.parametrize("nfw", [False, True])
@pytest.mark.parametrize("lensing", [False, True])
def test_adjoint_of_one_wavefront_per_group_is_the_sum_over_parts(nfw, lensing):
    """300,001 rays on 3,000 particles take one wavefront per ray group, parts
    of 50,000 several, with other far boxes and another particle pass; the
    gradient is linear in the rays, so the parts add up to it (FP32 words of
    boxes and profiles, summed in FP64: 2e-6 of the largest, as against the oracle)."""
    import paper_1312_1128_amd as g
    import torch

    gen = synth.rng(771)
    n, nr = 3000, 300_001
    x, y, m = gen.uniform(-1, 1, n), gen.uniform(-1, 1, n), gen.uniform(0.1, 1.0, n)
    s = gen.uniform(0.002, 0.2, n)
    s[gen.random(n) < 0.2] = 0.0
    say(f"[gpu] adjoint parts nfw={nfw} lensing={lensing}")
    tree = g.Tree().build(dev(x), dev(y), dev(m), dev(s), theta=0.4, q=5.0 if nfw else 3.0, leaf_size=8, order=6, nfw=nfw)
    rx, ry = dev(gen.uniform(-1, 1, nr)), dev(gen.uniform(-1, 1, nr))
    cot = torch.as_tensor(gen.normal(size=(5, nr)).astype(np.float32), device="cuda")

    def grad(parts):
        out = [torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(4)]
        for a in range(0, nr, parts):
            c = [v[a:a + parts].contiguous() for v in cot]
            kw = dict(gk=c[2], gg1=c[3], gg2=c[4]) if lensing else {}
            g.shoot_adjoint(tree, rx[a:a + parts].contiguous(), ry[a:a + parts].contiguous(), c[0], c[1], *out, **kw)
        torch.cuda.synchronize()
        return [o.cpu().numpy() for o in out]

    for name, whole, parts in zip("mxys", grad(nr), grad(50_000)):
        assert np.abs(whole).max() > 0
        assert np.abs(whole - parts).max() <= 2e-6 * np.abs(parts).max(), name


@pytest.mark.parametrize("bad", [(np.inf, 0.1), (0.1, -np.inf), (np.inf, -np.inf), (1e200, 0.1), (np.nan, 0.1)],
                         ids=lambda b: f"{b[0]:g},{b[1]:g}")
@pytest.mark.parametrize("nr", [70_000, 300_001])
def test_a_ray_at_infinity_leaves_its_group_alone(ora, nr, bad):
    """A ray with an infinite, overflowing or NaN coordinate among rays whose launch
    expands far boxes (several wavefronts per group and one), and in a batch: the
    other rays keep the values of the oracle tree."""
    import paper_1312_1128_amd as g
    import torch

    lens = lens_of(400, 631)
    rx, ry = synth.uniform_points(nr, 632, -0.7, 0.7)
    at = 1000
    idx = np.setdiff1d(np.union1d(np.arange(at - 130, at + 130), np.arange(0, nr, 97)), [at])
    T = ora.Tree(lens.x, lens.y, lens.m, lens.s, lens.q, 0.5, 4, 4)
    ref, ref_psi = T.shoot(rx[idx], ry[idx]), T.shoot_psi(rx[idx], ry[idx])
    rx[at], ry[at] = bad
    tree = build(lens, 0.5, 4, 4)
    say(f"[gpu] ray at {bad} of {nr}")
    assert_matches_oracle_tree(shoot(tree, rx, ry)[idx], ref)
    assert_matches_oracle_tree(shoot(tree, rx, ry, counts=True)[0][idx], ref)
    o = g.shoot_potential(tree, dev(rx), dev(ry))
    torch.cuda.synchronize()
    assert np.abs(o["psi"].double().cpu().numpy()[idx] - ref_psi).max() <= 2e-6 * np.abs(ref_psi).max()
    k = at + 130
    b = g.shoot_batched([tree, tree], [(dev(rx[:k]), dev(ry[:k])), (dev(rx[at + 1:k]), dev(ry[at + 1:k]))])
    torch.cuda.synchronize()
    got = np.stack([b[0][q].double().cpu().numpy() for q in ["a1", "a2", "kappa", "g1", "g2"]], axis=1)
    near = idx < k
    assert_matches_oracle_tree(got[idx[near]], ref[near])


@pytest.mark.parametrize("n", [1, 5, 90, 160, 300])
@pytest.mark.parametrize("nr", [70_000, 300_001, 530_001])
def test_small_trees_under_many_rays(ora, n, nr):
    """Trees of a few boxes up to the size from which far boxes are expanded (64), under
    launches that expand them on larger trees, with several wavefronts per group and
    one: the product walk, with counts, alpha only, plain FP32 sums and the potential."""
    import paper_1312_1128_amd as g
    import torch

    lens = lens_of(n, 641)
    rx, ry = synth.uniform_points(nr, 642, -0.7, 0.7)
    idx = np.union1d(synth.sample_rays(rx, ry, 1500, 643), np.arange(nr - 70, nr))
    tree = build(lens, 0.5, 6, 5)
    say(f"[gpu] {n} particles in {tree.info()['ncells']} boxes, {nr} rays")
    T = ora.Tree(lens.x, lens.y, lens.m, lens.s, lens.q, 0.5, 6, 5)
    ref, rc = T.shoot(rx[idx], ry[idx], counts=True)
    got = shoot(tree, rx, ry)[idx]
    assert_matches_oracle_tree(got, ref)
    withc, cnt = shoot(tree, rx, ry, counts=True)
    np.testing.assert_array_equal(cnt[idx], rc[:, [0, 1, 2, 4]])
    np.testing.assert_array_equal(withc[idx], got)
    np.testing.assert_array_equal(shoot(tree, rx, ry, alpha_only=True)[idx], got[:, :2])
    plain = shoot(tree, rx, ry, fp32_alpha=True)[idx]
    assert np.abs(plain[:, :2] - ref[:, :2]).max() <= 1e-4 * np.abs(ref[:, :2]).max()
    o = g.shoot_potential(tree, dev(rx), dev(ry))
    torch.cuda.synchronize()
    ref_psi = T.shoot_psi(rx[idx], ry[idx])
    assert np.abs(o["psi"].double().cpu().numpy()[idx] - ref_psi).max() <= 2e-6 * np.abs(ref_psi).max()


@pytest.mark.parametrize("n", [2047, 2500])
def test_uneven_lens(ora, n):
    """Equal mass per octave of radius over four decades, below and above the size from which
    such a lens's groups get more wavefronts: the walk against the oracle tree, the
    adjoint against its sum over parts that take other launch shapes."""
    import paper_1312_1128_amd as g
    import torch

    gen = synth.rng(651)
    rad, phi, nr = 10.0 ** gen.uniform(-4, -0.3, n), gen.uniform(0, 2 * np.pi, n), 280_001
    x, y, m, s = rad * np.cos(phi), rad * np.sin(phi), gen.uniform(0.5, 1.0, n), 6 * rad / np.sqrt(n)
    rx, ry = synth.uniform_points(nr, 652)
    rx[::3], ry[::3] = 1e-2 * rx[::3], 1e-2 * ry[::3]
    idx = np.union1d(synth.sample_rays(rx, ry, 2000, 653), np.arange(0, nr, 211))
    say(f"[gpu] uneven lens of {n}")
    tree = g.Tree().build(dev(x), dev(y), dev(m), dev(s), theta=0.4, q=3.0, leaf_size=8, order=6)
    T = ora.Tree(x, y, m, s, 3.0, 0.4, 8, 6)
    ref, rc = T.shoot(rx[idx], ry[idx], counts=True)
    got, cnt = shoot(tree, rx, ry, counts=True)
    np.testing.assert_array_equal(cnt[idx], rc[:, [0, 1, 2, 4]])
    assert_matches_oracle_tree(got[idx], ref)
    X, Y = dev(rx), dev(ry)
    cot = torch.as_tensor(gen.normal(size=(5, nr)).astype(np.float32), device="cuda")
    whole = g.shoot_adjoint(tree, X, Y, cot[0], cot[1], gk=cot[2], gg1=cot[3], gg2=cot[4])
    parts = None
    for a in range(0, nr, 30_000):
        c = [v[a:a + 30_000].contiguous() for v in cot]
        parts = g.shoot_adjoint(tree, X[a:a + 30_000].contiguous(), Y[a:a + 30_000].contiguous(), c[0], c[1],
                                *(parts or ()), gk=c[2], gg1=c[3], gg2=c[4])
    for name, w, p in zip("mxys", whole, parts):
        w, p = w.cpu().numpy(), p.cpu().numpy()
        assert np.abs(w).max() > 0
        assert np.abs(w - p).max() <= 2e-6 * np.abs(p).max(), name


@pytest.mark.parametrize("n,nr", [(2048, 1), (2048, 4097), (9000, 64), (9000, 65), (9000, 3000), (9000, 70_000),
                                  (9000, 140_000), (9000, 262_145)])
@pytest.mark.parametrize("theta", [0.0, 0.05, 0.1])
@pytest.mark.parametrize("nfw", [False, True])
def test_walks_that_open_most_of_the_tree(ora, n, nr, theta, nfw):
    """Opening angles so small that a launch of few groups splits the tree into box ranges (and
    just above), from 64 ranges to one: values and decision counts against the oracle tree, the
    walk's variants against each other, and the adjoint against its sum over parts."""
    import paper_1312_1128_amd as g
    import torch

    if nfw:
        lens, c = synth.nfw_halo_field(n, 661)
    else:
        lens, c = lens_of(n, 661), 3.0
    leaf, order = 10, 3
    rx, ry = synth.uniform_points(nr, 662, -0.6, 0.6)
    idx = np.unique(np.r_[0, nr - 1, np.linspace(0, nr - 1, 400).astype(int)])
    say(f"[gpu] open walk n={n} rays={nr} theta={theta} nfw={nfw}")
    tree = g.Tree().build(dev(lens.x), dev(lens.y), dev(lens.m), dev(lens.s), theta=theta, q=c, leaf_size=leaf, order=order,
                          nfw=nfw)
    T = ora.Tree(lens.x, lens.y, lens.m, lens.s, c, theta, leaf, order, nfw=nfw)
    ref, rc = T.shoot(rx[idx], ry[idx], counts=True)
    got = shoot(tree, rx, ry)
    assert_matches_oracle_tree(got[idx], ref)
    withc, cnt = shoot(tree, rx, ry, counts=True)
    np.testing.assert_array_equal(cnt[idx], rc[:, [0, 1, 2, 4]])
    np.testing.assert_array_equal(withc, got)
    np.testing.assert_array_equal(shoot(tree, rx, ry, alpha_only=True), got[:, :2])
    o = g.shoot_potential(tree, dev(rx), dev(ry))
    torch.cuda.synchronize()
    psi, ref_psi = o["psi"].double().cpu().numpy()[idx], T.shoot_psi(rx[idx], ry[idx])
    assert np.abs(psi - ref_psi).max() <= 2e-6 * np.abs(ref_psi).max()
    X, Y = dev(rx), dev(ry)
    cot = torch.as_tensor(synth.rng(663).normal(size=(5, nr)).astype(np.float32), device="cuda")
    whole = g.shoot_adjoint(tree, X, Y, cot[0], cot[1], gk=cot[2], gg1=cot[3], gg2=cot[4])
    parts, step = None, max(1, nr // 3 + 1)
    for a in range(0, nr, step):
        k = [v[a:a + step].contiguous() for v in cot]
        parts = g.shoot_adjoint(tree, X[a:a + step].contiguous(), Y[a:a + step].contiguous(), k[0], k[1], *(parts or ()),
                                gk=k[2], gg1=k[3], gg2=k[4])
    for name, w, p in zip("mxys", whole, parts):
        w, p = w.cpu().numpy(), p.cpu().numpy()
        assert np.abs(w).max() > 0
        assert np.abs(w - p).max() <= 2e-6 * np.abs(p).max(), name


@pytest.mark.parametrize("nr", [70_000, 530_001])
@pytest.mark.parametrize("order", range(13))
def test_far_adjoint_and_potential_at_every_order(ora, order, nr):
    """Rays in a small patch, in launches that expand far boxes (several wavefronts per
    group and one), at each order: the potential against the oracle tree, and
    the adjoint with alpha and with all cotangents against the sum over parts that expand none
    (FP32 words summed in FP64 on both sides: 2e-6 of the largest, as against the oracle)."""
    import paper_1312_1128_amd as g
    import torch

    lens = lens_of(1500, 651)
    gen = synth.rng(652)
    rx, ry = 0.2 + 0.02 * gen.random(nr), 0.1 + 0.02 * gen.random(nr)
    rx[:nr // 3] += 0.9
    tree = build(lens, 0.5, 4, order)
    say(f"[gpu] far adjoint and potential at order {order}, {nr} rays")
    drx, dry = dev(rx), dev(ry)
    idx = np.arange(0, nr, 61)
    T = ora.Tree(lens.x, lens.y, lens.m, lens.s, lens.q, 0.5, 4, order)
    ref = T.shoot_psi(rx[idx], ry[idx])
    psi = g.shoot_potential(tree, drx, dry)["psi"].double().cpu().numpy()[idx]
    assert np.abs(psi - ref).max() <= 2e-6 * np.abs(ref).max()
    cot = torch.as_tensor(gen.normal(size=(5, nr)).astype(np.float32), device="cuda")
    for lensing in (False, True):
        def grad(parts):
            out = [torch.zeros(lens.x.size, dtype=torch.float64, device="cuda") for _ in range(4)]
            for a in range(0, nr, parts):
                c = [v[a:a + parts].contiguous() for v in cot]
                kw = dict(gk=c[2], gg1=c[3], gg2=c[4]) if lensing else {}
                g.shoot_adjoint(tree, drx[a:a + parts].contiguous(), dry[a:a + parts].contiguous(), c[0], c[1], *out, **kw)
            return [o.cpu().numpy() for o in out]

        for name, whole, parts in zip("mxys", grad(nr), grad(50_000)):
            assert np.abs(whole).max() > 0
            assert np.abs(whole - parts).max() <= 2e-6 * np.abs(parts).max(), (name, lensing)


@pytest.mark.parametrize("n,nr", [(9000, 10_001), (9000, 25_001), (33_000, 10_001), (33_000, 60_001)])
@pytest.mark.parametrize("theta", [0.05, 0.1])
def test_open_adjoint_of_an_uneven_lens(n, nr, theta):
    """Over a lens with equal mass per octave of radius the adjoint is split into box ranges up to
    larger opening angles, by one or several wavefronts per range: against its sum over
    parts of 97 rays (two groups, in 64 ranges, several wavefronts each) and of 3,000."""
    import paper_1312_1128_amd as g
    import torch

    gen = synth.rng(671)
    rad, phi = 10.0 ** gen.uniform(-4, -0.3, n), gen.uniform(0, 2 * np.pi, n)
    x, y, m, s = rad * np.cos(phi), rad * np.sin(phi), gen.uniform(0.5, 1.0, n), 6 * rad / np.sqrt(n)
    rx, ry = synth.uniform_points(nr, 672)
    rx[::3], ry[::3] = 1e-2 * rx[::3], 1e-2 * ry[::3]
    say(f"[gpu] open adjoint of an uneven lens n={n} rays={nr} theta={theta}")
    tree = g.Tree().build(dev(x), dev(y), dev(m), dev(s), theta=theta, q=3.0, leaf_size=16, order=5)
    X, Y = dev(rx), dev(ry)
    cot = torch.as_tensor(gen.normal(size=(5, nr)).astype(np.float32), device="cuda")

    def grad(lo, hi, step):
        out = None
        for a in range(lo, hi, step):
            b = min(a + step, hi)
            c = [v[a:b].contiguous() for v in cot]
            out = g.shoot_adjoint(tree, X[a:b].contiguous(), Y[a:b].contiguous(), c[0], c[1], *(out or ()), gk=c[2], gg1=c[3],
                                  gg2=c[4])
        return [o.cpu().numpy() for o in out]

    for step, hi in ((97, 1500), (3000, nr)):
        for name, w, p in zip("mxys", grad(0, hi, hi), grad(0, hi, step)):
            assert np.abs(w).max() > 0
            assert np.abs(w - p).max() <= 2e-6 * np.abs(p).max(), (name, step)
