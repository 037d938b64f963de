"""GPU direct sum (FP64 and FP32) against oracle A, element by element."""
import numpy as np
import pytest

import synth
from gpu_helpers import dev, rel_err, say, stats

pytestmark = pytest.mark.gpu

# FP32 terms summed in FP64, against the FP64 brute force: largest measured per-ray
# errors alpha 2.8e-7, kappa 9.6e-7, gamma 1.9e-5 (a ray of the 1k point-mass field
# where the shear is a small difference of large terms); the bounds are ~3x those
FP32_MAX = {"alpha": 1e-6, "kappa": 3e-6, "gamma": 6e-5}


def run_direct(lens, rx, ry, fp64):
    import paper_1312_1128_amd as g
    import torch

    out = g.shoot_direct(dev(lens.x), dev(lens.y), dev(lens.m), dev(lens.s), lens.q, dev(rx), dev(ry), fp64=fp64)
    torch.cuda.synchronize()
    return np.stack([out[k].double().cpu().numpy() for k in ["a1", "a2", "kappa", "g1", "g2"]], axis=1)


@pytest.mark.parametrize("which", ["point_masses_1k", "blobs_3k", "nfw_50k"])
def test_direct_matches_oracle(ora, which):
    if which == "point_masses_1k":
        lens, rx, ry = synth.workload_point_masses_1k()
    elif which == "blobs_3k":
        lens = synth.gaussian_blobs(3000, 61, s_lo=0.001, s_hi=0.2)
        lens.s[::4] = 0.0
        rx, ry = synth.uniform_points(3001, 62)
    else:
        lens = synth.nfw_halo(50000, 63)
        rx, ry = synth.ray_grid(50)
    say(f"[gpu] direct {which}: n={lens.n} rays={rx.size}")
    ref = ora.direct(lens.x, lens.y, lens.m, lens.s, lens.q, rx, ry)
    d64 = run_direct(lens, rx, ry, True)
    ea, ek, eg = rel_err(d64, ref)
    stats("fp64 alpha", ea)
    assert ea.max() <= 1e-10 and eg.max() <= 1e-10
    if lens.s.max() > 0:
        ok = ref[:, 2] != 0
        assert np.all(ek[ok] <= 1e-10)
    d32 = run_direct(lens, rx, ry, False)
    ea, ek, eg = rel_err(d32, ref)
    stats("fp32 alpha", ea)
    stats("fp32 gamma", eg)
    zero = ref[:, 2] == 0
    assert np.all(d32[zero, 2] == 0.0)  # no particle holds the ray: kappa exactly 0
    if (~zero).any():
        stats("fp32 kappa", ek[~zero])
    # each FP32 term is within a few ulp, so per ray the error is a few 1e-7 of
    # the sum of the terms' magnitudes, which exceeds |gamma| where terms cancel
    assert ea.max() <= FP32_MAX["alpha"] and eg.max() <= FP32_MAX["gamma"]
    assert np.all(ek[~zero] <= FP32_MAX["kappa"])


@pytest.mark.parametrize("n,nr", [(1, 1), (63, 15), (64, 17), (255, 4097), (256, 8191), (1023, 8192), (1024, 8193),
                                  (1025, 16), (300, 131_071), (257, 131_073)])
@pytest.mark.parametrize("nfw", [False, True])
def test_direct_at_tile_and_workgroup_edges(ora, n, nr, nfw):
    """Particle counts around a tile, ray counts around the sizes where a
    workgroup takes 4, 16 or 64 rays; rays exactly on particles included."""
    import paper_1312_1128_amd as g
    import torch

    if nfw:
        lens, c = synth.nfw_halo_field(n, 71)
    else:
        lens, c = synth.gaussian_blobs(n, 71, s_lo=0.01, s_hi=0.2), 3.0
        lens.s[::5] = 0.0
    rx, ry = synth.uniform_points(nr, 72, -0.7, 0.7)
    k = min(n, nr) // 2
    rx[:k], ry[:k] = lens.x[:k], lens.y[:k]
    idx = np.union1d(synth.sample_rays(rx, ry, 4000, 73), [0, nr - 1])
    say(f"[gpu] direct edges n={n} rays={nr} nfw={nfw}")
    ref = (ora.direct_nfw if nfw else ora.direct)(lens.x, lens.y, lens.m, lens.s, c, rx[idx], ry[idx])
    for fp64, tol in ((True, 1e-10), (False, 1e-5)):
        o = g.shoot_direct(dev(lens.x), dev(lens.y), dev(lens.m), dev(lens.s), c, dev(rx), dev(ry), fp64=fp64, nfw=nfw)
        torch.cuda.synchronize()
        got = np.stack([o[q].double().cpu().numpy()[idx] for q in ["a1", "a2", "kappa", "g1", "g2"]], axis=1)
        for cols in (slice(0, 2), slice(2, 3), slice(3, 5)):
            mag = np.linalg.norm(ref[:, cols], axis=1)
            err = np.linalg.norm(got[:, cols] - ref[:, cols], axis=1)
            assert np.all(err <= tol * (mag + 1e-2 * mag.max() + 1e-300)), (fp64, cols)


@pytest.mark.parametrize("n,nr", [(17, 5), (65, 9000), (1025, 30), (257, 131_073)])
@pytest.mark.parametrize("nfw", [False, True])
def test_direct_next_to_the_origin(ora, n, nr, nfw):
    """Rays off the origin by less than FP32 (and FP64) can square, particle counts that fill no
    step of a workgroup: the places of a step that hold no particle add nothing."""
    import paper_1312_1128_amd as g
    import torch

    gen = synth.rng(81)
    phi, c = gen.uniform(0, 2 * np.pi, n), 3.0
    x, y, m = 0.4 * np.cos(phi), 0.4 * np.sin(phi), gen.uniform(0.5, 1.0, n)
    s = gen.uniform(0.01, 0.1, n)
    rx, ry = synth.uniform_points(nr, 82, -0.7, 0.7)
    tiny = np.array([1e-21, 3e-20, 1e-22, 1e-158, 1e-161])
    rx[:5], ry[:5] = tiny, -tiny
    idx = np.unique(np.r_[np.arange(5), np.arange(0, nr, 37)])
    say(f"[gpu] direct next to the origin n={n} rays={nr} nfw={nfw}")
    ref = (ora.direct_nfw if nfw else ora.direct)(x, y, m, s, c, rx[idx], ry[idx])
    for fp64, tol in ((True, 1e-10), (False, 1e-5)):
        o = g.shoot_direct(dev(x), dev(y), dev(m), dev(s), c, dev(rx), dev(ry), fp64=fp64, nfw=nfw)
        torch.cuda.synchronize()
        got = np.stack([o[q].double().cpu().numpy()[idx] for q in ["a1", "a2", "kappa", "g1", "g2"]], axis=1)
        for cols in (slice(0, 2), slice(2, 3), slice(3, 5)):
            mag = np.linalg.norm(ref[:, cols], axis=1)
            err = np.linalg.norm(got[:, cols] - ref[:, cols], axis=1)
            assert np.all(err <= tol * (mag + 1e-2 * mag.max() + 1e-300)), (fp64, cols)


def test_direct64_over_its_range():
    """One point mass at the origin, rays from 1e-150 to 1e150 away: alpha = d / r^2 and gamma =
    -(d1^2 - d2^2, 2 d1 d2) / r^4, which are finite numbers however r^4 over- or underflows."""
    import paper_1312_1128_amd as g
    import torch

    r, phi = 10.0 ** np.arange(-150, 151, 2.5), 0.7
    d = np.stack([r * np.cos(phi), r * np.sin(phi)])
    z = np.zeros(1)
    o = g.shoot_direct(dev(z), dev(z), dev(z + 1.0), dev(z), 3.0, dev(d[0]), dev(d[1]), fp64=True)
    torch.cuda.synchronize()
    got = {k: v.cpu().numpy() for k, v in o.items()}
    for k, ref in (("a1", np.cos(phi) / r), ("a2", np.sin(phi) / r)):
        np.testing.assert_allclose(got[k], ref, rtol=1e-13)
    with np.errstate(over="ignore", under="ignore"):
        ok = (r > 1e-150) & (r < 1e150)
        for k, ref in (("g1", -np.cos(2 * phi) / r[ok] / r[ok]), ("g2", -np.sin(2 * phi) / r[ok] / r[ok])):
            np.testing.assert_allclose(got[k][ok], ref, rtol=1e-12)
    # inside a Gaussian and just above the range of r^2: its centre's kappa and no shear
    r = 10.0 ** np.arange(-156, -139, 1.0)
    o = g.shoot_direct(dev(z), dev(z), dev(z + 1.0), dev(z + 0.1), 3.0, dev(r * np.cos(phi)), dev(r * np.sin(phi)), fp64=True)
    torch.cuda.synchronize()
    kappa = 50.0 / -np.expm1(-4.5)
    np.testing.assert_allclose(o["kappa"].cpu().numpy(), kappa, rtol=1e-13)
    for k in ("a1", "a2", "g1", "g2"):
        assert np.abs(o[k].cpu().numpy()).max() <= 1e-9 * kappa, k


def test_direct_of_more_rays_than_one_launch_has_threads_for():
    """2^30 + 300 rays: with four threads to a ray, more than the 2^32 threads of a launch."""
    import paper_1312_1128_amd as g
    import torch

    nr = (1 << 30) + 300
    say("[gpu] direct sum of 2^30 + 300 rays")
    p = [dev(np.array(v)) for v in ([0.3, -0.2], [0.1, 0.4], [1.0, 0.5], [0.05, 0.0])]
    rx = torch.linspace(-1.0, 1.0, nr, dtype=torch.float64, device="cuda")
    o = g.shoot_direct(*p, 3.0, rx, rx, alpha_only=True)
    for a, b in ((0, 4096), (nr // 2 - 2048, nr // 2 + 2048), (nr - 4096, nr)):
        e = g.shoot_direct(*p, 3.0, rx[a:b].contiguous(), rx[a:b].contiguous(), alpha_only=True)
        for k in ("a1", "a2"):
            torch.testing.assert_close(o[k][a:b], e[k], rtol=1e-6, atol=1e-6)
