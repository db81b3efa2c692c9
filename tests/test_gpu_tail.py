"""The last paths of a render and the last photons of a flux call end in kernels
of their own (four lanes a path).  With counters a call runs to its end in the
main kernel, so each call has both ways: the same paths and the same float32
sums, added to the float64 outputs in another order (2^-52 per addition of at
most a few hundred non-negative terms: 1e-12)."""
import numpy as np
import pytest
import torch

from gpu_common import ctx, device_field
from paper_1902_01137_amd import api, inputs
from paper_1902_01137_amd.inputs import Camera, GridParams, Optics, Sampling

pytestmark = pytest.mark.gpu


def _scene(ext):
    sc = inputs.scene_small()
    c = ctx()
    kd = device_field(sc.kc)
    op = vars(sc.optics) | {"ground_albedo": 0.4}
    if ext:
        op |= {"sun_half_angle_deg": 2.0, "phase_table": api.PhaseTable(c, *inputs.phase_table_tthg(n=61)),
               "kdist": (np.array([0.3, 0.5, 0.2]), np.array([0.0, 0.02, 0.05]))}
    g = api.build_grid(c, kd, sc.desc, GridParams(sc.grid.tau_tilde, 0.05 if ext else 0.0, sc.grid.criterion))
    return sc, c, kd, g, Optics(**op)


def _close(a, b):
    torch.testing.assert_close(a, b, rtol=1e-12, atol=1e-12)


# one path; less than a wave, a last tile in part; several items a lane; more items than resident lanes
@pytest.mark.parametrize("w,h,spp", [(1, 1, 1), (9, 5, 3), (61, 43, 16), (333, 217, 16)])
@pytest.mark.parametrize("est", [0, 1, 2])
@pytest.mark.parametrize("ext", [False, True], ids=["plain", "extended"])
@pytest.mark.parametrize("camera", [0, 2], ids=["pinhole", "irradiance"])
def test_views_end_the_same_either_way(w, h, spp, est, ext, camera):
    sc, c, kd, g, op = _scene(ext)
    cam = Camera(**{**vars(sc.camera), "type": camera, "width": w, "height": h})
    smp = Sampling(seed=23, spp=spp, flags=est, stream=3)
    s, s2 = api.render(c, g, kd, op, cam, smp)
    t, t2 = api.render(c, g, kd, op, cam, smp, counters=api.new_counters("cuda"))
    torch.cuda.synchronize()
    assert w * h == 1 or float(s.sum()) > 0.0
    _close(s, t)
    _close(s2, t2)


@pytest.mark.parametrize("w,h,spp", [(9, 5, 3), (61, 43, 16)])
def test_collected_vertices_are_the_same_either_way(w, h, spp):
    sc, c, kd, g, op = _scene(False)
    cam = Camera(**{**vars(sc.camera), "width": w, "height": h})
    smp = Sampling(seed=29, spp=spp)
    cap = 400 * w * h * spp
    out = [api.collect_vertices(c, g, kd, op, cam, smp, cap, counters=cnt) for cnt in (None, api.new_counters("cuda"))]
    (ra, na, sa, qa), (rb, nb, sb, qb) = out
    assert na == nb and 0 < na <= cap
    _close(sa, sb)
    _close(qa, qb)
    # (records come in any order)
    a, b = (r.cpu().numpy().view(np.uint32) for r in (ra, rb))
    assert np.array_equal(a[np.lexsort(a.T)], b[np.lexsort(b.T)])


# one photon, ends of waves, some waves, and more photons than resident lanes with a last chunk in part
@pytest.mark.parametrize("n", [1, 63, 65, 4097, 200_003, 1_300_001])
@pytest.mark.parametrize("gas", [0.0, 0.05])
def test_photons_end_the_same_either_way(n, gas):
    sc, c, kd, _, _ = _scene(False)
    g = api.build_grid(c, kd, sc.desc, GridParams(sc.grid.tau_tilde, gas, sc.grid.criterion))
    op = Optics(ssa=0.97, g=0.8, ground_albedo=0.4, sun_zenith_deg=35.0)
    smp = Sampling(seed=31, sample_offset=5)
    px = (7, 5)
    tally, glob = api.flux(c, g, kd, op, px, n, smp)
    cnt = api.new_counters("cuda")
    tally2, glob2 = api.flux(c, g, kd, op, px, n, smp, counters=cnt)
    torch.cuda.synchronize()
    assert api.counters_dict(cnt)["paths"] == n
    assert torch.equal(glob, glob2) and float(glob.sum()) == n
    # derivative scores have either sign: bounded by their squares' sums
    bound = 1e-12 * (1.0 + tally2[[0, 1, 2, 4, 4, 6, 6, 8, 8]].abs())
    assert bool(((tally - tally2).abs() <= bound).all())
    # the adjoint's replay meets the same photons
    grad = torch.from_numpy(np.random.default_rng(7).standard_normal((px[1], px[0]))).cuda()
    out = api.flux_adjoint(c, g, kd, op, px, n, smp, grad)
    want = torch.stack([(grad * tally2[k]).sum() for k in (3, 5, 7)])
    scale = torch.stack([(grad.abs() * (tally2[0] + tally2[k + 1])).sum() for k in (3, 5, 7)])
    assert bool(((out - want).abs() <= 1e-12 * (1.0 + scale)).all())
