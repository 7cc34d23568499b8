"""wk_score_chunks where its launch changes: one workgroup more per 64 candidates, other workgroups above 128 and 1,024."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_22718_amd as wk
from wkt import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [63, 64, 65, 127, 128, 129, 1023, 1024, 1025, 4095])
@pytest.mark.parametrize("norm_mode", [wk.WK_NORM_MAX, wk.WK_NORM_MINMAX, wk.WK_NORM_MEAN])
def test_exact_ties_across_workgroups(M, norm_mode):
    # poses on a coarse grid: many candidates at exactly the same distance, in different workgroups; lower id first
    rng = np.random.default_rng(M)
    poses = rng.integers(-1, 2, (M, 5)).astype(np.float32)
    cur = np.array([1, 0, -1, 0.5, 0.25], np.float32)
    R, d = M, dev()
    ids = torch.full((R,), -7, dtype=torch.int32, device=d)
    dist = torch.full((R,), -7.0, dtype=torch.float64, device=d)
    nf = torch.full((1,), -7, dtype=torch.int32, device=d)
    wk.wk_score_chunks(torch.from_numpy(poses).to(d), M, cur, norm_mode, R, ids, dist, nf)
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    _, _, o_all = oracle.score_chunks(poses, cur, R, norm_mode)
    assert int(nf.item()) == M
    np.testing.assert_array_equal(np.sort(ids), np.arange(M))
    np.testing.assert_allclose(dist, o_all[ids], rtol=0, atol=1e-7)   # as the bar of the other retrieval tests
    assert np.all(np.diff(dist) >= 0)
    assert np.all(np.diff(ids)[np.diff(dist) == 0] > 0)


# 16 candidates a workgroup, a row of 16 lanes for every pair of the others: one candidate, partial rows and workgroups, odd counts
@pytest.mark.parametrize("M", [1, 2, 3, 15, 16, 17, 31, 33, 255, 1009, 2049])
@pytest.mark.parametrize("norm_mode", [wk.WK_NORM_MAX, wk.WK_NORM_MINMAX, wk.WK_NORM_MEAN])
def test_top_of_any_count(M, norm_mode):
    rng = np.random.default_rng(7 * M)
    poses, cur = rng.normal(0, 2, (M, 5)).astype(np.float32), rng.normal(0, 2, 5).astype(np.float32)
    R, d = min(M, 12) + 2, dev()
    ids = torch.full((R,), -7, dtype=torch.int32, device=d)
    dist = torch.full((R,), -7.0, dtype=torch.float64, device=d)
    nf = torch.full((1,), -7, dtype=torch.int32, device=d)
    wk.wk_score_chunks(torch.from_numpy(poses).to(d), M, cur, norm_mode, R, ids, dist, nf)
    o_ids, o_dist, _ = oracle.score_chunks(poses, cur, R, norm_mode)
    n = int(nf.item())
    assert n == min(R, M)
    np.testing.assert_array_equal(ids.cpu().numpy()[:n], o_ids[:n])
    np.testing.assert_allclose(dist.cpu().numpy()[:n], o_dist[:n], rtol=1e-12, atol=1e-14)   # fp64 throughout
    assert (ids.cpu().numpy()[n:] == -1).all() and np.isinf(dist.cpu().numpy()[n:]).all()


# angles at and beside the ends of a quadrant, half turns, equal poses, tiny and large differences, beyond the reduction's range too
@pytest.mark.parametrize("kind", ["quadrants", "half_turns", "tiny", "turns", "beyond"])
def test_rotation_angles(kind):
    M, d, rng = 700, dev(), np.random.default_rng(5)
    off = rng.uniform(-1, 1, (M, 2)) * 10.0 ** rng.integers(-9, -1, (M, 1))
    yaw, pitch = {"quadrants": (rng.integers(-8, 9, M) * np.pi / 2, rng.integers(-8, 9, M) * np.pi / 2), "half_turns": (np.full(M, np.pi), np.zeros(M)),
                  "tiny": (np.zeros(M), np.zeros(M)), "turns": (rng.uniform(-2e5, 2e5, M), rng.uniform(-1, 1, M)),
                  "beyond": (rng.uniform(-1e8, 1e8, M), rng.uniform(-1, 1, M))}[kind]
    poses = np.zeros((M, 5), np.float32)
    poses[:, 3], poses[:, 4] = yaw + off[:, 0], pitch + off[:, 1]
    poses[:5] = poses[5]
    cur = np.zeros(5, np.float32)
    hD, he = (poses[:, c].astype(np.longdouble) / 2 for c in (3, 4))
    angle = 2 * np.arctan2(np.sqrt(np.sin(hD) ** 2 + (np.cos(hD) * np.sin(he)) ** 2), np.abs(np.cos(hD) * np.cos(he)))
    ids = torch.zeros(M, dtype=torch.int32, device=d)
    dist, nf = torch.zeros(M, dtype=torch.float64, device=d), torch.zeros(1, dtype=torch.int32, device=d)
    wk.wk_score_chunks(torch.from_numpy(poses).to(d), M, [0.0] * 5, wk.WK_NORM_MAX, M, ids, dist, nf)
    want = (angle / angle.max())[ids.cpu().numpy()]
    # a handful of roundings of 2^-53 and the division's; sines and cosines beside their zeros are as good as pi/2 in two parts is, 2^-106 of up to 2^20 of them
    np.testing.assert_allclose(dist.cpu().numpy(), want.astype(np.float64), rtol=2e-15, atol=1e-25)


# The angle's error is that of an arctangent of rounded sines and cosines: what numpy's functions give in fp64, and a tenth.  Beside a quarter turn two tenths: there sine,
# cosine and their sum under the root have their full weight, and are off by 0.30 to 0.31 units in the last place (rms over a quadrant) where numpy's are off by
# 0.29, each of them three roundings deep.
@pytest.mark.parametrize("kind", ["any", "wide", "right", "small"])
def test_rotation_precision(kind):
    M, d = 4096, dev()
    yaw, pitch = {"any": (np.pi, np.pi / 6), "wide": (30.0, 0.5), "right": (0.16, 0.1), "small": (0.2, 0.1)}[kind]
    errors = []
    for seed in range(24):   # (the largest angle's error is in all of a call)
        rng = np.random.default_rng(seed)
        poses = np.zeros((M, 5), np.float32)
        poses[:, 3] = rng.uniform(-yaw, yaw, M) + (np.pi / 2 if kind == "right" else 0)
        poses[:, 4] = rng.uniform(-pitch, pitch, M)

        def angles(t):
            hD, he = (poses[:, c].astype(t) / 2 for c in (3, 4))
            return 2 * np.arctan2(np.sqrt(np.sin(hD) ** 2 + (np.cos(hD) * np.sin(he)) ** 2), np.abs(np.cos(hD) * np.cos(he)))

        ids = torch.zeros(M, dtype=torch.int32, device=d)
        dist, nf = torch.zeros(M, dtype=torch.float64, device=d), torch.zeros(1, dtype=torch.int32, device=d)
        wk.wk_score_chunks(torch.from_numpy(poses).to(d), M, [0.0] * 5, wk.WK_NORM_MAX, M, ids, dist, nf)
        exact, plain = angles(np.longdouble), angles(np.float64)
        exact, plain = exact / exact.max(), plain / plain.max()
        got = np.empty(M)
        got[ids.cpu().numpy()] = dist.cpu().numpy()
        errors.append([(x - exact).astype(np.float64) for x in (got, plain)])
    off, bound = np.sqrt((np.array(errors) ** 2).mean(axis=(0, 2)))
    assert off <= (1.2 if kind == "right" else 1.1) * bound, (off, bound)
