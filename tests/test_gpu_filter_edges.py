"""The filter kernel at the edges of its 32-patch steps and tiles, against the FP64 oracle.

Tolerance: a contribution is rounded to a multiple of 2^-9 or finer (at most 2^-10 off), and the
fp16 hi/lo operands and FP32 sums leave about 2^-21 of values below 2^11 (2^-10) in each patch, so
an averaged pixel is within 2^-9 + 2^-9 = 2^-8 of the oracle as long as every keep/kill decision
agrees, which the FP64 re-decision of the values near the threshold ensures.
"""
import numpy as np
import pytest

import oracle
import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 2.0 ** -8


@pytest.fixture(scope="module")
def dn():
    import paper_2512_23569_amd as ht
    d = ht.Denoiser(0)
    yield d
    d.close()


# (h, w): fewer groups than a step holds, one row or column of groups, steps and tiles cut short by
# the last group, several tiles with remainders
@pytest.mark.parametrize("h,w,stride,window", [
    (12, 13, 4, 7), (15, 70, 5, 15), (71, 15, 3, 15), (33, 42, 4, 21), (64, 95, 3, 31), (53, 61, 2, 9),
])
@pytest.mark.parametrize("K", [4, 8, 16, 32])
@pytest.mark.parametrize("c", [1, 3])
# tau 0 keeps everything, 2 and 60 cross blocks that stay and blocks that die, 1e9 kills everything
@pytest.mark.parametrize("tau", [0.0, 2.0, 60.0, 1e9])
def test_step_and_tile_edges(dn, basis1, basis3, h, w, stride, window, K, c, tau):
    reach = min((window - 1) // 2, min(h, w) - 8) + 1
    if reach * reach < K:
        pytest.skip("the corner window holds fewer than K candidates")
    img = synth.add_awgn(synth.make_clean(h, w, c, 5 + K), 20.0, 11)
    p = dn.params(c, stride=stride, window=window, K=K)
    n_ref = len(oracle.ref_grid(h, 8, stride)) * len(oracle.ref_grid(w, 8, stride))
    taus = tau * (0.75 + 0.5 * np.arange(n_ref) / n_ref)   # another threshold for every group
    out = dn.denoise_tau(torch.from_numpy(img).cuda(), torch.from_numpy(taus).cuda(), p).cpu().numpy()
    U, V = basis3 if c == 3 else basis1
    ref = oracle.denoise(img, U, V, taus, s=stride, W=window, K=K)
    assert np.abs(out - ref).max() <= TOL


@pytest.mark.parametrize("c,K", [(3, 32), (3, 8), (1, 16)])
def test_more_values_at_the_threshold_than_the_list_holds(dn, basis1, basis3, c, K):
    """A flat image: every coefficient but the means is exactly 0, and with tau at 0.06 (guard band
    0.01 .. 0.11) none of them counts; with a two-level pattern whole tiles of coefficients sit at
    the same value, and tau there sends them all through the FP64 list."""
    img = np.full((40, 44, c), 100, np.uint8)
    img[::2, 1::2] = 104
    img = img if c == 3 else img[:, :, 0]
    U, V = basis3 if c == 3 else basis1
    p = dn.params(c, stride=4, window=15, K=K)
    n_ref = len(oracle.ref_grid(40, 8, 4)) * len(oracle.ref_grid(44, 8, 4))
    for tau in (0.06, 1.0, 3.0):
        taus = np.full(n_ref, tau)
        out = dn.denoise_tau(torch.from_numpy(img).cuda(), torch.from_numpy(taus).cuda(), p).cpu().numpy()
        ref = oracle.denoise(img, U, V, taus, s=4, W=15, K=K)
        assert np.abs(out - ref).max() <= TOL


# the counts of a video's pixels are made by tiles of 64 x 16 of the stacked frames
@pytest.mark.parametrize("T,h,w", [(1, 15, 63), (2, 16, 64), (3, 21, 65), (2, 40, 130)])
@pytest.mark.parametrize("c", [1, 3])
def test_video_count_tiles(dn, basis1, basis3, T, h, w, c):
    v = np.stack([synth.add_awgn(synth.make_clean(h, w, c, 7), 20.0, 30 + t) for t in range(T)])
    p = dn.params(c, stride=4, window=7, K=8)
    out = dn.denoise_video(torch.from_numpy(v).cuda(), 20.0, p, radius=1).cpu().numpy()
    idx, _ = oracle.block_match_video(v, 8, 4, 7, 8, 1)
    U, V = basis3 if c == 3 else basis1
    stacked = v.reshape((T * h,) + v.shape[2:])
    ref = oracle.filter_groups(stacked, idx, U, V, 20.0 * oracle.tau_multiplier(c, 8)).reshape(v.shape)
    assert np.abs(out - ref).max() <= TOL


# frames smaller than a window's reach, with tiles of few references: a pixel then lies in the regions of
# tiles many places before its own
@pytest.mark.parametrize("T,h,w,radius,stride,window,K", [
    (1, 70, 16, 0, 1, 27, 32), (2, 19, 13, 0, 2, 31, 32), (3, 12, 33, 1, 2, 27, 32), (2, 33, 12, 1, 1, 31, 8),
    (3, 21, 22, 2, 1, 31, 16), (2, 40, 41, 1, 1, 31, 32), (6, 30, 70, 2, 2, 31, 32),
])
@pytest.mark.parametrize("c", [1, 3])
def test_video_frames_smaller_than_the_windows(dn, basis1, basis3, T, h, w, radius, stride, window, K, c):
    v = np.stack([synth.add_awgn(synth.make_clean(h, w, c, 7), 20.0, 30 + t) for t in range(T)])
    p = dn.params(c, stride=stride, window=window, K=K)
    out = dn.denoise_video(torch.from_numpy(v).cuda(), 20.0, p, radius=radius).cpu().numpy()
    idx, _ = oracle.block_match_video(v, 8, stride, window, K, radius)
    U, V = basis3 if c == 3 else basis1
    stacked = v.reshape((T * h,) + v.shape[2:])
    ref = oracle.filter_groups(stacked, idx, U, V, 20.0 * oracle.tau_multiplier(c, K)).reshape(v.shape)
    assert np.abs(out - ref).max() <= TOL


# so many frames within the radius that their regions do not fit in LDS: sums straight to memory, with steps
# and tiles cut short by the last group
@pytest.mark.parametrize("K", [4, 8, 16, 32])
@pytest.mark.parametrize("c", [1, 3])
def test_video_sums_in_memory(dn, basis1, basis3, K, c):
    T, h, w = 64, 27, 30
    v = np.stack([synth.add_awgn(synth.make_clean(h, w, c, 7), 20.0, 30 + t) for t in range(T)])
    p = dn.params(c, stride=7, window=17, K=K)
    out = dn.denoise_video(torch.from_numpy(v).cuda(), 20.0, p, radius=31).cpu().numpy()
    idx, _ = oracle.block_match_video(v, 8, 7, 17, K, 31)
    U, V = basis3 if c == 3 else basis1
    stacked = v.reshape((T * h,) + v.shape[2:])
    ref = oracle.filter_groups(stacked, idx, U, V, 20.0 * oracle.tau_multiplier(c, K)).reshape(v.shape)
    assert np.abs(out - ref).max() <= TOL


# The list of values near the threshold (within 0.05 of it) holds 64 of each wave's pass over 32 patches x 16
# columns of every slice; the FP32 value decides the rest.  An image of few ones has many equal and small
# coefficients; the threshold lies in a gap of them that is wider than the FP32 values' error (their rows'
# norms stay below 8, so 2^-22 of the split basis and 2^-24 of each of up to 192 partial sums are below 1e-4).
@pytest.mark.parametrize("over", [True, False])
@pytest.mark.parametrize("K", [4, 8, 16, 32])
@pytest.mark.parametrize("c", [1, 3])
def test_values_near_the_threshold(dn, basis1, basis3, c, K, over):
    rng = np.random.default_rng(K + c)
    img = (rng.random((20, 24, c)) < 1 / 32).astype(np.uint8)
    img = img if c == 3 else img[:, :, 0]
    U, V = basis3 if c == 3 else basis1
    idx, _ = oracle.block_match(img, 8, 7, 15, K)
    a = img.reshape(20, 24, c).astype(np.float64)
    patches = [[oracle.patch_forward(U, V, a[i // 24:i // 24 + 8, i % 24:i % 24 + 8]) for i in row] for row in idx]
    S = np.abs(np.einsum("mk,gkijc->gmijc", oracle.haar(K), np.array(patches)))
    v = np.sort(S.ravel())
    v = v[np.searchsorted(v, 0.06):]
    best, tau = 0, 0.0
    for j in np.nonzero(np.diff(v) > 2.4e-4)[0]:
        t = (v[j] + v[j + 1]) / 2
        per_group = (np.abs(S - t) < 0.05).reshape(len(S), K, 4, 16, c).sum((1, 3, 4))
        # over: more than 64 in the average pass of 32 / K groups; else at most 64 in any, but some
        n = per_group.mean(0).max() * (32 // K) if K < 32 else per_group.max()
        if not over:
            most = np.sort(per_group, axis=0)[-(32 // K):].sum(0).max()
            n = per_group.sum() if most <= 64 else 0
        if n > best:
            best, tau = n, t
    assert best > (64 if over else 0)
    p = dn.params(c, stride=7, window=15, K=K)
    out = dn.denoise_tau(torch.from_numpy(img).cuda(), torch.full((len(S),), tau, dtype=torch.float64,
                                                                  device="cuda"), p).cpu().numpy()
    in_list, beyond = dn.guard_count()
    assert (np.abs(S - tau) < 0.05 - 1e-4).sum() <= in_list + beyond <= (np.abs(S - tau) < 0.05 + 1e-4).sum()
    assert in_list > 0 and (beyond > 0) == over
    assert np.abs(out - oracle.denoise(img, U, V, tau, s=7, W=15, K=K)).max() <= TOL
