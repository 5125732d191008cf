"""Block matching at the edges of its window classes and selection forms: the groups and distances
are whole numbers and equal the oracle's exactly."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dn():
    import paper_2512_23569_amd as ht
    d = ht.Denoiser(0)
    yield d
    d.close()


def _image(kind, h, w, c, seed):
    rng = np.random.default_rng(seed)
    shape = (h, w, c)
    if kind.endswith("stripes"):
        # rows of period 4: in windows clipped to 8 or 16 columns the near matches fall into a few lanes
        # of one half of the wave, and the keys under the bound are many more than K
        rows = np.array([0, 250, 0, 250] if kind == "wide_stripes" else [0, 10, 200, 100])
        img = np.broadcast_to(rows[np.arange(h) % 4][:, None, None], shape) + rng.integers(0, 3, shape)
        if kind != "stripes" and c == 3:
            img[..., 1] //= 8   # channel-sum distances, the wide ones beyond 2^22 from the smallest
    elif kind == "two_values":
        # the same two values everywhere: distances tie in large sets
        img = rng.integers(0, 2, (h // 8 + 1, w // 8 + 1, 1)).repeat(8, 0).repeat(8, 1)[:h, :w] * np.full(c, 90)
    elif kind == "red_blue":
        # no green: channel-sum distances, some beyond 2^22 from the smallest
        img = rng.integers(0, 2, (h, w, 1)) * np.full(c, 255)
        if c == 3:
            img[..., 1] = 0
    else:
        # green in one half of the image, channel sums in the other
        img = rng.integers(0, 256, shape)
        if c == 3:
            img[:, : w // 2, 1] //= 4
    return np.ascontiguousarray(img.astype(np.uint8) if c == 3 else img[..., 0].astype(np.uint8))


# windows at both ends of each class (256, 448, 640 and 961 positions), unions of 1 to 4 blocks of columns
@pytest.mark.parametrize("window,stride", [(7, 3), (15, 4), (17, 3), (21, 5), (23, 4), (25, 2), (27, 7), (31, 3), (31, 8), (31, 11)])
@pytest.mark.parametrize("K", [4, 16, 32])
@pytest.mark.parametrize("kind", ["stripes", "sum_stripes", "wide_stripes", "two_values", "red_blue", "mixed"])
@pytest.mark.parametrize("c", [1, 3])
def test_groups_equal_the_oracle(dn, window, stride, K, kind, c):
    h, w = 61, 83
    if ((window - 1) // 2 + 1) ** 2 < K:
        pytest.skip("the corner window holds fewer than K candidates")
    img = _image(kind, h, w, c, window + K)
    idx, dist = dn.block_match(torch.from_numpy(img).cuda(), dn.params(c, stride=stride, window=window, K=K))
    oi, od = oracle.block_match(img, 8, stride, window, K)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(dist.cpu().numpy(), od)


@pytest.mark.parametrize("window", [7, 13, 15, 17, 21, 25, 31])
@pytest.mark.parametrize("kind", ["stripes", "wide_stripes", "red_blue"])
def test_video_groups_equal_the_oracle(dn, window, kind):
    frames = np.stack([_image(kind, 40, 51, 3, 7 * t + window) for t in range(3)])
    idx, dist = dn.block_match_video(torch.from_numpy(frames).cuda(), dn.params(3, stride=5, window=window, K=16), 1)
    oi, od = oracle.block_match_video(frames, 8, 5, window, 16, 1)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(dist.cpu().numpy(), od)


# unions of 33 and 17 columns with more tiles than two per CU: the column left over goes a row per lane
@pytest.mark.parametrize("h,w,window,stride", [(431, 301, 21, 4), (330, 420, 27, 2), (270, 300, 11, 2), (300, 270, 15, 1)])
@pytest.mark.parametrize("c", [1, 3])
def test_groups_with_a_column_left_over(dn, h, w, window, stride, c):
    img = _image("mixed", h, w, c, window)
    idx, dist = dn.block_match(torch.from_numpy(img).cuda(), dn.params(c, stride=stride, window=window, K=16))
    oi, od = oracle.block_match(img, 8, stride, window, 16)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(dist.cpu().numpy(), od)


# steps wide enough that the row sums of the norm pass, not the table, size the table's place
@pytest.mark.parametrize("window,stride", [(7, 14), (15, 9), (15, 13), (15, 16), (21, 12), (21, 14)])
@pytest.mark.parametrize("c", [1, 3])
def test_groups_at_wide_steps(dn, window, stride, c):
    img = _image("mixed", 117, 141, c, window)
    x = torch.from_numpy(img).cuda()
    p = dn.params(c, stride=stride, window=window, K=16)
    idx, dist = dn.block_match(x, p)
    oi, od = oracle.block_match(img, 8, stride, window, 16)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(dist.cpu().numpy(), od)


# more than 512 tiles of windows of 23 and 25: unions without and with columns left over by blocks of 16, and
# tiles too large for two of them to share a CU
@pytest.mark.parametrize("h,w,window,stride", [(300, 290, 23, 3), (380, 420, 23, 4), (290, 301, 25, 3), (590, 600, 25, 6)])
@pytest.mark.parametrize("c", [1, 3])
def test_groups_of_many_tiles(dn, h, w, window, stride, c):
    img = _image("mixed", h, w, c, window)
    idx, dist = dn.block_match(torch.from_numpy(img).cuda(), dn.params(c, stride=stride, window=window, K=32))
    oi, od = oracle.block_match(img, 8, stride, window, 32)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(dist.cpu().numpy(), od)
