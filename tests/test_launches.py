"""What the library's calls launch: sizes and layouts over everything that the calls accept, checked
on the host (launch_checks.py) without a GPU."""
import pytest

import fake_hip


@pytest.mark.parametrize("check", ["match_lds", "match_lds_batched", "failed_basis_keeps_the_installed_one",
                                   "band_passes", "zeroed_memory", "large_videos", "video_sums", "image_sums", "match_forms",
                                   "large_cubes", "without_memory_for_the_fastest_tiles"])
def test_launches(check):
    fake_hip.run("launch_checks", check + "()")
