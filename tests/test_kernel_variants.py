"""Settings of the launch shape that select a kernel have one in the library."""
import pytest

from paper_1906_03065_amd import build


@pytest.mark.parametrize("storage", ["6__half", "14__hip_bfloat16"])
@pytest.mark.parametrize("kernel", ["11k_lb2d_ring", "16k_lb2d_ring_part"])
@pytest.mark.parametrize("ring", [3, 4])
@pytest.mark.parametrize("lanes", [64, 128, 192, 256])
def test_lanes_and_ring_of_the_16bit_march(lanes, ring, kernel, storage):
    with open(build.LIB, "rb") as f:
        names = f.read()
    for form in (0, 1):
        waves = 2 if form or ring == 4 else 3
        tag = f"{kernel}INS_12Split16StoreI{storage}Li9EEEfLi{lanes}ELi{ring}ELi{waves}ELi{form}EE".encode()
        assert tag in names, tag
