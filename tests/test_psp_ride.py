"""Host-side check of the projection's place (csrc/psp_ride.h, compiled by itself): in the rotation's launch or in one of
its own, at shapes where both were measured."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_00422_amd", "csrc")
DRIVER = """
#include <cstdio>
#include "psp_ride.h"
int main() {
    long long M, K, riders;
    int planes, f32;
    while (scanf("%lld %lld %lld %d %d", &M, &K, &riders, &planes, &f32) == 5) printf("%d\\n", psp_rides(M, K, riders, 256, planes, f32));
}
"""


@pytest.fixture(scope="module")
def rides(tmp_path_factory):
    d = tmp_path_factory.mktemp("ride")
    (d / "ride.cpp").write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(d / "ride"), str(d / "ride.cpp")], check=True)

    def run(M, K, r, f32, planes=False):
        tiles = (r + 15) // 16                          # column groups of two such tiles, where there are more
        riders = (M + 15) // 16 * ((K + 511) // 512) * ((tiles + 1) // 2 if tiles > 2 else 1)
        out = subprocess.run([str(d / "ride")], input=f"{M} {K} {riders} {int(planes)} {int(f32)}\n", text=True,
                             capture_output=True, check=True).stdout
        return out.strip() == "1"

    return run


# (tokens, K, rank), rides; microseconds of the rotation with the projection: riding, in a launch of its own, with the rotations of
# rotate_bf16_device.h and rotate_f32_device.h (those by strips: csrc/psp_ride.h).  The library asks the rule only of calls that no
# walking rotation takes.
@pytest.mark.parametrize("shape,want", [
    ((192, 5120, 37), True),                    # 13.9, 26.7
    ((320, 5120, 37), True),                    # 21.6, 32.4
    ((384, 4096, 37), True),                    # 18.5, 27.2
    ((256, 4096, 64), True),                    # 15.4, 23.4
    ((173, 8192, 64), True),                    # 25.2, 33.2
    ((192, 11008, 37), True),                   # 45.3, 55.8
    ((333, 4096, 32), True),
    ((257, 25600, 8), True),                    # by the shadow alone: the whole layer 174, 154
    ((384, 512, 64), True),
    ((769, 4096, 8), False),
    ((650, 1024, 64), False),                   # 814 workgroups
])
def test_fp32_tokens(rides, shape, want):
    assert rides(*shape, f32=True) == want


@pytest.mark.parametrize("shape,want", [
    ((128, 8192, 64), True),                    # 16.7, 21
    ((255, 8192, 64), False),                   # 29.8, 22.7
    ((128, 25600, 32), True),                   # 28.3, 34
    ((257, 5120, 32), True),                    # 16.8, 23
    ((192, 5120, 37), False),
    ((384, 512, 64), True),                     # 11.7, 18.5
])
def test_bf16_tokens(rides, shape, want):
    assert rides(*shape, f32=False) == want
    assert not rides(*shape, f32=False, planes=True)


SLOW = DRIVER.replace('%d %d", &M', '%d %d %d", &M').replace("int planes, f32;", "int planes, f32, slow;").replace(
    "&f32) == 5", "&f32, &slow) == 6").replace("planes, f32))", "planes, f32, slow))")


# (tokens, n1, n2, rank): bf16 tokens whose rotation takes longer than its row is long; microseconds: riding, in a launch of its own
@pytest.mark.parametrize("shape,want", [
    ((185, 172, 64, 8), True),                  # 30.4, 35.8
    ((185, 192, 64, 8), True),                  # 30.9, 34.9
    ((185, 256, 48, 8), True),                  # 34.6, 38.9
    ((185, 200, 80, 8), True),                  # 41.4, 47.1
    ((158, 163, 32, 64), True),                 # 26.1, 34.4
    ((400, 163, 32, 8), True),                  # 49.0, 56.1
    ((158, 172, 64, 64), True),                 # 34.7, 36.9
    ((230, 172, 64, 8), False),                 # 41.0, 35.8
    ((230, 200, 80, 8), False),                 # 54.1, 48.2
    ((230, 163, 32, 64), False),                # 37.8, 35.7
    ((400, 172, 64, 8), True),                  # 57.8, 62.6
    ((520, 200, 80, 8), True),                  # 117.7, 125.5
])
def test_tokens_of_slow_rotations(tmp_path, shape, want):
    (tmp_path / "ride.cpp").write_text(SLOW)
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-o", str(tmp_path / "ride"), str(tmp_path / "ride.cpp")], check=True)
    M, n1, n2, r = shape
    tiles, K = (r + 15) // 16, n1 * n2
    riders = (M + 15) // 16 * ((K + 511) // 512) * ((tiles + 1) // 2 if tiles > 2 else 1)
    out = subprocess.run([str(tmp_path / "ride")], input=f"{M} {K} {riders} 0 0 1\n", text=True, capture_output=True, check=True).stdout
    assert (out.strip() == "1") == want
