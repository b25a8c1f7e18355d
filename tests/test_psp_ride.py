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


# (tokens, K, rank), rides; microseconds of the rotation with the projection: riding, in a launch of its own
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
