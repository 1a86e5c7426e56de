"""The dispatch rules of the fp32 kernels, evaluated on the host at both sides of their lines (no GPU: a program that includes the
kernels' header and launches nothing)."""
import os
import subprocess

import pytest

from paper_2409_15373_amd import build

PROGRAM = """
#include <cstdio>
#include "jfa_common.h"
int main() {
    long long rows, B, max_len, H, max_streamed;
    while (scanf("%lld %lld %lld %lld %lld", &rows, &B, &max_len, &H, &max_streamed) == 5)
        printf("%d\\n", jfa::f32_direct_blocks(jfa::F32Form{false, (int)rows}, B, max_len, (int)H, max_streamed, 256));
}
"""


@pytest.fixture(scope="module")
def direct_blocks(tmp_path_factory):
    """(rows per block, B, max_len, H, longest stream) -> blocks per (sample, head) of a call without a schedule, 0: it has one."""
    if not os.path.exists(build.HIPCC):
        pytest.skip("needs hipcc")
    where = tmp_path_factory.mktemp("dispatch")
    source, program = str(where / "rule.hip"), str(where / "rule")
    with open(source, "w") as f:
        f.write(PROGRAM)
    subprocess.run([build.HIPCC, "--offload-arch=gfx950", "-std=c++17", "-w", "-I", build.CSRC, source, "-o", program], check=True)

    def ask(*calls):
        text = "\n".join(" ".join(map(str, c)) for c in calls)
        return [int(x) for x in subprocess.run([program], input=text, capture_output=True, text=True, check=True).stdout.split()]
    return ask


def test_a_launch_without_a_schedule_fits_a_grid(direct_blocks):
    """A grid's threads are counted in 32 bits: 2^22 workgroups of 64 or 256 threads are a launch, what is beyond has a schedule and a
    grid of the chip's size, up to the 2^30 samples that the entry points admit."""
    line = 1 << 22
    assert direct_blocks((32, line, 20, 1, 20), (32, line // 8, 32, 8, 32), (64, line // 8, 64, 8, 64)) == [1, 1, 1]
    beyond = [(32, line + 1, 20, 1, 20), (32, line // 8 + 1, 32, 8, 32), (64, line // 8 + 1, 64, 8, 64), (32, 1 << 26, 20, 1, 20),
              (64, 1 << 21, 64, 8, 128), (32, (1 << 30) - 1, 1, 1, 1)]
    assert direct_blocks(*beyond) == [0] * len(beyond)


def test_longer_streams_keep_their_order(direct_blocks):
    """One block per sample is no reason to give up the order, longest first, where more than 64 rows stream past it and there are more
    blocks than compute units."""
    assert direct_blocks((64, 2000, 64, 4, 65), (64, 3000, 64, 4, 128), (32, 300, 32, 4, 100)) == [0, 0, 0]
    assert direct_blocks((32, 3000, 30, 4, 64), (64, 200, 64, 4, 64), (64, 64, 64, 4, 128), (64, 64, 64, 4, 1000)) == [1, 1, 1, 1]
