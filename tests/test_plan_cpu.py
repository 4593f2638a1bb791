"""Plans of the attend call, on the CPU: a small host program against the library's own planner."""
import os
import subprocess

import pytest

from paper_2512_17917_amd import build as B

PROBE = r"""
#include <cstdio>
#include "kvr_launch.h"
// per input line: units heads rows slots retained vague -> side-by-side fits, LDS of the staged and the retained kernel,
// parts of a streamed list
int main() {
  int units, G, r, w, ret, vague;
  while (std::scanf("%d %d %d %d %d %d", &units, &G, &r, &w, &ret, &vague) == 6) {
    kvr::DevDesc d = {};
    d.B = 1; d.Hkv = units; d.Hq = units * G; d.G = G; d.r = r; d.w = w; d.sign_mask = 2;
    const kvr::AttendPlan p = kvr::attend_plan(d, KVR_BF16, ret, vague);
    std::printf("%d %d %d %d\n", (int)kvr::attend_side_fits(d, p), p.lds_bytes,
                kvr::retained_lds(G, p.rslice_tokens, true), p.streamed ? p.n_vslices : 0);
  }
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, exe = str(d / "probe.hip"), str(d / "probe")
    open(src, "w").write(PROBE)
    subprocess.run([B._hipcc(), "--offload-host-only", "-std=c++17", "-I", B.CSRC, src, "-L", os.path.dirname(B.OUT),
                    "-l:" + os.path.basename(B.OUT), f"-Wl,-rpath,{os.path.dirname(B.OUT)}", "-o", exe], check=True, capture_output=True)

    def ask(*rows):
        text = "".join(" ".join(map(str, x)) + "\n" for x in rows)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]
    return ask


@pytest.mark.parametrize("units", [64, 128, 192, 512])
def test_retained_kernel_fits_next_to_a_staged_one(plan, units):
    """Whatever the slices of the retained slots: beside the 64-channel kernel up to 312 slots per row with four heads
    (120 KB of chunk + 34 KB + 8.1 KB), and beside the three-row 16-channel kernel at every width it takes."""
    case = lambda G, w: (units, G, 3, w, 27 * w, 93 * w)
    for w, fits in [(6, 1), (273, 1), (291, 1), (300, 1), (312, 1), (313, 0), (333, 0), (334, 1), (700, 1), (1365, 1)]:
        ok, staged, ret, _ = plan(case(4, w))[0]
        assert ok == fits and (staged + ret + 128 <= 160 * 1024) == bool(fits), (w, staged, ret)
    assert all(p[0] for p in plan(*[case(1, w) for w in (300, 341, 342, 1365)]))


@pytest.mark.parametrize("units", [1, 3, 8, 40, 128, 129, 200, 256, 300])
def test_streamed_list_takes_one_turn_of_the_chip(plan, units):
    """Eight heads: as many parts as fit 256 workgroups, none below 256 tokens, none missing."""
    for vague in (64, 256, 257, 511, 1000, 5003, 25395, 130000):
        parts = plan((units, 8, 3, 60, 187, vague))[0][3]
        most = max(1, min(256 // units, -(-vague // 256)))
        assert 1 <= parts <= most and (parts == 1 or units * parts <= 256)
        tokens = -(-max(256, -(-vague // most)) // 16) * 16
        assert parts == -(-vague // tokens)
