"""Plans of the attend call, on the CPU: a small host program against the library's own planner."""
import os
import subprocess

import pytest

from paper_2512_17917_amd import build as B

PROBE = r"""
#include <cstdio>
#include "kvr_launch.h"
// per input line: units heads rows slots retained vague -> LDS of the retained kernel next to the staged one (0: not side
// by side), of the staged kernel, of the retained kernel alone,
// parts of the Vague list, channels per phase of the staged kernel (0: the list is not staged); then slices of the retained
// slots and their tokens, workgroups for them in the list's launch, LDS of that launch (0: a launch of their own), tokens that
// the parts hold at most, bytes of workspace, 1 if the slots of a plan for one launch have one of their own after all
int main() {
  int units, G, r, w, ret, vague;
  while (std::scanf("%d %d %d %d %d %d", &units, &G, &r, &w, &ret, &vague) == 6) {
    kvr::DevDesc d = {};
    d.B = 1; d.Hkv = units; d.Hq = units * G; d.G = G; d.r = r; d.w = w; d.sign_mask = 2;
    const kvr::AttendPlan p = kvr::attend_plan(d, KVR_BF16, ret, vague);
    const long long part = p.streamed ? p.vslice_tokens : p.ch == 64 ? 512 * kvr::STAGED64_KMAX : 512 * kvr::staged16_kmax(r);
    std::printf("%d %d %d %d %d %d %d %d %d %lld %zu %d\n", kvr::attend_side_lds(d, p), p.lds_bytes,
                kvr::retained_lds(G, p.rslice_tokens), p.n_vslices, p.staged ? p.ch : 0, p.n_rslices, p.rslice_tokens,
                p.pair ? p.n_ret_wgs : p.streamed ? p.stream.n_ret_wgs : 0, p.pair ? p.pair_lds : p.streamed ? p.stream.lds : 0,
                part * p.n_vslices, p.total_bytes, p.pair ? p.ret_own : p.streamed ? p.stream.own : 0);
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
    (120 KB of chunk + 34 KB + 8.1 KB), and beside the three-row 16-channel kernel at every width it takes; with the logits
    of a whole slice where there is room, else with those of the 512 tokens that fit its sums' place."""
    case = lambda G, w: (units, G, 3, w, 27 * w, 93 * w)
    for w, fits in [(6, 1), (273, 1), (291, 1), (300, 1), (312, 1), (313, 0), (333, 0), (334, 1), (700, 1), (1365, 1)]:
        side, staged, alone = plan(case(4, w))[0][:3]
        assert (side > 0) == bool(fits) and (staged + 8192 + 128 <= 160 * 1024) == bool(fits), (w, staged, side)
        assert side in ((alone, 8192) if fits else (0,)) and staged + side + 128 <= 160 * 1024
        assert side == alone or staged + alone + 128 > 160 * 1024 - 2 * 1280
    assert all(p[0] for p in plan(*[case(1, w) for w in (300, 341, 342, 1365)]))


def test_registers_next_to_a_staged_kernel(plan):
    """Four rows: 238 registers a wave in the 16-channel kernel, 194 and more in the general one with four heads; two
    waves of those leave no 128.  Everything else does, LDS permitting."""
    ok = [int(p[0] > 0) for p in plan((128, 4, 4, 819, 9000, 30000), (128, 1, 4, 300, 9000, 30000), (128, 4, 4, 1100, 9000, 30000),
                             (128, 2, 4, 1100, 9000, 30000), (128, 1, 4, 1030, 9000, 30000), (128, 4, 3, 1400, 9000, 30000),
                             (128, 8, 3, 60, 9000, 30000))]
    assert ok == [0, 0, 0, 1, 1, 1, 0]


@pytest.mark.parametrize("units", [1, 3, 8, 40, 128, 129, 200, 256, 300])
def test_streamed_list_takes_one_turn_of_the_chip(plan, units):
    """Eight heads: as many parts as fit 256 workgroups, none below 256 tokens, none missing."""
    for vague in (64, 256, 257, 511, 1000, 5003, 25395, 130000):
        parts = plan((units, 8, 3, 60, 187, vague))[0][3]
        most = max([1] + [n for n in range(2, 256 // units + 1) if -(-vague // n) >= 256])
        assert 1 <= parts <= most and (parts == 1 or units * parts <= 256)
        tokens = -(-max(256, -(-vague // most)) // 16) * 16
        assert parts == -(-vague // tokens)


@pytest.mark.parametrize("G,r,edges", [(4, 3, [(333, 64), (334, 16), (1365, 16), (1366, 16), (1685, 16), (1686, 8), (2666, 8), (2667, 0)]),
                                       (4, 4, [(1, 16), (1024, 16), (1025, 16), (1264, 16), (1265, 8), (2000, 8), (2001, 0)]),
                                       (2, 3, [(341, 64), (342, 16)]),
                                       (1, 4, [(1272, 16), (1273, 8), (2108, 8), (2109, 0)])])
def test_channels_per_phase(plan, G, r, edges):
    """The widest chunk whose LDS (chunk, statistics, q and nothing else) fits a workgroup's 160 KB; 8 channels up to
    8000 rows with four heads, 8432 with one."""
    for w, ch in edges:
        p = plan((16, G, r, w, 1000, 9000))[0]
        assert p[4] == ch and p[1] <= 160 * 1024, (w, p)
        if ch and r * w > 4096:
            assert p[1] == -(-r * w * ch * 2 // 1024) * 1024 + 2 * 32 * G * 4 + G * 256


@pytest.mark.parametrize("batch,ret_cap,vague_cap", [(1, 187, 64), (5, 4104, 12307), (8, 7374, 25395)])
def test_workspace_of_a_streamed_list(batch, ret_cap, vague_cap):
    """The streaming kernel's logits lie by tile and nowhere else: a listed token takes a record and one float per column (in
    kvr_attend_multi within its two rebuilt rows), a retained slot one float per column, and the rest are partial results."""
    import ctypes as C

    from paper_2512_17917_amd import binding as kvr
    units, areas = batch * 8, 6 * 256
    partials = lambda col, total: total % (units * col * 130 * 4) if total > 0 else -1           # [slices, col, 128 + 2] floats a unit
    list4 = (vague_cap + 3) // 4 * 4
    for heads, n_q in ((8, 0), (4, 4), (2, 2)):
        d = kvr.make_desc(batch, 8 * heads, 8, 3, 60, kvr.KVR_BF16, seed=1)
        col = heads * max(n_q, 1)
        if n_q:
            size = kvr.kvr_attend_multi_workspace_size(d, n_q, ret_cap, vague_cap)
            fixed = units * (2 * vague_cap * 256 + ret_cap * col * 4)
        else:
            size = kvr.kvr_workspace_size(d, kvr.KVR_OP_ATTEND, ret_cap, vague_cap)
            fixed = units * (list4 * (4 + col * 4) + ret_cap * col * 4)
        left = size - fixed                                    # whole partials and what the areas are rounded up by
        assert 0 < left and partials(col, left) <= areas, (heads, n_q, size, fixed)
        slices = left // (units * col * 130 * 4)
        assert slices <= -(-1536 // units) + 256 // units + 1 + (ret_cap + 127) // 128, slices


@pytest.mark.parametrize("G,r,w", [(1, 3, 100), (4, 3, 333), (4, 3, 700), (1, 4, 400), (4, 4, 819), (8, 3, 60)])
def test_one_launch_up_to_the_largest_sizes(plan, G, r, w):
    """Kernels that take the slots along, up to the sizes that the calls take (65535 units, 2^30 tokens: the question for a
    workspace reads no memory).  Slots and list are covered, the launch has workgroups for the slots in whole eights and fits
    LDS, and the workspace holds its parts."""
    cases = [(units, G, r, w, ret, vague) for units in (1, 9, 640, 4100, 65535) for ret in (1, 5000, 1 << 20, 1 << 30)
             for vague in (64, 40000, 1 << 22, 1 << 28, 1 << 30)]
    for (units, _, _, _, ret, vague), p in zip(cases, plan(*cases)):
        parts, slices, tokens, wgs, lds, listed, size, own = p[3], *p[5:]
        assert parts >= 1 and listed >= vague and slices * tokens >= ret > (slices - 1) * tokens, (units, ret, vague, p)
        assert (wgs == 0 if own else 8 <= wgs <= 256) and wgs % 8 == 0 and 0 < lds <= 160 * 1024, (units, ret, vague, p)
        assert size >= units * G * ((slices + parts) * 130 * 4 + (ret if G == 8 else ret + vague) * 4), (units, ret, vague, p)


@pytest.mark.parametrize("G,r,w", [(8, 3, 21), (4, 3, 53), (1, 3, 1), (4, 4, 20)])
def test_slots_are_not_left_a_few_cus(plan, G, r, w):
    """Lists that leave hardly a CU (246 units fill 31 of an XCD's 32): the slots of all units would be walked there one after
    another.  The slots of a launch take less than twice as many turns as on all CUs, or no longer than the list's workgroups."""
    cases = [(units, G, r, w, ret, vague) for units in (192, 224, 246, 300, 400, 512) for ret, vague in
             ((7, 220), (72, 216), (585, 1755), (1441, 4325), (3000, 800), (7000, 1400))]
    for (units, _, _, _, ret, vague), p in zip(cases, plan(*cases)):
        slices, tokens, wgs, own = p[5], p[6], p[7], p[11]
        if own:
            assert wgs == 0 and ret <= (256 if G == 8 else 64)
            continue
        turns = -(-units * slices // wgs)
        assert wgs >= 32 and turns * tokens <= 8 * 1024 + 16 * vague, (units, ret, vague, p)


SLOTS_AHEAD = [                              # units, heads, rows, slots per row, retained, listed
    (246, 4, 3, 21, 585, 1755, "first"),
    (128, 1, 3, 18, 507, 5108, "first"),
    (128, 4, 4, 20, 2025, 6975, "first"),
    (400, 4, 3, 1, 7, 220, "own"),
    (400, 2, 3, 2, 64, 300, "own"),
    (200, 4, 3, 6, 10112, 300, "lds"),       # one slice of all that LDS holds
    (200, 4, 3, 6, 10113, 300, "lds"),
    (246, 8, 3, 21, 585, 1755, "first"),
    (400, 8, 3, 1, 30, 220, "own"),
    (512, 8, 3, 4, 250, 1000, "own"),
]


@pytest.mark.parametrize("units,G,r,w,ret,vague,how", SLOTS_AHEAD)
def test_slots_ahead_of_the_list(plan, units, G, r, w, ret, vague, how):
    """first: workgroups for the slots on all CUs (at most one per slice, in whole eights); own: none in the list's launch."""
    p = plan((units, G, r, w, ret, vague))[0]
    slices, wgs, lds, own = p[5], p[7], p[8], p[11]
    assert own == (how == "own") and (wgs == 0) == (how == "own")
    assert how != "first" or wgs == min(256, -(-units * slices // 8) * 8)
    assert how != "lds" or (slices == 1 and lds > 155 * 1024) == (ret <= 10112)


SIDE_BY_SIDE = [                             # units, heads, rows, slots per row, retained, listed
    (128, 4, 3, 1400, 9500, 9400, "whole"),  # the retained kernel's capped form keeps the logits of a slice of 960 tokens
    (129, 4, 3, 1550, 6001, 9400, "whole"),  # 640, the last one 241
    (128, 2, 4, 1200, 9500, 9400, "whole"),
    (128, 4, 3, 1550, 9500, 9400, "parts"),  # of 512 tokens at a time
    (128, 2, 4, 1230, 9500, 9400, "parts"),
    (128, 1, 3, 1670, 9501, 9400, "parts"),
]


@pytest.mark.parametrize("units,G,r,w,ret,vague,how", SIDE_BY_SIDE)
def test_calls_that_fork(plan, units, G, r, w, ret, vague, how):
    """The general staged kernel, in more than two turns of the chip, with room for the retained kernel on a CU."""
    p = plan((units, G, r, w, ret, vague))[0]
    side, staged, alone, parts, ch, slices, tokens, wgs, lds = p[:9]
    assert ch == 16 and wgs == 0 and lds == 0 and units * parts >= 512 and staged + side + 128 <= 160 * 1024
    assert tokens > 512 and side == (alone if how == "whole" else 4 * G * 512) <= alone and (how == "whole") == (side == alone)


@pytest.mark.parametrize("units", [4, 12, 42, 60])
def test_parts_of_a_streamed_list_leave_the_slots_room(plan, units):
    """From 256 slots on: a unit's parts share an XCD of 32 CUs and fit it in one turn."""
    for ret, vague in ((300, 3000), (400, 12000), (510, 9000)):
        parts = plan((units, 8, 3, ret // 30, ret, vague))[0][3]
        assert -(-units // 8) * parts <= 32, (units, ret, vague, parts)


def test_slots_of_many_units_have_more_cus(plan):
    """Where workgroups would walk six slices or more (80 and 56 of them), beside the streaming kernel three, more CUs are taken
    from the list."""
    for case, least in (((512, 1, 3, 53, 1441, 4325), 128), ((400, 4, 3, 53, 1441, 4325), 80), ((400, 8, 3, 21, 585, 1755), 120),
                        ((320, 8, 3, 111, 3000, 900), 160), ((144, 8, 3, 341, 11000, 2800), 160)):
        assert plan(case)[0][7] >= least, case
