"""Dynamic LDS of the bulk insert's launches, on the CPU: a host program that puts its own launch calls and
hipFuncSetAttribute before the runtime's, so that nothing is launched and every launch is listed.  A kernel may ask for more
than 64 KB only where its limit was raised for it."""
import os
import subprocess

import pytest

from paper_2512_17917_amd import build as B

PROBE = r"""
#include <cstdio>
#include <map>
#include "kvr_launch.h"
static size_t asked;
static std::map<const void*, int> limit;
extern "C" hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute a, int value) {
  if (a == hipFuncAttributeMaxDynamicSharedMemorySize) limit[f] = value;
  return hipSuccess;
}
extern "C" hipError_t hipLaunchKernel(const void* f, dim3, dim3, void**, size_t lds, hipStream_t) {
  std::printf(" %zu:%d", lds, limit.count(f) ? limit[f] : 65536);
  return hipSuccess;
}
extern "C" hipError_t __hipPushCallConfiguration(dim3, dim3, size_t lds, hipStream_t) { asked = lds; return hipSuccess; }
extern "C" hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* st) {
  *g = dim3(1); *b = dim3(1); *lds = asked; *st = nullptr;
  return hipSuccess;
}
extern "C" hipError_t hipGetLastError() { return hipSuccess; }
// per input line: units rows slots tokens -> the launches' LDS and limits
int main() {
  int units, r, w, cap;
  while (std::scanf("%d %d %d %d", &units, &r, &w, &cap) == 4) {
    kvr::DevDesc d = {};
    d.B = 1; d.Hkv = d.Hq = units; d.G = 1; d.r = r; d.w = w;
    int32_t x = 0;                           // no kernel runs: never read
    const kvr::EncodePlan plan = kvr::encode_plan(d, cap);
    const hipError_t e = kvr::launch_encode(d, KVR_BF16, &x, &x, 1, &x, &x, &x, cap, &x, &x, nullptr, nullptr, &x, plan, nullptr);
    std::printf(" %d\n", (int)e);
  }
}
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    tmp_path = tmp_path_factory.mktemp("launches")
    src, exe = str(tmp_path / "probe.hip"), str(tmp_path / "probe")
    open(src, "w").write(PROBE)
    subprocess.run([B._hipcc(), "--offload-host-only", "-std=c++17", "-I", B.CSRC, src, "-L", os.path.dirname(B.OUT),
                    "-l:" + os.path.basename(B.OUT), f"-Wl,-rpath,{os.path.dirname(B.OUT)}", "-o", exe], check=True, capture_output=True)

    def ask(cases):
        out = subprocess.run([exe], input="".join(" ".join(map(str, c)) + "\n" for c in cases), capture_output=True, text=True, check=True).stdout
        assert len(out.splitlines()) == len(cases)
        for case, line in zip(cases, out.splitlines()):
            *launches, rc = line.split()
            assert rc == "0" and len(launches) == 3, (case, line)          # slot numbers, sort, sums
            yield case, [tuple(map(int, x.split(":"))) for x in launches]
    return ask


def test_bulk_insert_stays_within_its_lds_limit(launches):
    cases = [(2, 3, w, cap) for w in (1, 29, 273, 511, 4000, 5120, 7680, 8191, 8192) for cap in (65, 2000, 24575, 24576, 40000, 1 << 20)]
    # lists first that take the plain kernel: no limit was raised by an earlier call
    cases.sort(key=lambda c: -c[3])
    for case, asked in launches(cases):
        assert all(lds <= limit <= 160 * 1024 for lds, limit in asked), (case, asked)


def test_sort_of_few_waves_leaves_a_cu_room(launches):
    """The records of a list that fits go to LDS beside the table from seven waves on; with fewer, other workgroups have to find
    room on the CU: the table alone, whatever the list's length."""
    for (_, _, w, cap), asked in launches([(128, 3, w, cap) for w in (273, 1920, 1921, 2560, 4000, 8192) for cap in (1000, 20000)]):
        waves = min(16, max(1, (15360 - w) // w))
        table = (waves + 1) * w * 4
        assert asked[1][0] == (table + 4 + 4 * cap if waves >= 7 else table), (w, cap, asked)
