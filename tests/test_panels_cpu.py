"""The panel sweep's reads of the CSR stay in bounds: its source, on the CPU."""
import os
import re
import shutil
import subprocess

import pytest

KERNELS = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2210_01465_amd", "csrc",
                       "fl_kernels.hip")


def function(name: str) -> str:
    """The definition of a function of the kernel source, without comments."""
    text = re.sub(r"//[^\n]*", "", open(KERNELS).read())
    start = text.rindex("\n", 0, re.search(r"\b%s\(" % name, text).start()) + 1
    at, depth = text.index("{", start), 0
    while True:
        depth += {"{": 1, "}": -1}.get(text[at], 0)
        at += 1
        if depth == 0:
            return text[start:at]


# One lane at a time; a buffer load checks its vector offset against the
# descriptor's bytes and returns 0 past them, and adds the scalar offset
# unchecked.
LANES = r"""
#include <stdint.h>
#include <stdio.h>
#include <algorithm>
using std::max; using std::min;
#define __device__
#define __forceinline__ inline
constexpr int kPanelBlock = 512, kLongRows = 4;
struct PanelRows { int32_t begin[kPanelBlock], end[kPanelBlock]; float acc[kPanelBlock]; };
struct { int x; } threadIdx;
bool outside;
struct __amdgpu_buffer_rsrc_t { const int32_t *base; uint32_t bytes; };
__amdgpu_buffer_rsrc_t __builtin_amdgcn_make_buffer_rsrc(void *p, short, int bytes, int) {
    return {(const int32_t *)p, (uint32_t)bytes};
}
int32_t __builtin_amdgcn_raw_buffer_load_b32(__amdgpu_buffer_rsrc_t r, int v, int s, int) {
    if ((uint32_t)v + 4 > r.bytes) return 0;
    const int64_t at = (v + s) / 4;   // within the row?
    if (at < 0 || at >= (int64_t)(r.bytes / 4)) outside = true;
    return 0;
}
#define __builtin_amdgcn_readfirstlane(x) (x)
template <int L> float row_sum(float x) { return x; }
FUNCTION
int main() {
    int32_t len, data[4096] = {};
    float x[1] = {1.0f};
    while (scanf("%d", &len) == 1) {   // three rows of len edges
        PanelRows p;
        outside = false;
        for (int r = 0; r < 3; ++r) p.begin[r] = r * len, p.end[r] = (r + 1) * len;
        for (threadIdx.x = 0; threadIdx.x < 64; ++threadIdx.x) panel_sums_long(p, data, x, 3);
        printf("%d %d\n", len, (int)outside);
    }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_long_rows_read_their_own_edges_only(tmp_path):
    src, exe = tmp_path / "lanes.cpp", tmp_path / "lanes"
    src.write_text(LANES.replace("FUNCTION", function("panel_sums_long")))
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", str(src), "-o", str(exe)], check=True)
    lens = [0, 1, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 191, 192, 200, 255, 256, 257, 700]
    out = subprocess.run([str(exe)], input=" ".join(map(str, lens)), capture_output=True, text=True, check=True).stdout
    assert [int(line.split()[1]) for line in out.splitlines()] == [0] * len(lens), out


def test_the_waves_of_a_workgroup_leave_together():
    """Every wave stores the bounds of rows that other waves gather, and the
    first workgroup of a launch may set the stop flag while others start: a
    wave may not leave, before a barrier, on a reading of its own."""
    head = function("k_pr_iter_panels").split("__syncthreads")[0]
    assert "peek_stop" in head and "return" not in head
