"""What the traversal kernels keep in LDS: every wave's part lies inside the
bytes the launch asks for and apart from the other waves' (no barrier stands
between them), and the kernels that give a group of lanes to a ray store
nothing there but their stacks: the staging ring of the other path lies in
the same bytes, or past the end of a grouped launch's."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2001_09792_amd", "csrc")
LIB = os.path.join(ROOT, "paper_2001_09792_amd", "librg.so")
OBJDUMP = os.environ.get("LLVM_OBJDUMP", "/opt/rocm/llvm/bin/llvm-objdump")

LAYOUT = r"""
#include "trace_lds.h"
#include <cstdio>
using namespace rgt;
static int check(size_t begin, size_t end, size_t before, size_t total) {
    return begin < before || end <= begin || end > total;
}
int main() {
    int bad = 0;
    const int waves = kThreads / 64, depths[] = {8, 9, 16, 31, kMaxLdsStack};
    for (int K = 0; K <= 3; ++K)
        for (int depth : depths) {
            const size_t total = lanes_bytes(K, depth);
            size_t before = (size_t)depth * kThreads * 4;  // the lanes' stacks: entry e of thread t at e * kThreads + t
            for (int w = 0; w < waves; ++w) {
                bad += check(ring_at(K, depth, w), ring_at(K, depth, w) + ring_bytes(K), before, total);
                bad += ring_at(K, depth, w) % 8 != 0;  // its masks are 8-byte words
                before = ring_at(K, depth, w) + ring_bytes(K);
            }
        }
    for (int W = 4; W <= 8; W *= 2) {
        size_t before = 0;
        for (int w = 0; w < waves; ++w) {
            const size_t at = group_stacks_at(W, w), end = at + (size_t)(64 / W) * kStackCap * 4;
            bad += check(at, end, before, groups_bytes(W));
            before = end;
        }
    }
    // a lane's entries, in LDS and private memory, are as many as a group's
    for (int depth : depths) bad += depth + kPrivStack < kStackCap;
    std::printf("%d\n", bad);
    return bad != 0;
}
"""


def test_parts_are_apart_and_inside(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if not cxx:
        pytest.skip("no host compiler")
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text(LAYOUT)
    subprocess.check_call([cxx, "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)])
    assert subprocess.run([str(exe)], capture_output=True, text=True).stdout == "0\n"


def _kernels(tmp_path):
    """The traversal kernels in the built library: template arguments -> LDS store instructions."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(LIB, tmp_path)
    subprocess.check_call([OBJDUMP, "--offloading", lib], stdout=subprocess.DEVNULL, cwd=tmp_path)
    found = {}
    for name in sorted(os.listdir(tmp_path)):
        path = os.path.join(tmp_path, name)
        if not name.endswith("gfx950") or os.path.getsize(path) == 0:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", path], capture_output=True, text=True,
                              check=True).stdout
        kernel = None
        for line in text.splitlines():
            head = re.match(r"^[0-9a-f]+ <(.*)>:$", line)
            if head:
                args = re.search(r"k_traceILi(\d)ELb(\d)ELi(\d)ELb(\d)ELi(\d)EE", head.group(1))
                kernel = tuple(int(v) for v in args.groups()) if args else None
                if kernel:
                    found[kernel] = []
            elif kernel:
                op = re.match(r"\s+(ds_(?!read|bpermute|permute|swizzle)\w+)", line)
                if op:
                    found[kernel].append(op.group(1))
    return found


def test_grouped_kernels_store_their_stacks_alone(tmp_path):
    kernels = _kernels(tmp_path)
    grouped = {k: v for k, v in kernels.items() if k[4] == 1}
    # closest and any hit of trace calls and frames, with and without options, widths 4 and 8
    assert len(grouped) == 16
    for k, stores in grouped.items():
        assert stores == ["ds_write_b32"], (k, stores)
    # the search does see the ring: its masks are set up, merged and cleared by 8-byte words
    for k, stores in kernels.items():
        if k[4] != 1 and k[2] != 1:
            assert "ds_write_b64" in stores and "ds_or_b64" in stores, (k, stores)
