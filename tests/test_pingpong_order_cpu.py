"""The order of LDS accesses in the main loop of the bf16 MFMA products
(csrc/pingpong.h), checked on the CPU: the loop is compiled for the host with
its builtins replaced by functions that record one early and one late wave's
loads, LDS reads, waits, barriers and uses.  Between two barriers the waves run
in any order, so every relation between two waves has to follow from the
barriers and the explicit waits alone:

  * a unit is read only after every wave has waited for its own part of it;
  * a unit is overwritten only after every wave's reads of it have returned;
  * every product is of the same stage's halves, each taken once.
"""

import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER = os.path.join(ROOT, "paper_2506_20194_amd", "csrc", "pingpong.h")

COMMON = r"""
#pragma once
#include <cstdint>
#include <cstdio>
#include <cstring>
#define __device__
#define __forceinline__ inline
struct u32x4 { uint32_t v[4]; };
struct bf16x8 { uint32_t v[4]; };
struct f4 { float v[4]; };
struct { unsigned x; } threadIdx;
inline f4 use(const bf16x8& a, const bf16x8& b, f4 c) { printf("M %u %u\n", a.v[0], b.v[0]); return c; }
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, x, y, z) use(a, b, c)
#define __builtin_amdgcn_s_barrier() puts("B")
#define __builtin_amdgcn_s_waitcnt(i) printf("W %d %d\n", ((i) & 15) | (((i) >> 14 & 3) << 4), (i) >> 8 & 15)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_s_setprio(x) ((void)0)
"""

MAIN = r"""
#include "pingpong.h"
using namespace duo;
constexpr int HA = P_HA, LA = P_LA, LB = P_LB, NST = P_NST;
int main() {
  for (int w = 0; w < 2; ++w) {
    printf("wave\n");
    threadIdx.x = 256 * w;
    uint32_t id = 0;
    f4 acc[2 * HA][4] = {};
    auto issue = [](int op, int st, int par) { printf("I %d %d %d\n", op, st, par); };
    auto read_a = [&](int par, int h, u32x4 (&F)[2][HA]) {
      printf("R %u %d %d %d\n", ++id, h, par, 2 * HA);
      for (auto& s : F) for (auto& f : s) f.v[0] = id;
    };
    auto read_b = [&](int par, int h, u32x4 (&F)[2][2]) {
      printf("R %u %d %d %d\n", ++id, 2 + h, par, 4);
      for (auto& s : F) for (auto& f : s) f.v[0] = id;
    };
    pp::pp_loop<HA, LA, LB>(NST, acc, issue, read_a, read_b);
  }
}
"""


def _trace(tmp_path, ha, la, lb, nst):
    text = open(HEADER).read()
    text, n = re.subn(r'asm volatile\("s_nop[^;]*;', ";", text)
    assert n == 1
    (tmp_path / "pingpong.h").write_text(text)
    (tmp_path / "common.h").write_text(COMMON)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "trace")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", f"-DP_HA={ha}", f"-DP_LA={la}", f"-DP_LB={lb}", f"-DP_NST={nst}",
                    str(tmp_path / "main.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout
    return [[l.split() for l in w.strip().split("\n")] for w in out.split("wave\n")[1:]]


class Wave:
    """A wave's events, each at (segment, position): a segment lies between two
    of its barriers, and waves share the segments."""

    def __init__(self, events, la, lb):
        self.issue, self.landed = {}, {}  # (op, stage) -> when
        self.reads, self.done = {}, {}    # id -> (op, parity, when); id -> when its data had returned
        self.uses, self.barriers = [], 0
        loads, lds = [], []               # in flight, in order: (op, stage), id per instruction
        for pos, e in enumerate(events):
            at = (self.barriers, pos)
            if e[0] == "B":
                self.barriers += 1
            elif e[0] == "I":
                op, st, par = map(int, e[1:])
                assert st % 2 == par
                self.issue[op, st] = at
                loads += [(op, st)] * (la if op < 2 else lb)
            elif e[0] == "R":
                i, op, par, n = map(int, e[1:])
                self.reads[i] = (op, par, at)
                lds += [i] * n
            elif e[0] == "W":
                vm, lgkm = int(e[1]), int(e[2])
                if vm < 63:
                    for u in loads[:max(0, len(loads) - vm)]:
                        self.landed[u] = at  # the last of its loads
                    loads = loads[max(0, len(loads) - vm):]
                if lgkm < 15:
                    lds = self._return(lds, max(0, len(lds) - lgkm), at)
            else:
                a, b = int(e[1]), int(e[2])
                for i in (a, b):
                    if i in lds:  # the compiler's own wait: this read and those before it
                        lds = self._return(lds, len(lds) - lds[::-1].index(i), at)
                if not self.uses or self.uses[-1] != (a, b):
                    self.uses.append((a, b))
        assert not loads, "loads in flight at the end"
        # an unread last prefetch returns at the next wait, after the loop
        for i in lds:
            self.done[i] = (self.barriers, len(events))

    def _return(self, lds, n, at):
        for i in lds[:n]:
            self.done[i] = at
        return lds[n:]


def _before(x, wx, y, wy):
    """Event x of wave wx is ordered before event y of wave wy."""
    return x < y if wx == wy else x[0] < y[0]


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
@pytest.mark.parametrize("ha,la,lb", [(4, 2, 2), (2, 2, 1)])  # 256 x 256 tiles; 128 x 256
@pytest.mark.parametrize("nst", [1, 2, 3, 6, 7])
def test_lds_order(tmp_path, ha, la, lb, nst):
    waves = [Wave(e, la, lb) for e in _trace(tmp_path, ha, la, lb, nst)]
    assert waves[0].barriers == waves[1].barriers
    stage = {}
    for w, W in enumerate(waves):
        for i, (op, par, at) in W.reads.items():
            # what the slot holds: the last stage of that parity that has landed whole
            have = [st for (o, st) in W.issue if o == op and st % 2 == par
                    and all(_before(V.landed[o, st], v, at, w) for v, V in enumerate(waves))]
            assert have, ("read before its loads", w, op, par, at)
            stage[w, i] = st = max(have)
            for v, V in enumerate(waves):
                if (op, st + 2) in V.issue:
                    assert _before(W.done[i], w, V.issue[op, st + 2], v), \
                        ("overwritten while read", "unit", op, "stage", st, "by wave", v, "reader", w)
        want = {(st, ha_, hb_) for st in range(nst) for ha_ in (0, 1) for hb_ in (0, 1)}
        got = []
        for a, b in dict.fromkeys(W.uses):
            assert stage[w, a] == stage[w, b]
            got.append((stage[w, a], W.reads[a][0], W.reads[b][0] - 2))
        assert len(got) == len(want) and set(got) == want
