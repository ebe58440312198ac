"""The claim counters of a grouped launch (csrc/common.h), on the CPU: with the device functions
compiled for the host and the atomics stepped one by one, every order of the last arrivals of two
launches that overlap (which is not allowed, and may give wrong products) leaves the counters as a
launch has to find them, so that the launches after them are right again."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STUB = r"""
#pragma once
#include <cstdint>
#include <functional>
#define __device__
#define __host__
#define __forceinline__ inline
struct Dim { unsigned x = 0; };
extern Dim threadIdx, blockIdx, gridDim;
extern std::function<void()> between;      // runs once after the next atomic, before its caller goes on
template <class T> T step(T old) {
    if (between) { auto f = std::move(between); between = nullptr; f(); }
    return old;
}
inline unsigned atomicAdd(unsigned* p, unsigned v) { const unsigned o = *p; *p += v; return step(o); }
inline unsigned atomicInc(unsigned* p, unsigned v) { const unsigned o = *p; *p = o >= v ? 0 : o + 1; return step(o); }
inline unsigned long long __ballot(bool b) { return b; }
inline int __builtin_amdgcn_readfirstlane(int v) { return v; }
inline void __syncthreads() {}
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))
"""

MAIN = r"""
#include "common.h"
#include <cstdio>
#include <vector>
Dim threadIdx, blockIdx, gridDim;
std::function<void()> between;
int main() {
    int bad = 0, runs = 0;
    for (unsigned grid : {1u, 2u, 3u, 24u})
        for (unsigned ahead = 0; ahead <= grid; ++ahead)          // arrivals of the second launch before the first's last
            for (unsigned inside = 0; inside <= grid - ahead; ++inside) {   // and between that one's count and its stores
                cmp::TileQueues q{};
                std::vector<unsigned> counters(cmp::kQueueWords, 0);
                for (int x = 0; x < cmp::kXcds; ++x) counters[x * cmp::kQueuePitch] = 5 + x;   // claims made
                gridDim.x = grid;
                const cmp::TileClaims claims(q, counters.data());
                auto arrive = [&](unsigned n) { for (unsigned i = 0; i < n; ++i) claims.finish(); };
                arrive(grid - 1);
                arrive(ahead);
                between = [&, inside] { arrive(inside); };
                arrive(1);
                arrive(grid - ahead - inside);
                ++runs;
                for (unsigned w : counters) bad += w != 0;
                // a launch by itself afterwards
                for (int x = 0; x < cmp::kXcds; ++x) counters[x * cmp::kQueuePitch] = 7;
                arrive(grid - 1);
                bad += grid > 1 && counters[0] != 7;              // not before its last workgroup
                arrive(1);
                for (unsigned w : counters) bad += w != 0;
            }
    std::printf("runs %d bad %d\n", runs, bad);
    return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not found")
def test_counters_recover_from_overlapping_launches(tmp_path):
    os.makedirs(tmp_path / "hip")
    (tmp_path / "hip" / "hip_runtime.h").write_text(STUB)
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "claims")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-I", str(tmp_path),
                        "-I", os.path.join(ROOT, "paper_2311_03543_amd", "csrc"), str(tmp_path / "main.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and " bad 0" in r.stdout, (r.stdout, r.stderr)
