"""The hash set of count vectors on the CPU, against a memory that is as unordered as relaxed loads allow.

prune_set.h is compiled for the host with stand-ins for the device's functions.  The slot that a vector
is looked up in has just been published by somebody else.  A load that covers the state sees that; any
other load sees the slot as it was before, emptied but with the vector of an earlier call still in it,
unless the state was seen first and wait_memory() stands between.  Plain loads see a stale line.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2202_13538_amd", "csrc")

DEVICE_UTIL = r"""
#pragma once
#include <stddef.h>
#include <stdint.h>
#include <string.h>
#define __device__
#define __host__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 1
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
inline int min(int a, int b) { return a < b ? a : b; }
extern uint32_t stale[], present[];   // the slots as they were and as they are
extern bool state_seen, ordered;
inline bool in_slots(const void* p) { return p >= (const void*)stale && p < (const void*)(stale + 64); }
inline uint32_t* now(const void* p) { return present + ((const uint32_t*)p - stale); }
template <typename T> T __hip_atomic_load(const T* p, int, int) {
    T value;
    const bool state = in_slots(p) && ((const uint32_t*)p - stale) % 16 == 0;
    memcpy(&value, in_slots(p) && (state || ordered) ? (const void*)now(p) : (const void*)p, sizeof(T));
    state_seen = state_seen || state;
    return value;
}
template <typename T, typename U> void __hip_atomic_store(T* p, U value, int, int) {
    *p = (T)value;
    if (in_slots(p)) *now(p) = (uint32_t)value;
}
inline uint32_t atomicCAS(uint32_t* p, uint32_t expected, uint32_t value) {
    const uint32_t was = *now(p);
    if (was == expected) *p = *now(p) = value;
    return was;
}
inline unsigned long long atomicAdd(unsigned long long* p, unsigned long long x) { *p += x; return *p - x; }
inline uint32_t atomicOr(uint32_t* p, uint32_t x) { *p |= x; return *p; }
inline void __builtin_amdgcn_s_sleep(int) {}
inline void __builtin_amdgcn_fence(int, const char*) {}
inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t, uint32_t) { return 0; }
inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t, uint32_t) { return 0; }
inline uint32_t __builtin_amdgcn_alignbyte(uint32_t a, uint32_t b, uint32_t n) {
    return (uint32_t)(((uint64_t)a << 32 | b) >> (8 * n));
}
inline uint64_t __ballot(bool x) { return x; }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __shfl(int x, int, int) { return x; }
namespace surel {
constexpr int kWave = 64;
constexpr uint32_t kDevCapacity = 0x20u, kDevStall = 0x100u;
inline uint32_t wave_bcast_u32(uint32_t x, int) { return x; }
inline void wave_sync() {}
inline void wait_memory() { ordered = ordered || state_seen; }
}
"""

MAIN = r"""
#include <cstdio>
#include "prune_set.h"
alignas(64) uint32_t stale[64], present[64];
bool state_seen, ordered;
uint32_t members[64 * 9], ranks[64], err;
unsigned long long counters[3];

// looks (10, 11, ..) up where it lies from an earlier call and `published` is the present vector
template <int NW> int look_up(int differs_at) {
    uint32_t w[NW];
    memset(stale, 0, sizeof stale);
    for (int k = 0; k < NW; ++k) w[k] = stale[surel::kSlotVector + k] = 10u + k;
    memcpy(present, stale, sizeof stale);
    present[0] = surel::kSlotFull | 3u;
    if (differs_at >= 0) present[surel::kSlotVector + differs_at] = 99u;
    state_seen = ordered = false;
    counters[0] = 7, err = 0;
    const surel::VectorSet set{stale, 3u, 64, members, ranks, counters, 100u, &err};
    return surel::find_or_insert<NW>(w, 0u, set);
}
template <int NW> void print() {
    for (int k = -1; k < NW; ++k) printf("%d ", look_up<NW>(k));
    printf("%u\n", err);
}
int main() { print<1>(); print<2>(); print<3>(); print<4>(); print<8>(); }
"""


def test_a_vector_of_an_earlier_call_is_no_match(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler here")
    shutil.copy(os.path.join(CSRC, "prune_set.h"), tmp_path)
    (tmp_path / "device_util.h").write_text(DEVICE_UTIL)
    (tmp_path / "kernels.h").write_text("#pragma once\nnamespace surel { struct PruneScratch; }\n")
    (tmp_path / "main.cpp").write_text(MAIN)
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-o", str(tmp_path / "model"),
                    str(tmp_path / "main.cpp")], check=True)
    out = subprocess.run([str(tmp_path / "model")], capture_output=True, text=True, check=True).stdout
    for nw, line in zip((1, 2, 3, 4, 8), out.splitlines(), strict=True):
        # number 3 for the published vector itself; one that differs in any word is none, and the
        # vector looked for is inserted behind it, as number 7
        assert line.split() == ["3"] + ["7"] * nw + ["0"], f"{nw} words: {line}"
