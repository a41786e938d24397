// One workgroup of a kernel on the CPU: a fiber per lane, and waves that run in a stated order, each until it stands at a barrier of the workgroup.
// What a wave does between two barriers then happens long before, or long after, what the others do there: accesses that no barrier orders show as
// other results, and a branch that waves take differently as barriers of different lines that meet.  (Lanes of a wave keep step at cross-lane operations.)
// Covers what common.hpp, topk_parts.hpp, scan_single.hpp and scan_bytes.hpp need.
#pragma once
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <type_traits>
#include <ucontext.h>
#include <vector>

namespace emu {
struct Site { const char* file; int line; };
enum State { kRunning, kAtStep, kAtBarrier, kDone };
struct Lane {
    ucontext_t ctx;
    std::vector<char> stack;
    State state;
    Site at;
    uint64_t value;
};
inline std::vector<Lane> lanes;
inline std::vector<uint64_t> seen;            // what the lanes brought to the wave's last cross-lane operation
inline ucontext_t scheduler;
inline int current;
inline long long counted, barriers;          // additions to counters in LDS; barriers that all lanes have passed
inline long long scored;                     // pieces that a lane has scored exactly (a marker of the scoring functions; long rows: several to a piece)
inline std::function<void()> body;
alignas(16) inline unsigned char lds[160 * 1024];

inline void stop(State s, Site at) {
    Lane& l = lanes[current];
    l.state = s;
    l.at = at;
    swapcontext(&l.ctx, &scheduler);
}
inline const uint64_t* step(uint64_t v, int line) {   // all lanes' values
    lanes[current].value = v;
    stop(kAtStep, {"a cross-lane operation", line});
    return &seen[current / 64 * 64];
}
inline void entry() {
    body();
    stop(kDone, {"the end", 0});
}

// Runs `kernel` by `threads` lanes; `order`: waves, the foremost that can go on does (none: in turn, an operation each).  False, with a line on stdout, where waves part.
inline bool run(int threads, const std::vector<int>& order, std::function<void()> kernel) {
    body = kernel;
    lanes.resize(threads);
    seen.assign(threads, 0);
    for (Lane& l : lanes) {
        l.stack.resize(128 * 1024);
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.data();
        l.ctx.uc_stack.ss_size = l.stack.size();
        l.ctx.uc_link = nullptr;
        makecontext(&l.ctx, entry, 0);
        l.state = kRunning;
    }
    auto resume = [&](int i) {
        current = i;
        lanes[i].state = kRunning;
        swapcontext(&scheduler, &lanes[i].ctx);
    };
    std::vector<State> wave(threads / 64, kRunning);
    std::vector<bool> wave_free(threads / 64, true);           // (may leave the barrier that its lanes stand at)
    for (int last = -1;;) {
        int w = -1;
        const int waves = (int)wave.size();
        for (int i = 0; i < waves && w < 0; ++i) {
            const int o = order.empty() ? (last + 1 + i) % waves : order[i];
            if (wave[o] == kRunning) w = o;
        }
        last = w;
        if (w < 0) {                                           // every wave at a barrier, or at its end
            for (int i = 1; i < threads; ++i)
                if (lanes[i].state != lanes[0].state || lanes[i].at.line != lanes[0].at.line || strcmp(lanes[i].at.file, lanes[0].at.file) != 0) {
                    printf("wave %d waits at %s:%d, wave 0 at %s:%d\n", i / 64, lanes[i].at.file, lanes[i].at.line, lanes[0].at.file, lanes[0].at.line);
                    return false;
                }
            if (wave[0] == kDone) return true;
            ++barriers;
            wave.assign(wave.size(), kRunning);
            wave_free.assign(wave.size(), true);
            continue;
        }
        for (int i = w * 64; i < w * 64 + 64; ++i)
            if (lanes[i].state != kAtBarrier || wave_free[w]) resume(i);
        wave_free[w] = false;
        int steps = 0, line = 0, ends = 0;                     // (lanes that a branch leaves out of an operation wait at the barrier behind it)
        for (int i = w * 64; i < w * 64 + 64; ++i) {
            const Lane& l = lanes[i];
            seen[i] = l.state == kAtStep ? l.value : 0;
            ends += l.state == kDone;
            if (l.state != kAtStep) continue;
            if (steps++ > 0 && l.at.line != line) {
                printf("wave %d: lanes at operations of lines %d and %d\n", w, line, l.at.line);
                return false;
            }
            line = l.at.line;
        }
        if (ends != 0 && ends != 64) {
            printf("wave %d: %d lanes have ended\n", w, ends);
            return false;
        }
        if (steps == 0) wave[w] = lanes[w * 64].state;
    }
}

inline uint64_t ballot(bool p, int line) {
    const uint64_t* v = step(p, line);
    uint64_t mask = 0;
    for (int i = 0; i < 64; ++i) mask |= (v[i] & 1) << i;
    return mask;
}
inline int readlane(int x, int from, int line) { return (int)step((uint32_t)x, line)[from]; }
inline int dpp(int old, int x, int ctrl, int row_mask, int line) {
    const uint64_t* v = step((uint32_t)x, line);
    const int lane = current % 64, row = lane / 16;
    if (!(row_mask >> row & 1)) return old;
    int from = -1;
    if (ctrl < 0x100) from = (lane & ~3) | (ctrl >> (lane % 4 * 2) & 3);
    else if (ctrl > 0x110 && ctrl < 0x120) from = lane % 16 >= ctrl - 0x110 ? lane - (ctrl - 0x110) : -1;
    else if (ctrl == 0x140) from = lane ^ 15;
    else if (ctrl == 0x141) from = lane ^ 7;
    else if (ctrl == 0x142) from = row > 0 ? row * 16 - 1 : -1;
    else if (ctrl == 0x143) from = row > 1 ? 31 : -1;
    else abort();
    return from < 0 ? old : (int)v[from];
}
struct Index { int x, y; };
struct ThreadIndex { operator int() const { return current; } };
inline struct { ThreadIndex x; } thread_index;
inline Index block_index{0, 0}, grid{1, 1};
}  // namespace emu

struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
struct float4 { float x, y, z, w; };
struct ulonglong2 { unsigned long long x, y; };
inline uint4 make_uint4(uint32_t x, uint32_t y, uint32_t z, uint32_t w) { return {x, y, z, w}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
template <typename T, typename F> inline T bits_as(F f) { static_assert(sizeof(T) == sizeof(F), ""); T t; memcpy(&t, &f, sizeof t); return t; }
inline uint32_t __float_as_uint(float f) { return bits_as<uint32_t>(f); }
inline int __float_as_int(float f) { return bits_as<int>(f); }
inline float __uint_as_float(uint32_t u) { return bits_as<float>(u); }
inline float __int_as_float(int i) { return bits_as<float>(i); }
inline int min(int a, int b) { return a < b ? a : b; }
inline int max(int a, int b) { return a > b ? a : b; }
inline uint32_t min(uint32_t a, uint32_t b) { return a < b ? a : b; }
inline uint32_t max(uint32_t a, uint32_t b) { return a > b ? a : b; }
template <typename T> inline T atomicAdd(T* p, T v) { ++emu::counted; const T old = *p; *p += v; return old; }
inline uint64_t wall_clock64() { return 0; }

#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __forceinline__ inline
#define __noinline__
#define __launch_bounds__(...)
#define __align__(n) alignas(n)
#define threadIdx emu::thread_index
#define blockIdx emu::block_index
#define gridDim emu::grid
#define __syncthreads() emu::stop(emu::kAtBarrier, {__FILE__, __LINE__})
#define __ballot(p) emu::ballot(p, __LINE__)
#define __builtin_amdgcn_ballot_w64(p) emu::ballot(p, __LINE__)
#define __popcll(x) __builtin_popcountll(x)
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() ((void)emu::step(0, __LINE__))
#define __builtin_amdgcn_sched_barrier(x) ((void)++emu::scored)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_readlane(v, l) emu::readlane(v, l, __LINE__)
#define __builtin_amdgcn_readfirstlane(v) emu::readlane(v, 0, __LINE__)
#define __builtin_amdgcn_update_dpp(old, v, ctrl, rows, banks, bound) emu::dpp(old, v, ctrl, rows, __LINE__)
#define __builtin_amdgcn_alignbyte(hi, lo, n) ((uint32_t)((((uint64_t)(hi) << 32) | (lo)) >> (8 * (n))))
#define __builtin_amdgcn_atomic_inc32(p, most, order, scope) ((*(p))++)
