// Eq. 5 + TopK for catalogues beyond what one set of registers holds (scan_long_kernel): the single query over tens of millions of
// items, and queries side by side whose tables of two-byte sub-ids leave no room for lists per wave.
// Part of kernels.hpp, which includes these parts inside namespace pqk in this order:
// common.hpp, subitem_scores.hpp, topk_parts.hpp, select_small.hpp, scan_single.hpp, scan_bytes.hpp, scan_short.hpp, scan_pair.hpp, scan_long.hpp, scan_subset.hpp,
// scan_batched.hpp, scan_filter.hpp, fold.hpp, comparison.hpp.
#pragma once

constexpr int kLongThreads = 512;
constexpr int kLongScores = 32;                       // scores a thread holds per segment
constexpr int kLongCand = 2816;                       // keys of the candidate array: several segments' worth at K = 512

template <int NT>
struct LongSelectLds {
    uint64_t cand[kLongCand];
    uint32_t hist[kBins];
    float wave_min[NT / kWave], wave_max[NT / kWave];
    int ncand;
    int count[3];                                     // hits of a segment, of the next, and one being cleared
};

// A segment: what a thread scores between two looks at the candidates.
template <int P>
struct LongShape {
    static constexpr int kVPU = Round<P>::kVPU, kIPV = Round<P>::kIPV;
    static constexpr int kUnits = kLongScores / kIPV;                    // units of a segment per thread
    static constexpr int kRingUnits = kVPU == 4 ? 4 : 8;   // units whose codes are on their way or here
    static_assert(kUnits % kRingUnits == 0, "a unit's place in the ring is the same in every segment");
};

// The n keys of L.cand, best first, in place.
template <int NT>
__device__ __forceinline__ void long_order(LongSelectLds<NT>& L, int n, int tid) {
    constexpr int NW = NT / kWave, R = (kLongCand + NT - 1) / NT;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    float mn = __builtin_inff(), mx = -__builtin_inff();
    for (int t = tid; t < n; t += NT) { const float v = score_of_key(L.cand[t]); mn = fminf(mn, v); mx = fmaxf(mx, v); }
    wave_minmax(mn, mx);
    if (lane == 0) { L.wave_min[wave] = mn; L.wave_max[wave] = mx; }
    __syncthreads();
    float lo = L.wave_min[0], hi = L.wave_max[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) { lo = fminf(lo, L.wave_min[w]); hi = fmaxf(hi, L.wave_max[w]); }
    float scale = hi > lo ? (float)kBins / (hi - lo) : 0.0f;
    if (!(scale > 0.0f) || scale > 3.0e38f) scale = 0.0f;
    if (bucket_sort<NT, R>(L.cand, n, lo, scale, L.hist, tid)) return;
    // (too many in one bucket: by counting, from registers to their places)
    uint64_t mine[R];
    int rank[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        mine[r] = r * NT + tid < n ? L.cand[r * NT + tid] : 0ull;
        rank[r] = 0;
    }
    for (int u = 0; u < n; ++u) {
        const uint64_t x = L.cand[u];
#pragma unroll
        for (int r = 0; r < R; ++r) rank[r] += x > mine[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (mine[r] != 0ull) L.cand[rank[r]] = mine[r];
    __syncthreads();
}

// grid = (item blocks, B); one query per workgroup of kLongThreads (512).  As in scan_short_kernel, unit u of thread t of workgroup g is
// number (u * blocks + g) * NT + t; a segment is kUnits of them, its scores in registers, the codes of the next units under way in a
// ring that runs on across segments.  The first segment gives a floor that K of the threads' best scores reach; after it the scores
// at or above it (about K per segment) are appended to the candidates, without a barrier when all segments' can be expected to fit.
// Otherwise each segment's are counted first (one barrier); where the array would overflow, the segment's own floor is taken,
// then the candidates are cut back to their K best; ties that still do not fit are decided by the exact K-th key.  The candidates are
// ordered once, at the end.
// What bounds it: the codes from memory (two-byte sub-ids, 50M items of m = 8: 800 MB, 5.9 TB/s) or the lookups.  C copies of the tables
// (m <= 8) cut the bank conflicts of the lookups, from 8.7 lanes per clock and CU to 14.  512 threads: with 1024 the scores,
// the ring and the cutting back do not fit the registers (m = 8, 9M items 32 us per step against 25).
// One user, microseconds per step before (general kernel) and now: m = 8, 9M items, K = 10 / 100 / 512 28.7 / 40.0 / 78.8 -> 25.8 / 30.6 /
// 37.0; two-byte sub-ids, m = 8, 50M items 152 / 178 / 582 -> 141 / 149 / 161.
//   M, CW: splits, bytes per sub-id; C: copies
template <int M, int CW, int C>
__global__ __launch_bounds__(kLongThreads) void scan_long_kernel(const uint8_t* codes, const float* S, void* result, float* out_scores, uint32_t N,
                                                                   int b, int K) {
    ScanArgs a;                                               // (plain arguments: see scan_short_kernel)
    a.codes = codes; a.S = S; a.N = N; a.m = M; a.b = b; a.K = K;
    a.ws_keys = static_cast<uint64_t*>(result); a.out_ids = out_scores != nullptr ? static_cast<int*>(result) : nullptr;
    a.out_scores = out_scores;
    constexpr int NT = kLongThreads, NW = NT / kWave, P = M * CW;
    using Sh = LongShape<P>;
    constexpr int VPU = Sh::kVPU, IPV = Sh::kIPV, U = Sh::kUnits, kRingUnits = Sh::kRingUnits;
    constexpr bool kTail = P < 16 || (CW == 1 && P == 16);
    constexpr int R = U * IPV + (kTail ? 1 : 0);
    static_assert(C == 1 || CW == 1, "copies of one-byte sub-ids' tables only");
    __shared__ __align__(16) float lut_static[CW == 1 ? M * kLutStride * C : 4];
    extern __shared__ __align__(16) unsigned char smem[];
    float* const lut_base = CW == 1 ? lut_static : reinterpret_cast<float*>(smem);
    LongSelectLds<NT>& L = *reinterpret_cast<LongSelectLds<NT>*>(smem + (CW == 1 ? 0 : align16((size_t)M * b * sizeof(float))));
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int q = blockIdx.y, nblk = gridDim.x, blk = blockIdx.x;

    const uint32_t total_units = (uint32_t)(P <= 16 ? ((uint64_t)N * P) / 16 : N), last_unit = total_units - 1;
    const uint32_t first = (uint32_t)blk * NT + (uint32_t)tid, stride = (uint32_t)nblk * NT;
    const uint32_t own = first < last_unit ? first : last_unit;   // what loads past the end read
    const uint32_t segments = (total_units + stride * U - 1) / (stride * U);   // (the host keeps the product below 2^32)

    uint32_t w[kRingUnits][4 * VPU];
    uint32_t ahead = first;                                   // the next unit to ask for
    auto fetch = [&](int slot) {
        const uint4* base = reinterpret_cast<const uint4*>(codes) + (size_t)(ahead <= last_unit ? ahead : own) * VPU;
#pragma unroll
        for (int j = 0; j < VPU; ++j) {
            const uint4 x = base[j];
            w[slot][4 * j] = x.x; w[slot][4 * j + 1] = x.y; w[slot][4 * j + 2] = x.z; w[slot][4 * j + 3] = x.w;
        }
        ahead += stride;
    };
    auto fetch_first = [&]() {
#pragma unroll
        for (int u = 0; u < kRingUnits; ++u) fetch(u);
    };

    // ---- the query's tables to LDS
    const float* Sq = S + (size_t)q * M * b;
    if constexpr (CW == 2) {
        const int total = M * b;
        fetch_first();
        if ((total & 3) == 0 && ((uintptr_t)Sq & 15) == 0) {
            const float4* src = reinterpret_cast<const float4*>(Sq);
            float4* dst = reinterpret_cast<float4*>(lut_base);
#pragma unroll 4
            for (int e = tid; e < (total >> 2); e += NT) dst[e] = src[e];
        } else {
#pragma unroll 4
            for (int e = tid; e < total; e += NT) lut_base[e] = Sq[e];
        }
    } else if constexpr (C > 1) {
        // thread t writes the 16-byte pieces t, t + NT, ... of the replicated tables (a quarter of the copies of an entry each)
        constexpr int kPieces = M * kLutStride * (C / 4), kPer = kPieces / NT;
        static_assert(kPieces % NT == 0, "whole pieces");
        float tv[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = (tid + i * NT) / (C / 4), k = e / kLutStride, j = e % kLutStride;
            tv[i] = j < b ? Sq[k * b + j] : 0.0f;
        }
        fetch_first();
#pragma unroll
        for (int i = 0; i < kPer; ++i) reinterpret_cast<float4*>(lut_base)[tid + i * NT] = make_float4(tv[i], tv[i], tv[i], tv[i]);
    } else {
        constexpr int kPer = M * kLutStride / NT;
        static_assert(M * kLutStride % NT == 0, "whole rows");
        float tv[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = tid + i * NT, k = e / kLutStride, j = e % kLutStride;
            tv[i] = j < b ? Sq[k * b + j] : 0.0f;
        }
        fetch_first();
#pragma unroll
        for (int i = 0; i < kPer; ++i) lut_base[tid + i * NT] = tv[i];
    }
    if (tid < 3) L.count[tid] = 0;
    __syncthreads();
    const float* const lut = lut_base + (C > 1 ? lane % C : 0);

    const float ninf = -__builtin_inff();
    const bool both = K > NT / 2;                             // the floor is taken from the best of a thread's even and of its odd slots
    // No barrier between segments when what their number can be expected to add fits; if it did not, all once more with them.
    bool free_run = (uint64_t)segments * (uint32_t)(K + K / 2 + 32) <= (uint32_t)kLongCand;
    float f = ninf;                                           // K items of this workgroup reach it
    int held = 0;                                             // candidates in L.cand: every item so far that reaches f
    const uint32_t tail_item = total_units * IPV + (uint32_t)lane;   // the fewer than 16 / M items after the last whole vector
again:
    for (uint32_t seg = 0; seg < segments; ++seg) {
        // ---- Eq. 5 for a segment
        float sc[R];
        const uint32_t unit0 = first + seg * U * stride;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool have = unit0 + (uint32_t)u * stride < total_units;
            const uint32_t* const x = w[u % kRingUnits];
            float part[IPV];
            if (__ballot(have) != 0) {                        // (a wave wholly past the end looks nothing up)
                if constexpr (CW == 2) {
                    if constexpr (P > 16) part[0] = score_wide16<M>(lut, b, x);
                    else score_vector16<M>(lut, b, x, part);
                } else if constexpr (M > 16) part[0] = score_wide<M>(lut, x);
                else score_vector<M, C>(lut, x, part);
            } else {
#pragma unroll
                for (int e = 0; e < IPV; ++e) part[e] = 0.0f;
            }
            // (neither the loads nor the lookups of later units move up to here: registers)
            asm volatile("" : "+v"(ahead) : "v"(part[0]));
            fetch(u % kRingUnits);
            constexpr int kWindow = VPU >= 2 ? 1 : 2;
#pragma unroll
            for (int j = 0; j < 4 * VPU; ++j) asm volatile("" : "+v"(w[(u + kWindow) % kRingUnits][j]) : "v"(part[0]));
#pragma unroll
            for (int e = 0; e < IPV; ++e) sc[u * IPV + e] = have ? part[e] : empty_score();
        }
        if constexpr (kTail) {
            float tail_sc = empty_score();
            if (seg + 1 == segments && blk == 0 && wave == 0 && tail_item < N) {
                const uint8_t* row = codes + (size_t)tail_item * P;
                if constexpr (CW == 2) {
                    const uint16_t* g = reinterpret_cast<const uint16_t*>(row);
                    tail_sc = lut[g[0]];
#pragma unroll
                    for (int k = 1; k < M; ++k) tail_sc = tail_sc + lut[(size_t)k * b + g[k]];
                } else {
                    tail_sc = lut[row[0] * C];
#pragma unroll
                    for (int k = 1; k < M; ++k) tail_sc = tail_sc + lut[(k * kLutStride + row[k]) * C];
                }
            }
            sc[R - 1] = tail_sc;
        }
        auto id_of = [&](int slot) -> uint32_t {
            if (kTail && slot == R - 1) return tail_item;
            uint32_t unit0 = first + seg * U * stride;
            asm volatile("" : "+v"(unit0));                   // (nor R ids)
            return (unit0 + (uint32_t)(slot / IPV) * stride) * IPV + (uint32_t)(slot % IPV);
        };
        float best = ninf, other = ninf;
#pragma unroll
        for (int i = 0; i < R; ++i) {                         // (an empty slot's NaN never wins)
            if (i % 2 == 0) best = fmaxf(best, sc[i]);
            else other = fmaxf(other, sc[i]);
        }
        if (!both) { best = fmaxf(best, other); other = ninf; }

        // ---- what reaches the floor joins the candidates
        auto count_hits = [&]() -> int {
            int total = 0;
            if (__ballot(fmaxf(best, other) >= f) != 0) {
#pragma unroll
                for (int i = 0; i < R; ++i) total += __popcll(__ballot(sc[i] >= f));
            }
            return total;
        };
        auto append = [&](int at) {
            float again = f;                                  // (compared anew: R masks do not fit the scalar registers)
            asm volatile("" : "+v"(again));
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const uint64_t mask = __ballot(sc[i] >= again);
                if (mask == 0) continue;
                if (sc[i] >= again) L.cand[at + __popcll(mask & ((1ull << lane) - 1ull))] = make_key(sc[i] + 0.0f, id_of(i));
                at += __popcll(mask);
            }
        };
        auto place = [&](int* counter, int total) -> int {
            int at = 0;
            if (total != 0) {
                if (lane == 0) at = atomicAdd(counter, total);
                at = __builtin_amdgcn_readfirstlane(at);
            }
            return at;
        };
        if (seg != 0 && free_run) {
            const int total = count_hits(), at = held + place(&L.count[0], total);
            if (total != 0 && at + total <= kLongCand) append(at);
            continue;
        }
        if (seg != 0) {
            int* const counter = &L.count[seg % 3];
            const int total = count_hits(), at = place(counter, total);
            __syncthreads();
            const int n = *counter;
            if (tid == 0) L.count[(seg + 2) % 3] = 0;         // (its last readers are past this barrier, its next users before the next)
            if (held + n <= kLongCand) {
                if (total != 0) append(held + at);
                held += n;
                continue;
            }
        }
        // the first segment, or more hits than there is room for: this segment's own floor
        {
            float mn = fminf(best > ninf ? best : -ninf, other > ninf ? other : -ninf), mx = fmaxf(best, other);
            wave_minmax(mn, mx);
            if (lane == 0) { L.wave_min[wave] = mn; L.wave_max[wave] = mx; }
            for (int i = tid; i < kMidBins; i += NT) L.hist[i] = 0u;
            if (tid == 0) L.ncand = 0;
            __syncthreads();
            float lo = L.wave_min[0], hi = L.wave_max[0];
#pragma unroll
            for (int v = 1; v < NW; ++v) { lo = fminf(lo, L.wave_min[v]); hi = fmaxf(hi, L.wave_max[v]); }
            float scale = hi > lo ? (float)kMidBins / (hi - lo) : 0.0f;
            if (!(scale > 0.0f) || scale > 3.0e38f) scale = 0.0f;
            if (best > ninf) atomicAdd(&L.hist[bucket_of<kMidBins>(best, lo, scale)], 1u);
            if (other > ninf) atomicAdd(&L.hist[bucket_of<kMidBins>(other, lo, scale)], 1u);
            __syncthreads();
            f = fmaxf(f, floor_of_hist<kMidBins>(L.hist, K, lo, scale, lane));
        }
        bool cut_back = false;
        for (;;) {
            const int total = count_hits(), at = place(&L.ncand, total);
            __syncthreads();
            const int n = L.ncand;
            if (held + n <= kLongCand) {
                if (total != 0) append(held + at);
                held += n;
                break;
            }
            if (!cut_back && held > K) {                      // the K best of the candidates so far, and their floor
                cut_back = true;
                long_order<NT>(L, held, tid);
                held = K;
                f = fmaxf(f, score_of_key(L.cand[K - 1]));
                if (tid == 0) L.ncand = 0;
                __syncthreads();
                continue;
            }
            // ties: the K-th best key, the largest that K keys reach, bit by bit
            constexpr int kPer = (kLongCand + NT - 1) / NT;
            uint64_t old[kPer];
#pragma unroll
            for (int r = 0; r < kPer; ++r) old[r] = r * NT + tid < held ? L.cand[r * NT + tid] : 0ull;
            uint64_t kth = 0ull;
            for (int bit = 63; bit >= 0; --bit) {
                const uint64_t t = kth | (1ull << bit);
                int reach = 0;
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    float x = sc[i];                          // (made anew in every step: R keys do not fit the registers)
                    asm volatile("" : "+v"(x));
                    reach += __popcll(__ballot(x == x && make_key(x + 0.0f, id_of(i)) >= t));
                }
#pragma unroll
                for (int r = 0; r < kPer; ++r) reach += __popcll(__ballot(old[r] >= t));
                if (tid == 0) L.hist[bit] = 0u;
                __syncthreads();
                if (lane == 0) atomicAdd(&L.hist[bit], (uint32_t)reach);
                __syncthreads();
                if (L.hist[bit] >= (uint32_t)K) kth = t;
            }
            if (tid == 0) L.ncand = 0;
            __syncthreads();
#pragma unroll
            for (int i = 0; i < R; ++i) {
                float x = sc[i];
                asm volatile("" : "+v"(x));
                const uint64_t key = make_key(x + 0.0f, id_of(i));
                if (x == x && key >= kth) L.cand[atomicAdd(&L.ncand, 1)] = key;
            }
#pragma unroll
            for (int r = 0; r < kPer; ++r)
                if (old[r] >= kth && old[r] != 0ull) L.cand[atomicAdd(&L.ncand, 1)] = old[r];
            __syncthreads();
            held = L.ncand;                                   // = K: keys are distinct
            f = fmaxf(f, score_of_key(kth));
            break;
        }
    }
    __syncthreads();
    if (free_run) {
        const int n = held + L.count[0];
        if (n > kLongCand) {
            __syncthreads();
            if (tid == 0) L.count[0] = 0;
            free_run = false;
            f = ninf;
            held = 0;
            ahead = first;
            fetch_first();
            __syncthreads();
            goto again;
        }
        held = n;
    }

    // ---- the K best, ordered
    if (held <= kRankByCount) {
        const int n8 = (held + 7) & ~7;
        if (tid < n8 - held) L.cand[held + tid] = 0ull;
        __syncthreads();
        rank_emit<NT>(L.cand, held, K, tid, [&](int rank, uint64_t key) { emit_key(a, q, nblk, blk, rank, key); });
    } else {
        long_order<NT>(L, held, tid);
        for (int t = tid; t < K; t += NT) emit_key(a, q, nblk, blk, t, t < held ? L.cand[t] : 0ull);
    }
}
