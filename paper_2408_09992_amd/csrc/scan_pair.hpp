// Eq. 5 + TopK for a few queries over catalogues short enough that a workgroup's share fits its registers (scan_pair_kernel): as
// scan_short_kernel, two queries per workgroup.
// Part of kernels.hpp, which includes these parts inside namespace pqk in this order:
// common.hpp, subitem_scores.hpp, topk_parts.hpp, select_small.hpp, scan_single.hpp, scan_bytes.hpp, scan_short.hpp, scan_pair.hpp, scan_long.hpp, scan_subset.hpp,
// scan_batched.hpp, scan_filter.hpp, fold.hpp, comparison.hpp.
#pragma once

// Units (16-byte code vectors for rows of up to 16 bytes, items for longer rows) a thread takes at most: up to 80 scores, of two
// queries each item.  `row`: bytes of an item's row.
__host__ __device__ constexpr int pair_max_units(int row) { return row == 4 ? 8 : row == 8 ? 20 : row == 64 ? 24 : 40; }
// ... and holds the codes of all at once; beyond, the next ones' are requested as the sums go along.
__host__ __device__ constexpr int pair_held_units(int row) { return row == 64 ? 2 : row == 32 ? 4 : 8; }
// the instance that takes `units` units per thread, and the most the next smaller one takes
__host__ __device__ constexpr int pair_instance(int units, int held) {
    return units <= held ? units : units <= 4 ? 4 : units <= 8 ? 8 : units <= 12 ? 12 : units <= 16 ? 16 : units <= 20 ? 20 : units <= 24 ? 24 : units <= 32 ? 32 : 40;
}
__host__ __device__ constexpr int pair_sure_units(int u, int held) {
    return u <= held ? u - 1 : u == 4 ? held : u == 8 ? (held < 4 ? 4 : held) : u <= 24 ? u - 4 : u - 8;
}
__host__ __device__ constexpr bool pair_has(int u, int row) { return u <= pair_max_units(row) && pair_instance(u, pair_held_units(row)) == u; }
__host__ __device__ constexpr size_t pair_table_bytes(int m, int b, int cw) { return align16((size_t)m * (cw == 1 ? kLutStride : b) * sizeof(float2)); }

// The scores of one unit for both queries: the left-to-right sums of score_vector() and score_wide().
//   STRIDE: entries per split (0: `stride`)
template <int M, int CW, int STRIDE>
__device__ __forceinline__ void pair_scores(const float2* lut, int stride, uint32_t* w, float* s0, float* s1) {
    constexpr int kCodes = CW == 1 ? 16 : 8;                  // per code vector
    constexpr int VPU = M > kCodes ? M / kCodes : 1;
    float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int j = 0; j < VPU; ++j) {
        float2 v[kCodes];
#pragma unroll
        for (int c = 0; c < kCodes; ++c) {
            const uint32_t word = w[4 * j + (CW == 1 ? c >> 2 : c >> 1)];
            const uint32_t code = CW == 1 ? (word >> ((c & 3) * 8)) & 0xFFu : (c & 1) ? word >> 16 : word & 0xFFFFu;
            v[c] = lut[((j * kCodes + c) % M) * (STRIDE ? STRIDE : stride) + code];
        }
        __builtin_amdgcn_sched_barrier(0);                    // keep the reads ahead of the sums
#pragma unroll
        for (int c = 0; c < kCodes; ++c) {
            const int k = (j * kCodes + c) % M;
            acc.x = k == 0 ? v[c].x : acc.x + v[c].x;
            acc.y = k == 0 ? v[c].y : acc.y + v[c].y;
            if (k == M - 1) {
                const int e = M > kCodes ? 0 : c / M;
                s0[e] = acc.x; s1[e] = acc.y;
            }
        }
        if constexpr (VPU >= 4) {                             // (two vectors' values do not fit the registers beside the rest)
            asm volatile("" : "+v"(acc.x), "+v"(acc.y));
            if (j + 1 < VPU) asm volatile("" : "+v"(w[4 * j + 4]), "+v"(w[4 * j + 5]), "+v"(w[4 * j + 6]), "+v"(w[4 * j + 7]));
        }
    }
}

// The tables of queries q0 and q0 + 1 (`two`; else q0 once more) to LDS, interleaved: two entries of each at a time when size and address
// allow.  `then`: more loads, asked for behind the tables' (FIRST) or by the caller before.  Behind tables that one batch of loads brings (one-byte sub-ids,
// m <= 16), since loads return in order and codes come from further away (45,000 items, m = 8, 200 queries 16.7 us before, now 16.4; lists: 20,000
// candidates, m = 16, 100 queries 16.0 and 15.2).  Before tables of several batches, which would wait for the codes between them (m = 64, 2109 items, 328
// queries 13.2 us and, behind the first, 13.8, 7490, 710 62.3 and 63.8; two bytes, 100,000 items, b = 500, 40 queries 12.4 and 12.9).
__host__ __device__ constexpr bool pair_tables_first(int m, int cw, int threads) { return cw == 1 && m * kLutStride / 2 <= 4 * threads; }
template <int M, int CW, int NT, bool FIRST, typename Then>
__device__ __forceinline__ void pair_tables(float2* lut, const float* S, int q0, bool two, int b, int tid, Then&& then) {
    const float* S0 = S + (size_t)q0 * M * b;
    const float* S1 = two ? S0 + (size_t)M * b : S0;
    const int total = M * b;
    static_assert(!FIRST || M * kLutStride / 2 >= NT, "every thread has a part of the one batch");
    if ((CW == 2 || b == kLutStride) && (total & 1) == 0 && ((uintptr_t)S & 7) == 0) {
        constexpr int kBatch = CW == 2 || M * kLutStride / 2 > 4 * NT ? 4 : (M * kLutStride / 2 + NT - 1) / NT;   // (requested together, before the first store)
        const float2* src0 = reinterpret_cast<const float2*>(S0);
        const float2* src1 = reinterpret_cast<const float2*>(S1);
        const int pieces = total >> 1;
        for (int e0 = tid; FIRST || e0 < pieces; e0 += kBatch * NT) {
            float2 x[kBatch], y[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) { const int e = min(e0 + i * NT, pieces - 1); x[i] = src0[e]; y[i] = src1[e]; }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (FIRST) {
                then();
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
                if (e0 + i * NT < pieces) reinterpret_cast<float4*>(lut)[e0 + i * NT] = make_float4(x[i].x, y[i].x, x[i].y, y[i].y);
            if constexpr (FIRST) break;                       // (one batch, and every thread asks for its codes)
        }
    } else if constexpr (CW == 2) {
#pragma unroll 4
        for (int e = tid; e < total; e += NT) lut[e] = make_float2(S0[e], S1[e]);
    } else {
        // fewer than 256 sub-ids per split, or an odd address: element by element, rows padded with zeros
        if constexpr (FIRST) then();
#pragma unroll 4
        for (int e = tid; e < M * kLutStride; e += NT) {
            const int k = e / kLutStride, j = e % kLutStride;
            lut[e] = j < b ? make_float2(S0[k * b + j], S1[k * b + j]) : make_float2(0.0f, 0.0f);
        }
    }
}

// grid = (item blocks, (B + 1) / 2); queries 2y and 2y + 1 per workgroup, their tables' entries side by side in LDS (dynamic): one
// 8-byte read gives both queries' values, at the rate of a 4-byte one.  The share, its requests and the sums are scan_short_kernel's,
// over a grid of twice the blocks per query; the selection shares its barriers (select_mid_k_pair).  An odd batch's last query is scored
// twice and written once.  What bounds it: the LDS gathers, half of scan_short_kernel's, then the selection, twice as much of it for a
// score looked up.  512 threads: with 1024 the selection's fixed costs per wave weigh more than the latencies that more waves hide
// (14.9 and 16.0 us below).  Steps without Eq. 4, one query per workgroup and two (us): two-byte sub-ids, m = 8, b = 1024, 1.28M items,
// four queries, K = 10: 17.3 and 14.9; m = 8, 65,603 items, 97 queries: 20.5 and 14.6; m = 16, 300,000, 12, K = 48: 20.0 and 16.6; m = 32,
// 500,000, 8, K = 10: 29.5 and 21.5; m = 64, 30,000, 300: 141 and 81; m = 64, 51,826, 129, K = 20: 113 and 77.
// (waves per SIMD: seven units of m = 4 need 129 registers when left to themselves, with 128 a compute unit holds two workgroups: 28,058 items, 496
// queries 20.2 and 15.8 us)
__host__ __device__ constexpr int pair_waves(int m, int u, int cw) { return m == 4 && cw == 1 && u == 7 ? 4 : 1; }
template <int M, int U, int NT, int CW = 1>
__global__ __launch_bounds__(NT, pair_waves(M, U, CW)) void scan_pair_kernel(const uint8_t* codes, const float* S, void* out, float* out_scores, uint32_t N, int b, int B, int K) {
    ScanArgs a;                                               // (plain arguments: see scan_short_kernel)
    a.codes = codes; a.S = S; a.N = N; a.m = M; a.b = b; a.K = K;
    a.ws_keys = static_cast<uint64_t*>(out); a.out_ids = out_scores != nullptr ? static_cast<int*>(out) : nullptr;
    a.out_scores = out_scores;
    constexpr int P = M * CW;
    constexpr int VPU = Round<P>::kVPU, IPV = Round<P>::kIPV;  // vectors per unit, items per unit
    constexpr bool kTail = P < 16;                             // items after the last whole code vector may exist (a slot is kept for them)
    constexpr int R = U * IPV + (kTail ? 1 : 0);
    constexpr int kHeld = pair_held_units(P), kSure = pair_sure_units(U, kHeld);
    constexpr int kRing = U <= kHeld ? U : kHeld;              // units whose codes are on their way or here
    static_assert(CW == 1 || CW == 2, "one- or two-byte sub-ids");
    static_assert(U >= 1 && U <= pair_max_units(P), "units per thread");
    extern __shared__ __align__(16) unsigned char smem[];
    float2* const lut = reinterpret_cast<float2*>(smem);
    unsigned char* const sel = smem + pair_table_bytes(M, b, CW);   // what the selection needs, for this K
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int q0 = blockIdx.y * 2, nblk = gridDim.x, blk = blockIdx.x;
    const bool two = q0 + 1 < B;

    const uint32_t total_units = (uint32_t)(P <= 16 ? (a.N * P) / 16 : a.N);   // whole code vectors (P <= 16) or items; >= 1
    const uint32_t last_unit = total_units - 1;
    const uint32_t first = (uint32_t)blk * NT + (uint32_t)tid, stride = (uint32_t)nblk * NT;   // unit u: first + u * stride

    uint32_t w[kRing][4 * VPU];
    uint32_t ahead = first;
    auto fetch = [&](int u) {                                 // (branch-free: a unit past the end re-reads another)
        const uint32_t at = ahead + (uint32_t)u * stride;
        const uint4* base = reinterpret_cast<const uint4*>(a.codes) + (size_t)min(at, last_unit) * VPU;
#pragma unroll
        for (int j = 0; j < VPU; ++j) {
            const uint4 x = base[j];
            uint32_t* const to = w[u % kRing] + 4 * j;
            to[0] = x.x; to[1] = x.y; to[2] = x.z; to[3] = x.w;
        }
    };
    if constexpr (pair_tables_first(M, CW, NT)) {
        pair_tables<M, CW, NT, true>(lut, a.S, q0, two, b, tid, [&]() {
#pragma unroll
            for (int u = 0; u < kRing; ++u) fetch(u);
        });
    } else {
#pragma unroll
        for (int u = 0; u < kRing; ++u) fetch(u);
        pair_tables<M, CW, NT, false>(lut, a.S, q0, two, b, tid, []() {});
    }
    auto& select = *reinterpret_cast<MidSelectLds<NT>(*)[2]>(sel);
    mid_select_clear<NT>(select[0], tid);
    mid_select_clear<NT>(select[1], tid);
    __syncthreads();

    // ---- Eq. 5 for everything this thread holds
    constexpr int kStride = CW == 1 ? kLutStride : 0;
    float sc[2][R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool have = u < kSure || first + (uint32_t)u * stride < total_units;
        uint32_t* const x = w[u % kRing];
        float p0[IPV], p1[IPV];
        if (u < kSure || __ballot(have) != 0) {               // (a wave wholly past the end looks nothing up)
            pair_scores<M, CW, kStride>(lut, b, x, p0, p1);
        } else {
#pragma unroll
            for (int e = 0; e < IPV; ++e) p0[e] = p1[e] = 0.0f;
        }
        // (every sum stands before the lookups of the unit after the next begin, or the compiler moves all units' lookups to the front
        // and runs out of registers)
#pragma unroll
        for (int e = 0; e < IPV; ++e) asm volatile("" : "+v"(p0[e]), "+v"(p1[e]));
        if (u + kRing < U) {
            asm volatile("" : "+v"(ahead));
            fetch(u + kRing);
        }
        constexpr int kWindow = VPU >= 2 ? 1 : 2;             // units whose lookups are under way together
        if (U > kWindow && u + kWindow < U) {
#pragma unroll
            for (int j = 0; j < 4 * VPU; ++j) asm volatile("" : "+v"(w[(u + kWindow) % kRing][j]));
        }
#pragma unroll
        for (int e = 0; e < IPV; ++e) {
            sc[0][u * IPV + e] = have ? p0[e] : empty_score();
            sc[1][u * IPV + e] = have ? p1[e] : empty_score();
        }
    }
    if constexpr (kTail) {
        // the fewer than 16 / P items after the last whole code vector: one per lane of the first wave of block 0
        sc[0][R - 1] = sc[1][R - 1] = empty_score();
        if (blk == 0 && wave == 0) {
            const uint32_t item = total_units * IPV + lane;
            if (item < (uint32_t)a.N) {
                const uint8_t* row = a.codes + (size_t)item * P;
                float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const uint32_t code = CW == 2 ? reinterpret_cast<const uint16_t*>(row)[k] : row[k];
                    const float2 v = lut[k * (kStride ? kStride : b) + code];
                    acc.x = k == 0 ? v.x : acc.x + v.x;
                    acc.y = k == 0 ? v.y : acc.y + v.y;
                }
                sc[0][R - 1] = acc.x; sc[1][R - 1] = acc.y;
            }
        }
    }

    // ---- each query's K best, ranked, straight to the workspace or the result
    auto id_of = [&](int slot) -> uint32_t {
        if (kTail && slot == R - 1) return total_units * IPV + (uint32_t)lane;
        return (first + (uint32_t)(slot / IPV) * stride) * IPV + (uint32_t)(slot % IPV);
    };
    auto emit = [&](int h, int rank, uint64_t key) {
        if (h == 0 || two) emit_key(a, q0 + h, nblk, blk, rank, key);
    };
    select_mid_k_pair<NT>(sc, id_of, K, select, tid, emit);
}
