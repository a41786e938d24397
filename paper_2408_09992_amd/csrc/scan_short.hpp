// Eq. 5 + TopK for catalogues short enough that a workgroup's share fits its registers (scan_short_kernel): the scan of
// every single-query call over up to a few million items, the headline workload among them.
// Part of kernels.hpp, which includes these parts inside namespace pqk in this order:
// common.hpp, subitem_scores.hpp, topk_parts.hpp, select_small.hpp, scan_single.hpp, scan_bytes.hpp, scan_short.hpp, scan_pair.hpp, scan_long.hpp, scan_subset.hpp,
// scan_batched.hpp, scan_filter.hpp, fold.hpp, comparison.hpp.
#pragma once

// Most units (16-byte code vectors for rows of up to 16 bytes, items for longer rows) a thread holds ALL AT ONCE: everything is
// requested before the tables are even there.
__host__ __device__ constexpr int short_held_units(int m) {
    return m == 1 ? 2 : m == 2 ? 2 : m == 4 ? 6 : m == 8 ? 12 : m == 16 ? 12 : m == 32 ? 8 : 4;
}
__host__ __device__ constexpr int short16_held_units(int m) { return m == 16 ? 6 : 12; }   // two-byte sub-ids (m = 4, 8, 16)
// Beyond, the scores of up to 64 items per thread stay in registers and only the next units' codes with them: instances of 16, 24,
// ... units, each for every count down to the next smaller instance's.  Against the general kernel, whose lists, running floors and
// final merge cost more the more results there are (one user, microseconds per step for K = 10, 100, 512): 5M items at m = 8
// 24.7, 34.9, 70.8 -> 19.0, 23.1, 28.7; 8.3M at m = 4 21.8, 32.2, 68.4 -> 17.6, 21.9, 28.6; 3.5M at m = 64 55.7, 60.0, 96.1 -> 51.4,
// 55.2, 60.3.  At 64 items it ends: registers (at m = 8 the general kernel's sixteen copies of the tables are as fast there).
__host__ __device__ constexpr int short_max_units(int m) { return m <= 2 ? 2 : m == 4 ? 16 : m == 8 ? 32 : m == 16 ? 48 : 32; }
__host__ __device__ constexpr int short16_max_units(int m) { return m == 4 ? 32 : m == 8 ? 48 : 32; }
// the instance that takes `units` units per thread (at most short_max_units), and the most the next smaller one takes
__host__ __device__ constexpr int short_instance(int units, int held) {
    return units <= held ? units : units <= 8 && held < 8 ? 8 : units <= 12 && held < 12 ? 12 : units <= 16 ? 16 : units <= 24 ? 24 : units <= 32 ? 32 : 48;
}
__host__ __device__ constexpr int short_sure_units(int u, int held) {
    return u <= held ? u - 1 : u == 8 ? held : u == 12 ? (held < 8 ? 8 : held) : u == 16 ? (held > 12 ? held : 12) : u == 24 ? 16 : u == 32 ? 24 : 32;
}

__host__ __device__ constexpr bool short_selects_small(int K, int u, int row) { return K <= small_k_max(row) && u * (row < 16 ? 16 / row : 1) <= 24; }
__host__ __device__ constexpr bool short_has(int u, int held, int most) { return u <= most && short_instance(u, held) == u; }

// grid = (item blocks, B); one query per workgroup; a thread holds U units of its workgroup's share: unit u of thread t
// of workgroup g is number (u * blocks + g) * NT + t of the catalogue's units (slot u of all workgroups together is one
// contiguous stretch of G).  The host picks U = ceil(units / (blocks * NT)), so nothing is loaded or looked up in vain
// but the last, ragged slot.  Same lookups and left-to-right sums as scan_topk_kernel (score_vector, score_wide); what
// differs is everything around them: all codes are requested before anything else happens, no lists, no histogram, one
// barrier after the tables' and one in the selection.  This step is all latency (the code matrix is a few
// microseconds of traffic), and a wave's latency is its instruction count: a kernel of its own, a few KB of code.
//   M: splits; CW: bytes per sub-id.  An item's row takes P = M * CW bytes (1, 2, 4, 8, 16: 16 / P items per code vector;
//   32, 64: P / 16 vectors per item).  CW = 2 (M = 4, 8, 16): the query's m x b table lies in dynamic LDS as in memory.
// The arguments are plain values, not a struct: they fit the scalar registers the hardware loads before a wave starts
// (amdgpu-kernarg-preload-count), and the kernel's first loads go out without a round trip for their addresses.
// (Few units: 64 vector registers are enough, for four workgroups on a CU when many queries each take one.)
template <int M, int U, int NT, bool STAMP = false, int CW = 1>
__global__ __launch_bounds__(NT, M * CW <= 16 && U <= 3 ? 8 : 1) void scan_short_kernel(const uint8_t* codes, const float* S, void* out, float* out_scores, uint32_t N,
                                                        int b, int K, uint64_t* stamps) {
    ScanArgs a;                                               // (what the shared parts below expect; never in memory)
    a.codes = codes; a.S = S; a.N = N; a.m = M; a.b = b; a.K = K;
    // out_scores: with one workgroup per query `out` is the ids of the result; without, the workspace's lists
    a.ws_keys = static_cast<uint64_t*>(out); a.out_ids = out_scores != nullptr ? static_cast<int*>(out) : nullptr;
    a.out_scores = out_scores; a.stamps = stamps;
    constexpr int NW = NT / kWave;
    constexpr int P = M * CW;
    constexpr int VPU = Round<P>::kVPU, IPV = Round<P>::kIPV;  // vectors per unit, items per unit
    constexpr bool kTail = P < 16 || (CW == 1 && P == 16);     // items after the last whole code vector may exist (a slot is kept for them)
    constexpr int R = U * IPV + (kTail ? 1 : 0);
    static_assert(CW == 1 || CW == 2, "one- or two-byte sub-ids");
    constexpr int kHeld = CW == 1 ? short_held_units(M) : short16_held_units(M);
    constexpr int kSure = short_sure_units(U, kHeld);          // slots that lie wholly inside the catalogue
    constexpr int kRingUnits = U <= kHeld ? U : (VPU >= 4 || U * IPV > 48 ? 4 : 8);   // units whose codes are on their way or here
    constexpr int kWindow = VPU >= 2 ? 1 : 2;                  // units whose lookups are under way together
    static_assert(U >= 1 && U <= (CW == 1 ? short_max_units(M) : short16_max_units(M)), "units per thread");
    __shared__ __align__(16) float lut_static[CW == 1 ? M * kLutStride : 4];
    extern __shared__ __align__(16) unsigned char smem[];
    float* const lut = CW == 1 ? lut_static : reinterpret_cast<float*>(smem);
    unsigned char* const sel = smem + (CW == 1 ? 0 : align16((size_t)M * b * sizeof(float)));   // what the selection needs, for this K
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int q = blockIdx.y, nblk = gridDim.x, blk = blockIdx.x;
    uint64_t* const rec = STAMP ? a.stamps + (((size_t)q * nblk + blk) * NW + wave) * kStampSlots : nullptr;
    stamp<STAMP>(rec, kStampEntry, lane);

    const uint32_t total_units = (uint32_t)(P <= 16 ? (a.N * P) / 16 : a.N);   // whole code vectors (P <= 16) or items; >= 1
    const uint32_t last_unit = total_units - 1;
    const uint32_t first = (uint32_t)blk * NT + (uint32_t)tid, stride = (uint32_t)nblk * NT;   // unit u: first + u * stride

    // ---- table values requested, then all codes, then the tables go to LDS
    uint32_t w[kRingUnits][4 * VPU];
    uint32_t ahead = first;
    auto fetch = [&](int u) {                                 // (branch-free: a unit past the end re-reads another)
        const uint32_t at = ahead + (uint32_t)u * stride;
        const uint4* base = reinterpret_cast<const uint4*>(a.codes) + (size_t)(U <= kHeld ? min(at, last_unit) : u < kSure || at <= last_unit ? at : min(first, last_unit)) * VPU;
#pragma unroll
        for (int j = 0; j < VPU; ++j) {
            const uint4 x = base[j];
            uint32_t* const to = w[u % kRingUnits] + 4 * j;
            to[0] = x.x; to[1] = x.y; to[2] = x.z; to[3] = x.w;
        }
    };
    auto fetch_codes = [&]() {
#pragma unroll
        for (int u = 0; u < kRingUnits; ++u) fetch(u);
    };
    const float* Sq = a.S + (size_t)q * M * b;
    if constexpr (CW == 2) {
        // the m x b table as it lies in memory, in 16-byte pieces when its size and address allow
        const int total = M * b;
        fetch_codes();
        if ((total & 3) == 0 && ((uintptr_t)Sq & 15) == 0) {
            const float4* src = reinterpret_cast<const float4*>(Sq);
            float4* dst = reinterpret_cast<float4*>(lut);
#pragma unroll 4
            for (int e = tid; e < (total >> 2); e += NT) dst[e] = src[e];
        } else {
#pragma unroll 4
            for (int e = tid; e < total; e += NT) lut[e] = Sq[e];
        }
    } else if (b == kLutStride && ((uintptr_t)Sq & 15) == 0) {
        constexpr int kPieces = M * kLutStride / 4;
        constexpr int kPer = (kPieces + NT - 1) / NT;
        const float4* src = reinterpret_cast<const float4*>(Sq);
        float4 t4[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            t4[i] = (kPieces % NT == 0 || tid + i * NT < kPieces) ? src[tid + i * NT] : make_float4(0, 0, 0, 0);
        fetch_codes();
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (kPieces % NT == 0 || tid + i * NT < kPieces) reinterpret_cast<float4*>(lut)[tid + i * NT] = t4[i];
    } else {
        // fewer than 256 sub-ids per split, or a table that is only 4-byte aligned: element by element, rows padded with zeros
        constexpr int kPer = (M * kLutStride + NT - 1) / NT;
        float tv[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = tid + i * NT, k = e / kLutStride, j = e % kLutStride;
            tv[i] = (e < M * kLutStride && j < b) ? Sq[k * b + j] : 0.0f;
        }
        fetch_codes();
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (tid + i * NT < M * kLutStride) lut[tid + i * NT] = tv[i];
    }
    const bool small = short_selects_small(K, U, P);
    if (small) small_select_clear<NT>(*reinterpret_cast<SmallSelectLds<NT>*>(sel), tid);
    else mid_select_clear<NT>(*reinterpret_cast<MidSelectLds<NT>*>(sel), tid);
    stamp<STAMP>(rec, kStampRequested, lane);
    __syncthreads();
    stamp<STAMP>(rec, kStampTables, lane);
    if constexpr (STAMP) {
        __builtin_amdgcn_s_waitcnt(0);                        // every outstanding load: the codes are here
        stamp<STAMP>(rec, kStampCodes, lane);
    }

    // ---- Eq. 5 for everything this thread holds.  Only the last slot can reach past the end (the host's choice of U
    // makes slots 0 .. U-2 whole); what it holds there is nothing
    float sc[R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const bool have = u < kSure || first + (uint32_t)u * stride < total_units;
        const uint32_t* const x = w[u % kRingUnits];
        float part[IPV];
        if (u < kSure || __ballot(have) != 0) {               // (a wave wholly past the end looks nothing up)
            if constexpr (CW == 2) {
                if constexpr (P > 16) part[0] = score_wide16<M>(lut, b, x);
                else score_vector16<M>(lut, b, x, part);
            } else if constexpr (M > 16) part[0] = score_wide<M>(lut, x);
            else score_vector<M, 1>(lut, x, part);
        } else {
#pragma unroll
            for (int e = 0; e < IPV; ++e) part[e] = 0.0f;
        }
        if (u + kRingUnits < U) {
            asm volatile("" : "+v"(ahead) : "v"(part[0]));
            fetch(u + kRingUnits);
        }
        if constexpr (U > kHeld) {
            // the next unit's lookups wait for this unit's scores, or the compiler moves every unit's loads and lookups to the
            // front and runs out of registers
#pragma unroll
            for (int j = 0; j < 4 * VPU; ++j) asm volatile("" : "+v"(w[(u + kWindow) % kRingUnits][j]) : "v"(part[0]));
        }
#pragma unroll
        for (int e = 0; e < IPV; ++e) sc[u * IPV + e] = have ? part[e] : empty_score();
    }
    if constexpr (kTail) {
        // the fewer than 16 / M items after the last whole code vector: one per lane of the first wave of block 0
        float tail_sc = empty_score();
        if (blk == 0 && wave == 0) {
            const uint32_t tail_item = total_units * IPV + lane;
            if (tail_item < (uint32_t)a.N) {
                const uint8_t* row = a.codes + (size_t)tail_item * P;
                if constexpr (CW == 2) {
                    const uint16_t* g = reinterpret_cast<const uint16_t*>(row);
                    tail_sc = lut[g[0]];
#pragma unroll
                    for (int k = 1; k < M; ++k) tail_sc = tail_sc + lut[(size_t)k * b + g[k]];
                } else {
                    tail_sc = lut[row[0]];
#pragma unroll
                    for (int k = 1; k < M; ++k) tail_sc = tail_sc + lut[k * kLutStride + row[k]];
                }
            }
        }
        sc[R - 1] = tail_sc;
    }
    stamp<STAMP>(rec, kStampScored, lane);

    // ---- the workgroup's K best, ranked, straight to the workspace or the result
    auto id_of = [&](int slot) -> uint32_t {
        if (kTail && slot == R - 1) return total_units * IPV + (uint32_t)lane;
        return (first + (uint32_t)(slot / IPV) * stride) * IPV + (uint32_t)(slot % IPV);
    };
    auto emit = [&](int rank, uint64_t key) { emit_key(a, q, nblk, blk, rank, key); };
    if (small) select_small_k<NT, R, STAMP>(sc, id_of, K, *reinterpret_cast<SmallSelectLds<NT>*>(sel), tid, emit, rec);
    else select_mid_k<NT, R, STAMP>(sc, id_of, K, *reinterpret_cast<MidSelectLds<NT>*>(sel), tid, emit, rec);
    stamp<STAMP>(rec, kStampEnd, lane);
}
