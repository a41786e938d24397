// Eq. 5 + TopK for one query over a long catalogue (scan_bytes_kernel): one-byte upper bounds dismiss nearly all items, the few that are left
// are scored exactly.
// Part of kernels.hpp, which includes these parts inside namespace pqk in this order:
// common.hpp, subitem_scores.hpp, topk_parts.hpp, select_small.hpp, scan_single.hpp, scan_bytes.hpp, scan_short.hpp, scan_pair.hpp, scan_long.hpp,
// scan_subset.hpp, scan_batched.hpp, scan_filter.hpp, fold.hpp, comparison.hpp.
//
// What bounds the exact scans is the LDS: random four-byte lookups in tables of 1 KB per split collide in its banks (9 to 10 return per clock and
// CU, 14 from sixteen copies).  A table of 256 BYTES is 64 words, two to a bank of 32: lanes that look up the same word are served together, so a lookup
// collides two ways at most: 15 return per clock and CU (48 % of the LDS's cycles are conflicts), as from sixteen copies of the exact tables, which only rows of eight
// and fewer have room for and whose 128 KB take 5 us to write.  (This kernel without floors, lists and exact scores, which only adds such bytes up, took 66.3 us for 400 MB of codes at
// m = 8 and 71.7 at 64, without the lookups too 65.0.)
// A byte counts steps above a base of its split, rounded up: an item's sum of counts bounds its score from above.  One query's sums are added in
// 32 bits, so the counts use all 256 values whatever the row length is.  Items whose sum is below T, the floor's image, cannot reach the
// floor; a wave with any other scores its vector exactly, by the same left-to-right fp32 chain as everywhere, and only exact scores enter lists, floors
// and results: bit for bit the other kernels' results, whatever the tables are.
// 50M items, m = 8, K = 10 and 100: calls 78.9 -> 68.6 and 88.4 -> 75.6 us (16 copies of the tables in LDS; 5.8 TB/s now); 20M, m = 16 68.6 -> 55.9; 6M, m = 32 45.8 -> 37.7.  A
// wave's second unit is asked for when the tables are there, and from then on one at a time: asked for before, every further unit costs a microsecond, since the
// sample waits for all of them.
#pragma once

constexpr int kBytesThreads = kBigThreads;
constexpr float kBytesReach = 3.0f;               // counts reach so many spreads below a split's largest entry

// The bounds of one query, the same in every lane.
struct ByteBounds {
    float off, inv;                               // counts of a score s: (s - off) * inv
    __device__ __forceinline__ uint32_t threshold(float floor_ge, int m) const {   // no item whose counts add up to less reaches the floor
        const float t = floorf((floor_ge - off) * inv - 0.02f);
        return (uint32_t)fminf(fmaxf(t, 0.0f), (float)(255 * m + 1));
    }
};

// bytes of a split's counts (two-byte sub-ids: whole words)
__host__ __device__ constexpr int bytes_stride(int b, int cw) { return cw == 1 ? kLutStride : (b + 3) & ~3; }
__host__ __device__ constexpr size_t bytes_table_bytes(int m, int b, int cw) {
    return align16((size_t)m * (cw == 1 ? kLutStride : b) * sizeof(float)) + align16((size_t)m * bytes_stride(b, cw));
}

// M, CW: splits, bytes per sub-id.  Two-byte sub-ids: tables in dynamic LDS, exact ones as they lie in memory.
// STAMP: measurement instance that also records wall-clock stamps per wave.
template <int M, int CW = 1, bool STAMP = false>
__global__ __launch_bounds__(kBytesThreads) void scan_bytes_kernel(ScanArgs a) {
    constexpr int NT = kBytesThreads, NW = NT / kWave;
    constexpr int P = M * CW;                                  // bytes of an item's row
    constexpr int VPI = P > 16 ? P / 16 : 1, IPV = P > 16 ? 1 : 16 / P;   // vectors of a piece, items of a piece
    constexpr int kSplits = (M + NW - 1) / NW;                 // of a wave, while the tables are made
    constexpr int kParts = CW == 1 ? 1 : NW / M;               // waves of a split, likewise
    __shared__ __align__(16) float lut_static[CW == 1 ? M * kLutStride : 4];
    __shared__ __align__(16) uint8_t counts_static[CW == 1 ? M * kLutStride : 4];
    __shared__ float largest[M * kParts], spreads[M * kParts];
    __shared__ int crowd;                                      // scores in the bucket of the sample's K-th best, when it was found
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int q = blockIdx.y, nblk = gridDim.x, blk = blockIdx.x, K = a.K, b = a.b;
    uint64_t* const rec = STAMP ? a.stamps + (((size_t)q * nblk + blk) * NW + wave) * kStampSlots : nullptr;
    stamp<STAMP>(rec, kStampEntry, lane);
    const int stride = CW == 1 ? kLutStride : b, count_stride = bytes_stride(b, CW);
    float* const lut = CW == 1 ? lut_static : reinterpret_cast<float*>(smem);
    uint8_t* const counts = CW == 1 ? counts_static : smem + align16((size_t)M * b * sizeof(float));
    const ScanLds L = carve_scan(smem + (CW == 1 ? 0 : bytes_table_bytes(M, b, CW)), 0, a.cap, a.candmax, NW);
    Ctl* const ctl = L.ctl;
    // pieces: code vectors that lie wholly inside the catalogue, or items whose rows take several (the host sees to it: one at least)
    const uint32_t total = (uint32_t)(P <= 16 ? (a.N * P) / 16 : a.N), last = total - 1, n_scan = total * IPV;
    // unit i: a piece per lane, what wave i % NW takes of step i / NW.  (Two pieces to a unit: 50M items, m = 8, 71.1 -> 74.1 us a call, four 100.)
    auto piece_of = [&](uint32_t i) -> uint32_t { return ((i / NW) * (uint32_t)nblk + (uint32_t)blk) * NT + (i % NW) * kWave + (uint32_t)lane; };
    // (loads past the end: a line of the wave's own, not one for thousands of waves that get there together)
    const uint32_t own = (uint32_t)(blk * NW + wave) * 4u, spare = own < last ? own : last;
    auto fetch = [&](uint32_t i, uint32_t (&w)[4 * VPI]) {
        const uint32_t p = piece_of(i);
#pragma unroll
        for (int j = 0; j < VPI; ++j) {
            const uint4 x = reinterpret_cast<const uint4*>(a.codes)[(size_t)(p <= last ? p : spare) * VPI + j];
            w[4 * j] = x.x; w[4 * j + 1] = x.y; w[4 * j + 2] = x.z; w[4 * j + 3] = x.w;
        }
    };
    // The sample: the first unit of the first `sampling` waves; of long rows, which take longer to score, fewer items.
    const int sampling = K > 16 ? NW : P == 64 ? NW / 4 : P == 32 ? NW / 2 : NW;
    const float* const Sq = a.S + (size_t)q * M * b;
    uint32_t w[2][4 * VPI], unit[2] = {(uint32_t)wave, 0};
    // a split's largest entry, and how far below it the best of the middle lane's entries lies: about a sixth of all lie less far (a lane having four).  (A
    // mean would be carried away by one masked entry.)
    const auto clear = [&]() {
        for (int i = tid; i < kBins; i += NT) L.hist[i] = 0;
        if (tid == 0) { ctl->shared_floor = -__builtin_inff(); ctl->ncand = 0; ctl->next_unit = 2 * NW; }
        stamp<STAMP>(rec, kStampRequested, lane);
    };
    auto middle = [&](const uint32_t image, int want) -> float {   // the want-th smallest image of a float >= 0, to an eighth of itself
        uint32_t at = 0;
#pragma unroll
        for (uint32_t bit = 0x40000000u; bit >= 0x200000u; bit >>= 1)
            if (__popcll(__ballot(image < (at | bit))) < want) at |= bit;
        return __uint_as_float(at + 0x100000u);
    };
    if constexpr (CW == 1) {
        // ---- the tables on their way, a wave per split, four entries per lane, then the first codes
        float v[kSplits][4];
        if (b == kLutStride && ((uintptr_t)Sq & 15) == 0) {
#pragma unroll
            for (int i = 0; i < kSplits; ++i) {
                const int k = wave + i * NW;
                const float4 x = reinterpret_cast<const float4*>(Sq)[(k < M ? k : 0) * kWave + lane];
                v[i][0] = x.x; v[i][1] = x.y; v[i][2] = x.z; v[i][3] = x.w;
            }
        } else {
#pragma unroll
            for (int i = 0; i < kSplits; ++i)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int k = wave + i * NW, j = lane * 4 + c;
                    v[i][c] = (k < M && j < b) ? Sq[k * b + j] : 0.0f;   // (sub-ids beyond the alphabet score 0)
                }
        }
        fetch(unit[0], w[0]);
        clear();
        {
            float mx[kSplits];
            uint32_t image[kSplits], at[kSplits];
            const int lanes = (b + 3) / 4, want = lanes / 2 > 0 ? lanes / 2 : 1;
#pragma unroll
            for (int i = 0; i < kSplits; ++i) {
                const int k = wave + i * NW;
                if (k < M) reinterpret_cast<float4*>(lut)[k * kWave + lane] = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
                const float best = fmaxf(fmaxf(v[i][0], v[i][1]), fmaxf(v[i][2], v[i][3]));
                float mn = best;
                mx[i] = best;
                wave_minmax(mn, mx[i]);
                const float below = mx[i] - best;                  // (>= 0, or NaN)
                image[i] = (lane < lanes && below >= 0.0f) ? __float_as_uint(below) : 0x7F800000u;
                at[i] = 0;
            }
#pragma unroll
            for (uint32_t bit = 0x40000000u; bit >= 0x200000u; bit >>= 1)   // the want-th smallest, to an eighth of itself
#pragma unroll
                for (int i = 0; i < kSplits; ++i)
                    if (__popcll(__ballot(image[i] < (at[i] | bit))) < want) at[i] |= bit;
#pragma unroll
            for (int i = 0; i < kSplits; ++i) {
                const int k = wave + i * NW;
                if (lane == 0 && k < M) { largest[k] = mx[i]; spreads[k] = __uint_as_float(at[i] + 0x100000u); }
            }
        }
    } else {
        // ---- the query's m x b table as it lies in memory, behind the first codes; then a split's entries by kParts waves
        const int entries = M * b;
        fetch(unit[0], w[0]);
        if ((entries & 3) == 0 && ((uintptr_t)Sq & 15) == 0) {
#pragma unroll 4
            for (int e = tid; e < entries >> 2; e += NT) reinterpret_cast<float4*>(lut)[e] = reinterpret_cast<const float4*>(Sq)[e];
        } else {
#pragma unroll 4
            for (int e = tid; e < entries; e += NT) lut[e] = Sq[e];
        }
        clear();
        __syncthreads();
        const int k = wave / kParts, j0 = wave % kParts * kWave + lane;
        float best = -__builtin_inff();
        for (int j = j0; j < b; j += kParts * kWave) best = fmaxf(best, lut[k * b + j]);
        float mn = best, mx = best;
        wave_minmax(mn, mx);
        const float below = mx - best;                         // (>= 0, or NaN)
        const int lanes = b - wave % kParts * kWave < kWave ? b - wave % kParts * kWave : kWave;
        const float spread = middle(j0 < b && below >= 0.0f ? __float_as_uint(below) : 0x7F800000u, lanes / 2 > 0 ? lanes / 2 : 1);
        if (lane == 0) { largest[wave] = mx; spreads[wave] = spread; }
    }
    __syncthreads();
    stamp<STAMP>(rec, kStampTables, lane);
    unit[1] = (uint32_t)(NW + wave);
    fetch(unit[1], w[1]);

    WaveTopK top{L.lists + (size_t)wave * a.cap, a.cap, K, 0, 0, 0ull, -__builtin_inff()};
    auto largest_of = [&](int k) -> float {
        float l = largest[k * kParts];
#pragma unroll
        for (int i = 1; i < kParts; ++i) l = fmaxf(l, largest[k * kParts + i]);
        return l;
    };
    // ---- counts: 255 steps below every split's largest entry, what lies deeper counts as that
    float step, inv, span;                                     // span: what the splits' spreads add up to
    {
        const float l = lane < M ? largest_of(lane < M ? lane : 0) : 0.0f;
        float s = 0.0f;
        if (lane < M) {
            s = l - largest[lane * kParts] + spreads[lane * kParts];
#pragma unroll
            for (int i = 1; i < kParts; ++i) s = fminf(s, l - largest[lane * kParts + i] + spreads[lane * kParts + i]);
        }
        float none = 0.0f, widest = s;
        wave_minmax(none, widest);
        span = wave_sum_f32(s);
        step = widest * (kBytesReach / 255.0f);
        inv = 1.0f / step;
        if (!(inv < 1.0e30f) || !(step < 1.0e30f) || __ballot(!(fabsf(l) < 1.0e30f)) != 0) { inv = 0.0f; step = 0.0f; }   // degenerate: every item is scored
    }
    const int words = count_stride / 4;                        // of a split's counts
    for (int i = tid; i < M * words; i += NT) {
        const int k = i / (CW == 1 ? kWave : words), j = (i - k * words) * 4;
        const float base = largest_of(k) - 255.0f * step;
        float e[4];
        if constexpr (CW == 1) {
            const float4 x = reinterpret_cast<const float4*>(lut)[i];
            e[0] = x.x; e[1] = x.y; e[2] = x.z; e[3] = x.w;
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) e[c] = lut[k * b + (j + c < b ? j + c : b - 1)];
        }
        uint32_t word = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) word |= (uint32_t)fminf(fmaxf(ceilf((e[c] - base) * inv + 2.5e-4f), 0.0f), 255.0f) << (8 * c);
        reinterpret_cast<uint32_t*>(counts)[i] = word;
    }
    // exact scores of a piece
    auto score = [&](const uint32_t (&w)[4 * VPI], float (&sc)[IPV]) {
        if constexpr (CW == 2 && P > 16) sc[0] = score_wide16<M>(lut, stride, w);
        else if constexpr (CW == 2) score_vector16<M>(lut, stride, w, sc);
        else if constexpr (M > 16) sc[0] = score_wide<M>(lut, w);
        else score_vector<M>(lut, w, sc);
    };
    float hlo, hscale;
    {
        // ---- the sample's items, exactly: a histogram over their range gives the first floor (it lives on: every score that enters
        // a list is counted, and the waves take turns reading off the floor that allows)
        float sc[IPV], mn = __builtin_inff(), mx = -__builtin_inff();
        auto finite = [](float x) { return fminf(fmaxf(x, -1.0e30f), 1.0e30f); };   // (a range that buckets can divide)
        const uint32_t p = piece_of(unit[0]);
        const bool mine = wave < sampling && p <= last;
        if (wave < sampling) score(w[0], sc);
        if (mine) {
#pragma unroll
            for (int e = 0; e < IPV; ++e) { mn = fminf(mn, finite(sc[e])); mx = fmaxf(mx, finite(sc[e])); }
        }
        stamp<STAMP>(rec, kStampScored, lane);
        set_range<NW>(mn, mx, ctl, tid, hlo, hscale, 1.25f);
        if (mine) {
#pragma unroll
            for (int e = 0; e < IPV; ++e) atomicAdd(&L.hist[bucket_of(sc[e], hlo, hscale)], 1u);
        }
        __syncthreads();
        if (wave == 0) {
            find_cut(L.hist, K, ctl, lane);
            if (lane == 0) {
                ctl->shared_floor = next_up(ctl->cut);
                crowd = (int)L.hist[ctl->bstar];
            }
        }
        __syncthreads();
        // A score far from the others (an item with a masked sub-id, at -1e9) stretches the range until the buckets tell nothing apart: while the K-th
        // best shares its bucket with many that are no better, or buckets are too wide for floors to rise by, that bucket alone is taken apart again.  (An
        // entry of every split at -1e9: 50M items, m = 8 146 us without this, 72 with, 4M, m = 64 98 and 53; buckets too wide, half a split at -1e9: 28M,
        // m = 8, K = 512 451 and 76.)
        bool in[IPV];
#pragma unroll
        for (int e = 0; e < IPV; ++e) in[e] = mine;
        int left = K;                                          // the left-th best of what is `in` is sought
        float lo = hlo, per = hscale;
        float floor_ge = next_up(ctl->cut);                    // (K of the sample's scores reach it, and every later one)
        bool narrowed = per * span < 128.0f;                   // (degenerate ranges among them)
#pragma unroll 1
        for (int pass = 0; pass < 8; ++pass) {
            // (one decision: waves that leave count into the histogram at once, so nobody looks there)
            const int bstar = ctl->bstar;
            if (__builtin_expect((crowd <= 2 * left + kWave && !(per * span < 128.0f)) || !(per > 0.0f), 1)) break;
            narrowed = true;
            __syncthreads();
#pragma unroll
            for (int e = 0; e < IPV; ++e) {
                const int bucket = in[e] ? bucket_of(sc[e], lo, per) : -1;
                const uint64_t above = __ballot(bucket > bstar);
                if (lane == 0 && above != 0) (void)atomicAdd(&ctl->ncand, __popcll(above));
                in[e] = bucket == bstar;
            }
            for (int t = tid; t < kBins; t += NT) L.hist[t] = 0;
            __syncthreads();
            left -= ctl->ncand;
            mn = __builtin_inff();
            mx = -__builtin_inff();
#pragma unroll
            for (int e = 0; e < IPV; ++e)
                if (in[e]) { mn = fminf(mn, finite(sc[e])); mx = fmaxf(mx, finite(sc[e])); }
            __syncthreads();                                   // (set_range() clears the counter that was read)
            set_range<NW>(mn, mx, ctl, tid, lo, per);
            if (lo > -1.0e30f) floor_ge = fmaxf(floor_ge, lo); // (the lowest of what is `in`: the best floor there is where all are alike)
#pragma unroll
            for (int e = 0; e < IPV; ++e)
                if (in[e]) atomicAdd(&L.hist[bucket_of(sc[e], lo, per)], 1u);
            __syncthreads();
            if (wave == 0) {
                find_cut(L.hist, left, ctl, lane);
                if (lane == 0) crowd = (int)L.hist[ctl->bstar];
            }
            __syncthreads();
            floor_ge = fmaxf(floor_ge, next_up(ctl->cut));
        }
        if (__builtin_expect(narrowed, 0)) {                   // the histogram again, from the floor on
            __syncthreads();
            for (int t = tid; t < kBins; t += NT) L.hist[t] = 0;
            hlo = floor_ge;
            hscale = floor_ge > -__builtin_inff() && span > 0.0f && (float)kBins / span < 3.0e38f ? (float)kBins / span : 0.0f;
            __syncthreads();
#pragma unroll
            for (int e = 0; e < IPV; ++e)
                if (mine && sc[e] >= floor_ge) atomicAdd(&L.hist[bucket_of(sc[e], hlo, hscale)], 1u);
            if (tid == 0) ctl->shared_floor = floor_ge;
            __syncthreads();
        }
        top.floor_ge = floor_ge;
        if (wave < sampling) {
#pragma unroll
            for (int e = 0; e < IPV; ++e) {
                const bool take = mine && sc[e] >= top.floor_ge;
                const uint64_t mask = __ballot(take);
                if (mask != 0) top.append(mask, take, sc[e], p * IPV + (uint32_t)e, lane);
            }
        }
    }

    // ---- the bounds.  An item with an entry further than sum_max - floor below its split's largest is below the floor whatever its others are (a chain is
    // monotone in each term), so no entry that matters is larger than that.
    ByteBounds bounds;
    {
        const float l = lane < M ? largest_of(lane < M ? lane : 0) : 0.0f, sum_max = wave_sum_f32(l), depth = sum_max - top.floor_ge;
        // what fp32 chains of M additions (scores, sums of bases) can be off by
        const float slack = 4.0f * (float)(M + 1) * 5.9604645e-8f * wave_sum_f32(lane < M ? fmaxf(fabsf(l), fabsf(l - depth)) + 255.0f * step : 0.0f);
        bounds.off = sum_max - (float)M * 255.0f * step + slack;
        bounds.inv = fabsf(bounds.off) < 1.0e30f ? inv : 0.0f;
        if (bounds.inv == 0.0f) bounds.off = 0.0f;
    }

    stamp<STAMP>(rec, kStampOffered, lane);
    // ---- stream
    int turn = wave, gap = NW;                                 // units until this wave's next turn; grows by a quarter
    // Tables whose bounds say little let many lanes of most units pass: after three such units in a row a wave goes on without bounds for a while, each time for
    // longer, and looks again (after the first such unit from then on).  (Few lanes of every unit, as many results have until floors have risen, cost less than doing without.
    // Bounds given up for good after 32 units of which any lane passes, which 30 units a wave never get to, and as it is: 8M items, m = 64, Cauchy 138 us and 115,
    // +1e4 140 and 113, denormal 171 and 139, m = 32 +1e4 77 and 64; 50M, m = 8, K = 100, ordinary 75.7 and 76.2.)
    constexpr int kManyLanes = 24, kMostCredit = 4, kMostRest = 64;
    // (A wave has two units on its way, so whatever a unit does besides is waited for: one without hits sets the credit, one with few lanes too, and the loop has one bound.  A
    // credit that every unit counts up or down and the loop asks for, and a K-th key compared with every unit's before: 40M, m = 8, K = 100 64.9 us, and 64.5 now; 28M, K = 512 74.4 and 73.7; 40M, m = 4, K = 100
    // 42.9 and 42.6; tables whose bounds say little the same.)
    const uint32_t per_step = (uint32_t)NT * (uint32_t)nblk, units = (total + per_step - 1) / per_step * NW;
    int credit = kMostCredit, rest = 16;
    uint32_t until = units;                                    // 0: the loop at hand ends
    auto process = [&](auto bounded, const uint32_t (&w)[4 * VPI], uint32_t i) {
        top.floor_ge = fmaxf(top.floor_ge, lds_peek(&ctl->shared_floor));
        if (--turn < 0) {
            gap += gap >> 2;
            turn = gap;
            const float f = floor_of_hist<kBins>(L.hist, K, hlo, hscale, lane);
            if (lane == 0 && f > lds_peek(&ctl->shared_floor)) lds_poke(&ctl->shared_floor, f);   // (a racing lower store is still a floor)
            top.floor_ge = fmaxf(top.floor_ge, f);
        }
        const uint32_t t = bounds.threshold(top.floor_ge, M);
        uint32_t any = ~0u;
        if constexpr (decltype(bounded)::value) {
            uint32_t sum[IPV];
            any = 0;
#pragma unroll
            for (int j = 0; j < VPI; ++j) {
                constexpr int kIds = 16 / CW;                  // of a vector
                uint32_t x[kIds];
#pragma unroll
                for (int c = 0; c < kIds; ++c) {
                    const uint32_t word = w[4 * j + c * CW / 4], id = CW == 2 ? (c & 1 ? word >> 16 : word & 0xFFFFu) : (word >> (c % 4 * 8)) & 0xFFu;
                    x[c] = counts[(j * kIds + c) % M * count_stride + id];
                }
#pragma unroll
                for (int c = 0; c < kIds; ++c) {
                    const int e = P > 16 ? 0 : c / M;
                    sum[e] = (P > 16 ? j == 0 && c == 0 : c % M == 0) ? x[c] : sum[e] + x[c];
                }
            }
#pragma unroll
            for (int e = 0; e < IPV; ++e) any = any > sum[e] ? any : sum[e];
        }
        const uint32_t p = piece_of(i);
        const bool hit = any >= t && p <= last;
        const uint64_t hits = __builtin_amdgcn_ballot_w64(hit);
        if constexpr (decltype(bounded)::value) {
            if (hits == 0) { credit = kMostCredit; return; }
            if (__builtin_expect(__popcll(hits) >= kManyLanes, 0)) {
                credit -= 2;
                if (credit < 0) until = 0;
            } else {
                credit = kMostCredit;
            }
        } else if (--credit < 0) {
            until = 0;
        }
        float sc[IPV];
        if (hit) score(w, sc);                                 // (the lookups of a few lanes collide less)
#pragma unroll
        for (int e = 0; e < IPV; ++e) {
            const bool take = hit && sc[e] >= top.floor_ge;
            const uint64_t mask = __ballot(take);
            if (mask != 0) {
                if (take) atomicAdd(&L.hist[bucket_of(sc[e], hlo, hscale)], 1u);
                top.append(mask, take, sc[e], p * IPV + (uint32_t)e, lane);
            }
        }
        // A list that has been sorted: K of its keys are no worse than the K-th, and what this wave has yet to see has higher ids than all of them, so
        // ties with the K-th come too late.  (All scores alike, 50M items, m = 8, K = 10: 1217 us without this, 115.)
        if (__builtin_expect(top.sorted, 0)) {
            top.sorted = false;
            const float kth = score_of_key(top.thr);
            if (lane == 0 && kth > lds_peek(&ctl->shared_floor)) lds_poke(&ctl->shared_floor, kth);
            top.floor_ge = fmaxf(top.floor_ge, next_up(kth));
        }
    };
    // Units are handed out by a counter in LDS: waves that fall behind do not hold the others up.  (A request is answered a unit later.)
    int pending = 0;
    auto request = [&]() { if (lane == 0) pending = (int)__builtin_amdgcn_atomic_inc32(reinterpret_cast<uint32_t*>(&ctl->next_unit), ~0u, __ATOMIC_RELAXED, "workgroup"); };
    request();
    bool seen = wave < sampling;
    auto stream = [&](auto bounded) {
        while (unit[0] < until) {                              // (slot 0 holds the older one)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (!seen && unit[i] < units) process(bounded, w[i], unit[i]);
                seen = false;
                unit[i] = (uint32_t)__builtin_amdgcn_readfirstlane(pending);
                request();
                fetch(unit[i], w[i]);
            }
        }
    };
    while (unit[0] < units) {
        stream(std::true_type());
        credit = rest;
        until = units;
        rest = rest < kMostRest ? 2 * rest : kMostRest;
        stream(std::false_type());
        credit = 0;
        until = units;
    }
    if constexpr (P <= 16) {
        // the fewer than 16 / P items after the last whole code vector, one per lane of one wave
        if (blk == 0 && wave == 0) {
            const uint32_t item = n_scan + (uint32_t)lane;
            float sc = 0.0f;
            bool take = false;
            if (item < (uint32_t)a.N) {
                const uint8_t* const row = a.codes + (size_t)item * P;
                auto id = [&](int k) -> uint32_t { return CW == 2 ? (uint32_t)reinterpret_cast<const uint16_t*>(row)[k] : (uint32_t)row[k]; };
                sc = lut[id(0)];
#pragma unroll
                for (int k = 1; k < M; ++k) sc = sc + lut[k * stride + id(k)];
                take = sc >= top.floor_ge;
            }
            const uint64_t mask = __ballot(take);
            if (mask != 0) top.append(mask, take, sc, item, lane);
        }
    }
    stamp<STAMP>(rec, kStampStreamed, lane);
    workgroup_select<NT>(L, ctl, top, K, a.cap, a.candmax, tid, K >= 32, hlo, hscale);
    stamp<STAMP>(rec, kStampSelected, lane);
    for (int t = tid; t < K; t += NT) emit_key(a, q, nblk, blk, t, L.sorted[t]);
    stamp<STAMP>(rec, kStampEnd, lane);
}
