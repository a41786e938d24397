// TopK for small K straight from registers: the selection shared by the short catalogue scan and the small fold.
// Part of kernels.hpp, which includes these parts inside namespace pqk in this order:
// common.hpp, subitem_scores.hpp, topk_parts.hpp, select_small.hpp, scan_single.hpp, scan_bytes.hpp, scan_short.hpp, scan_pair.hpp, scan_long.hpp, scan_subset.hpp,
// scan_batched.hpp, scan_filter.hpp, fold.hpp, comparison.hpp.
//
// These kernels run for a few microseconds with two to four waves per SIMD, so a wave's time is its instruction count
// (a vector instruction occupies its SIMD for four cycles) plus the latencies it cannot hide: everything here is
// written for few instructions and few LDS round trips, not for throughput.
#pragma once

// K up to which a workgroup's scan selects by select_small_k(); above, select_mid_k(), with two barriers more, ranks fewer candidates, the
// more so the more scores a thread holds.  `row`: bytes of an item's row.  One user's steps without Eq. 4 (us; small and mid): m = 4,
// 10,000 items, K = 2 4.5 and 5.4, 5 5.2 and 5.4, 10 6.3 and 5.5; 1M, K = 2 7.0 and 7.0, 5 7.7 and 7.4, 10 8.1 and 7.6; m = 8, 1.28M, K = 5 8.6 and
// 8.7, 10 9.0 and 8.9, 12 9.5 and 9.2, 8000, K = 10 6.0 and 6.8; m = 16, 600,000, K = 12 9.6 and 9.0; m = 32, 500,000, K = 12 10.2 and 10.3.
__host__ __device__ constexpr int small_k_max(int row) { return row == 4 ? 3 : row <= 16 ? 10 : 12; }
constexpr int kSmallCand = 512;                       // keys of its candidate array
constexpr int kSmallFloorSteps = 3;                   // four-way search steps of a wave's floor: a 64th of the lanes' range (5 % more candidates than the exact floor gives)

// An empty slot's score: a quiet NaN.  It never wins a maximum and no comparison with it holds, so empty slots need
// no flags of their own (scores of items are never NaN: the inputs are finite).
__device__ __forceinline__ float empty_score() { return __uint_as_float(0x7FC00000u); }

// LDS a workgroup needs for select_small_k(): the candidate array (16-byte aligned), one key per wave, a counter.
template <int NT>
struct SmallSelectLds {
    uint64_t cand[kSmallCand];
    uint64_t wave_best[NT / kWave];
    int ncand;
    uint32_t floor_bits;   // order-preserving image of the highest floor a wave has found so far (0: none yet)
};

// Before the workgroup barrier that precedes select_small_k(): an empty candidate array and counter.
template <int NT>
__device__ __forceinline__ void small_select_clear(SmallSelectLds<NT>& L, int tid) {
    static_assert(kSmallCand % 2 == 0, "cleared two keys at a time");
    for (int i = tid; i < kSmallCand / 2; i += NT) reinterpret_cast<ulonglong2*>(L.cand)[i] = make_ulonglong2(0ull, 0ull);
    if (tid == 0) { L.ncand = 0; L.floor_bits = 0u; }
}

// max over the wave of a 64-bit key, in every lane (DPP steps inside quads and rows, readlane across the four rows)
template <int CTRL>
__device__ __forceinline__ uint64_t dpp_max_key(uint64_t k) {
    const uint32_t lo = dpp_u32<CTRL>((uint32_t)k, (uint32_t)k), hi = dpp_u32<CTRL>((uint32_t)(k >> 32), (uint32_t)(k >> 32));
    const uint64_t o = ((uint64_t)hi << 32) | lo;
    return o > k ? o : k;
}
__device__ __forceinline__ uint64_t wave_max_key(uint64_t k) {
    k = dpp_max_key<kDppQuadSwap1>(k);
    k = dpp_max_key<kDppQuadSwap2>(k);
    k = dpp_max_key<kDppRowHalfMirror>(k);
    k = dpp_max_key<kDppRowMirror>(k);
    uint64_t best = 0;
#pragma unroll
    for (int row = 0; row < 4; ++row) {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)k, row * 16);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(k >> 32), row * 16);
        const uint64_t o = ((uint64_t)hi << 32) | lo;
        best = o > best ? o : best;
    }
    return best;
}

// Sorted exact K best of the n keys in cand[0..n) (LDS; zero up to the next multiple of 8) by counting: a key's position
// is the number of keys that beat it.  Rank r goes to emit(r, key); ranks from n on (fewer than K keys exist) get 0.
// With four or two threads per key each counts over a part of the keys (the loop is bound by the latency of its LDS reads).
// No barrier inside: the caller's barrier has made cand[] complete.
template <int NT, typename Emit>
__device__ __forceinline__ void rank_emit(const uint64_t* cand, int n, int K, int tid, Emit&& emit) {
    const int n8 = (n + 7) & ~7;
    auto count8 = [&](int u, uint64_t mine) -> uint32_t {
        const ulonglong2 p0 = *reinterpret_cast<const ulonglong2*>(cand + u);
        const ulonglong2 p1 = *reinterpret_cast<const ulonglong2*>(cand + u + 2);
        const ulonglong2 p2 = *reinterpret_cast<const ulonglong2*>(cand + u + 4);
        const ulonglong2 p3 = *reinterpret_cast<const ulonglong2*>(cand + u + 6);
        return (uint32_t)((p0.x > mine) + (p0.y > mine) + (p1.x > mine) + (p1.y > mine) + (p2.x > mine) + (p2.y > mine) +
                          (p3.x > mine) + (p3.y > mine));
    };
    auto shared = [&](auto lanes) {                           // (n8 is a multiple of 8: four lanes of a key are all in or all out)
        constexpr int kLanes = decltype(lanes)::value;
        const int t = tid / kLanes, part = tid % kLanes;
        if (t < n8) {
            const uint64_t mine = cand[t];
            uint32_t rank = 0;
#pragma unroll 2
            for (int u = part * 8; u < n8; u += kLanes * 8) rank += count8(u, mine);
            rank += dpp_u32<kDppQuadSwap1>(0u, rank);
            if constexpr (kLanes == 4) rank += dpp_u32<kDppQuadSwap2>(0u, rank);
            if (part == 0 && mine != 0ull && rank < (uint32_t)K) emit((int)rank, mine);
        }
    };
    if (n8 * 4 <= NT) {
        shared(std::integral_constant<int, 4>());
    } else if (n8 * 2 <= NT) {
        shared(std::integral_constant<int, 2>());
    } else {
        for (int t = tid; t < n; t += NT) {
            const uint64_t mine = cand[t];
            uint32_t rank = 0;
            for (int u = 0; u < n8; u += 8) rank += count8(u, mine);
            if (mine != 0ull && rank < (uint32_t)K) emit((int)rank, mine);
        }
    }
    for (int t = n + tid; t < K; t += NT) emit(t, 0ull);
}

// The workgroup's exact, sorted K best (1 <= K < kRegisterSelectMinK: a wave's 64 lanes give its floor) of the items its threads hold in registers: thread-local
// slots i = 0 .. R-1 with score sc[i] (empty_score() where a slot holds nothing) and item id id_of(i).  Rank r goes to
// emit(r, key) (0 for ranks that do not exist).  L: cleared by small_select_clear() before the caller's last barrier.
//
// Every wave finds, with wave operations only, a floor that K of its lanes' best scores reach; every one of the wave's K
// best items reaches it, and few others do (a dozen of a wave's hundreds of scores at K = 10).  One ballot per slot
// marks them.  Usually no lane holds two (the ballots' population counts tell): a lane then picks its one candidate by
// the ballots, positions come from the union of the ballots and ONE counter update per wave, and the wave makes one LDS
// write.  Otherwise lanes count their candidates, positions come from a prefix sum, and each lane writes its j-th
// candidate in the wave's j-th write.  After one barrier the workgroup ranks the candidates by counting.  More
// candidates than the array holds (heavy ties) take a slow path that is exact for any input: K times, the best
// remaining key of the workgroup is found and emitted.
// STAMP / rec: measurement instances record wall-clock stamps (candidates written, K best ranked).
template <int NT, int R, bool STAMP = false, typename IdOf, typename Emit>
__device__ __forceinline__ void select_small_k(const float (&sc)[R], IdOf&& id_of, int K, SmallSelectLds<NT>& L, int tid,
                                               Emit&& emit, uint64_t* rec = nullptr) {
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    float best = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < R; ++i) best = fmaxf(best, sc[i]);    // (an empty slot's NaN never wins)
    // A floor that some wave has found holds for the whole workgroup (that wave alone has K items at or above it), so a
    // wave that gets here later takes it and saves the search.  (In the short scan the second wave of every SIMD
    // finishes its lookups most of a microsecond after the first: its selection is what the workgroup waits for.)
    const uint32_t seen = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_peek(&L.floor_bits));
    float f;
    if (seen != 0u) {
        f = float_of_orderable(seen);
    } else {
        f = wave_floor_for_k<kSmallFloorSteps>(best, K);
        if (lane == 0 && f > -__builtin_inff()) atomicMax(&L.floor_bits, orderable_bits(f));
    }
    bool mine[R];                                             // this lane's slot i is a candidate
    bool any_mine = false;
    uint64_t any = 0ull;
    int total = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        mine[i] = sc[i] >= f;
        const uint64_t mask = __ballot(mine[i]);
        any_mine = any_mine || mine[i];
        any |= mask;
        total += __popcll(mask);
    }
    int base = 0;
    if (lane == 0 && total != 0) base = atomicAdd(&L.ncand, total);
    if (total == __popcll(any)) {
        // no lane holds two candidates: a lane's candidate is its one marked slot
        float s = 0.0f;
        uint32_t item = 0;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            s = mine[i] ? sc[i] : s;
            item = mine[i] ? id_of(i) : item;
        }
        base = __builtin_amdgcn_readfirstlane(base);
        const int pos = base + __popcll(any & ((1ull << lane) - 1ull));
        if (any_mine && pos < kSmallCand) L.cand[pos] = make_key(s + 0.0f, item);
    } else {
        uint32_t c = 0;
#pragma unroll
        for (int i = 0; i < R; ++i) c += mine[i] ? 1u : 0u;
        const uint32_t upto = wave_prefix_sum(c);
        base = __builtin_amdgcn_readfirstlane(base);
        const int pos = base + (int)(upto - c);
        for (uint32_t j = 0; __ballot(c > j) != 0; ++j) {     // the wave's j-th write: every lane's j-th candidate
            float s = 0.0f;
            uint32_t item = 0, seen = 0;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const bool hit = mine[i] && seen == j;
                s = hit ? sc[i] : s;
                item = hit ? id_of(i) : item;
                seen += mine[i] ? 1u : 0u;
            }
            if (c > j && pos + (int)j < kSmallCand) L.cand[pos + (int)j] = make_key(s + 0.0f, item);
        }
    }
    stamp<STAMP>(rec, kStampOffered, lane);
    __syncthreads();
    const int n = L.ncand;
    if (n <= kSmallCand) {
        rank_emit<NT>(L.cand, n, K, tid, emit);
        stamp<STAMP>(rec, kStampSelected, lane);
        return;
    }
    // heavy ties: more candidates than the array holds
    uint64_t last = ~0ull;                                    // every key is smaller
    for (int r = 0; r < K; ++r) {
        uint64_t mine = 0ull;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint64_t key = make_key(sc[i] + 0.0f, id_of(i));
            if (sc[i] == sc[i] && key < last && key > mine) mine = key;   // (sc == sc: the slot holds an item)
        }
        mine = wave_max_key(mine);
        if (lane == 0) L.wave_best[wave] = mine;
        __syncthreads();
        uint64_t top = 0ull;
#pragma unroll
        for (int w = 0; w < NT / kWave; ++w) top = L.wave_best[w] > top ? L.wave_best[w] : top;
        if (tid == 0) emit(r, top);                           // (0 once nothing is left)
        last = top;                                           // (0: no key is smaller, the remaining ranks get 0)
        __syncthreads();
    }
}

// ---- larger K
constexpr int kMidCand = 1408;                        // keys of the candidate array
constexpr int kMidBins = 256;                         // buckets of the histogram of the threads' best scores

template <int NT>
struct MidSelectLds {
    uint64_t cand[kMidCand];
    uint32_t hist[kBins];                             // (kMidBins counters of it, then the buckets of the final order)
    float wave_min[NT / kWave], wave_max[NT / kWave];
    int ncand;
};

// Before the workgroup barrier that precedes select_mid_k().
template <int NT>
__device__ __forceinline__ void mid_select_clear(MidSelectLds<NT>& L, int tid) {
    for (int i = tid; i < kMidBins; i += NT) L.hist[i] = 0u;
    if (tid == 0) L.ncand = 0;
}

// As select_small_k(), for K <= 2 * NT.  The floor is one that K of the THREADS' best scores reach
// (K > NT / 2: of the best of their even and of their odd slots), taken from a histogram of those alone: 512 counts instead
// of the 11,000 that all scores would be, and for K = 100 only a tenth more candidates than K: three barriers, then the
// candidates are ordered.  (1.28M items, one user: K = 100 18.4 -> 16.6 us per step, K = 31 18.0 -> 14.9; where it beats
// the waves' own floors, which let eight times K pass: small_k_max().)
// More candidates than the array holds (heavy ties): the exact K-th key is found bit by bit first.
// Between its barriers: mid_range() the threads' best scores and their range, mid_count() the histogram, mid_collect() the
// candidates, mid_order() (with barriers of its own) the candidates in order.
struct MidBest { float best, other, lo, hi, scale; };
template <int NT, int R>
__device__ __forceinline__ MidBest mid_range(const float (&sc)[R], int K, MidSelectLds<NT>& L, int tid) {
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const float ninf = -__builtin_inff();
    float best = ninf, other = ninf;
#pragma unroll
    for (int i = 0; i < R; ++i) {                             // (an empty slot's NaN never wins)
        if (i % 2 == 0) best = fmaxf(best, sc[i]);
        else other = fmaxf(other, sc[i]);
    }
    const bool both = K > NT / 2;
    if (!both) { best = fmaxf(best, other); other = ninf; }
    float mx = fmaxf(best, other), mn = fminf(best > ninf ? best : -ninf, other > ninf ? other : -ninf);
    wave_minmax(mn, mx);
    if (lane == 0) { L.wave_min[wave] = mn; L.wave_max[wave] = mx; }
    return {best, other, 0.0f, 0.0f, 0.0f};
}
template <int NT>
__device__ __forceinline__ void mid_count(MidBest& t, int K, MidSelectLds<NT>& L) {
    constexpr int NW = NT / kWave;
    const float ninf = -__builtin_inff();
    t.lo = L.wave_min[0]; t.hi = L.wave_max[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) { t.lo = fminf(t.lo, L.wave_min[w]); t.hi = fmaxf(t.hi, L.wave_max[w]); }
    t.scale = t.hi > t.lo ? (float)kMidBins / (t.hi - t.lo) : 0.0f;
    if (!(t.scale > 0.0f) || t.scale > 3.0e38f) t.scale = 0.0f;
    if (t.best > ninf) atomicAdd(&L.hist[bucket_of<kMidBins>(t.best, t.lo, t.scale)], 1u);
    if (K > NT / 2 && t.other > ninf) atomicAdd(&L.hist[bucket_of<kMidBins>(t.other, t.lo, t.scale)], 1u);
}
// returns the floor
template <int NT, int R, typename IdOf>
__device__ __forceinline__ float mid_collect(const float (&sc)[R], IdOf&& id_of, const MidBest& t, int K, MidSelectLds<NT>& L, int tid) {
    const int lane = tid & (kWave - 1);
    const float f = floor_of_hist<kMidBins>(L.hist, K, t.lo, t.scale, lane);   // (every wave for itself)
    int total = 0;
#pragma unroll
    for (int i = 0; i < R; ++i) total += __popcll(__ballot(sc[i] >= f));
    if (total != 0) {
        int at = 0;
        if (lane == 0) at = atomicAdd(&L.ncand, total);
        at = __builtin_amdgcn_readfirstlane(at);
        float again = f;                                      // (compared anew: R masks do not fit the scalar registers)
        asm volatile("" : "+v"(again));
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const uint64_t mask = __ballot(sc[i] >= again);
            if (mask == 0) continue;
            const int pos = at + __popcll(mask & ((1ull << lane) - 1ull));
            if (sc[i] >= again && pos < kMidCand) L.cand[pos] = make_key(sc[i] + 0.0f, id_of(i));
            at += __popcll(mask);
        }
    }
    return f;
}
template <int NT, int R, typename IdOf, typename Emit>
__device__ __forceinline__ void mid_order(const float (&sc)[R], IdOf&& id_of, float f, float hi, int K, MidSelectLds<NT>& L, int tid, Emit&& emit) {
    constexpr int NW = NT / kWave;
    const int lane = tid & (kWave - 1), wave = tid / kWave;
    const float ninf = -__builtin_inff();
    int n = L.ncand;
    if (n > kMidCand) {
        // the K-th best key: the largest that K keys reach (K keys exist: there are more than kMidCand)
        uint64_t kth = 0ull;
        for (int bit = 63; bit >= 0; --bit) {
            const uint64_t t = kth | (1ull << bit);
            int reach = 0;
#pragma unroll
            for (int i = 0; i < R; ++i) {
                float x = sc[i];                              // (made anew in every step: R keys do not fit the registers)
                asm volatile("" : "+v"(x));
                reach += __popcll(__ballot(x == x && make_key(x + 0.0f, id_of(i)) >= t));
            }
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
        __syncthreads();
        n = L.ncand;                                          // = K: keys are distinct
    }
    if (n <= kRankByCount) {
        const int n8 = (n + 7) & ~7;
        if (tid < n8 - n) L.cand[n + tid] = 0ull;
        __syncthreads();
        rank_emit<NT>(L.cand, n, K, tid, emit);
    } else {
        // by buckets over the candidates' own range (from the floor up, where there is one)
        float lo = f;
        if (!(f > ninf)) {
            float mn = -ninf;
            for (int t = tid; t < n; t += NT) mn = fminf(mn, score_of_key(L.cand[t]));
            float mx = mn;
            wave_minmax(mn, mx);
            if (lane == 0) L.wave_min[wave] = mn;
            __syncthreads();
            lo = L.wave_min[0];
#pragma unroll
            for (int w = 1; w < NW; ++w) lo = fminf(lo, L.wave_min[w]);
        }
        float scale = hi > lo ? (float)kBins / (hi - lo) : 0.0f;
        if (!(scale > 0.0f) || scale > 3.0e38f) scale = 0.0f;
        if (!bucket_sort<NT, (kMidCand + NT - 1) / NT>(L.cand, n, lo, scale, L.hist, tid)) {
            // (too many in one bucket: by counting, from registers to their places)
            uint64_t mine[(kMidCand + NT - 1) / NT];
            int rank[(kMidCand + NT - 1) / NT];
#pragma unroll
            for (int r = 0; r < (kMidCand + NT - 1) / NT; ++r) {
                mine[r] = r * NT + tid < n ? L.cand[r * NT + tid] : 0ull;
                rank[r] = 0;
            }
            for (int u = 0; u < n; ++u) {
                const uint64_t x = L.cand[u];
#pragma unroll
                for (int r = 0; r < (kMidCand + NT - 1) / NT; ++r) rank[r] += x > mine[r];
            }
#pragma unroll
            for (int r = 0; r < (kMidCand + NT - 1) / NT; ++r)
                if (mine[r] != 0ull && rank[r] < K) emit(rank[r], mine[r]);
            for (int t = n + tid; t < K; t += NT) emit(t, 0ull);
            return;
        }
        for (int t = tid; t < K; t += NT) emit(t, t < n ? L.cand[t] : 0ull);
    }
}
template <int NT, int R, bool STAMP = false, typename IdOf, typename Emit>
__device__ __forceinline__ void select_mid_k(const float (&sc)[R], IdOf&& id_of, int K, MidSelectLds<NT>& L, int tid, Emit&& emit,
                                             uint64_t* rec = nullptr) {
    const int lane = tid & (kWave - 1);
    MidBest t = mid_range<NT>(sc, K, L, tid);
    __syncthreads();
    mid_count<NT>(t, K, L);
    __syncthreads();
    const float f = mid_collect<NT>(sc, id_of, t, K, L, tid);
    stamp<STAMP>(rec, kStampOffered, lane);
    __syncthreads();
    mid_order<NT>(sc, id_of, f, t.hi, K, L, tid, emit);
    stamp<STAMP>(rec, kStampSelected, lane);
}
// The same for two queries' scores of the same items, with one set of barriers up to the candidates; few candidates are ranked by
// half of the threads for each query.  (For K <= 12 too: the waves' own floors of select_small_k() let twice the candidates through,
// more than its array holds: 1.28M items, two-byte sub-ids, four queries: 20.9 us per step, with this 14.9.)  emit(h, rank, key): of query h.
template <int NT, int R, typename IdOf, typename Emit>
__device__ __forceinline__ void select_mid_k_pair(const float (&sc)[2][R], IdOf&& id_of, int K, MidSelectLds<NT> (&L)[2], int tid, Emit&& emit) {
    MidBest t[2] = {mid_range<NT>(sc[0], K, L[0], tid), mid_range<NT>(sc[1], K, L[1], tid)};
    __syncthreads();
    mid_count<NT>(t[0], K, L[0]);
    mid_count<NT>(t[1], K, L[1]);
    __syncthreads();
    const float f0 = mid_collect<NT>(sc[0], id_of, t[0], K, L[0], tid);
    const float f1 = mid_collect<NT>(sc[1], id_of, t[1], K, L[1], tid);
    __syncthreads();
    const int n0 = L[0].ncand, n1 = L[1].ncand;
    if (n0 <= kRankByCount && n1 <= kRankByCount) {
        const int h = __builtin_amdgcn_readfirstlane(tid >= NT / 2 ? 1 : 0), me = tid - h * (NT / 2);
        const int n = h != 0 ? n1 : n0, n8 = (n + 7) & ~7;
        if (me < n8 - n) L[h].cand[n + me] = 0ull;
        __syncthreads();
        rank_emit<NT / 2>(L[h].cand, n, K, me, [&](int rank, uint64_t key) { emit(h, rank, key); });
        return;
    }
    mid_order<NT>(sc[0], id_of, f0, t[0].hi, K, L[0], tid, [&](int rank, uint64_t key) { emit(0, rank, key); });
    mid_order<NT>(sc[1], id_of, f1, t[1].hi, K, L[1], tid, [&](int rank, uint64_t key) { emit(1, rank, key); });
}
