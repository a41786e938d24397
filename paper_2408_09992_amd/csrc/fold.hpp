// The last launch of every TopK call: the workgroups' lists -> the final sorted K per query (fold_lists_kernel,
// fold_small_kernel).
// Part of kernels.hpp, which includes these parts inside namespace pqk in this order:
// common.hpp, subitem_scores.hpp, topk_parts.hpp, select_small.hpp, scan_single.hpp, scan_bytes.hpp, scan_short.hpp, scan_pair.hpp, scan_long.hpp, scan_subset.hpp,
// scan_batched.hpp, scan_filter.hpp, fold.hpp, comparison.hpp.
#pragma once

struct FoldArgs {
    const uint64_t* ws_keys;   // [B][nlists][K]: per query, nlists lists of K keys, sorted best first, zeros at the end
    int nlists, K;
    int chunk, depth, need, groups, group_mask;   // fold_lists_kernel: see there
    int* out_ids;              // [B][K]
    float* out_scores;
    uint64_t* stamps;          // STAMP instances only: wall-clock stamps, kStampSlots per wave
};

constexpr int kFoldThreads = 1024;                // a CU per query: as many threads as a workgroup has (238 queries, K = 440: 8.8 us with 256, 5.7)
constexpr int kFoldThreadsMany = 256;             // more queries: several workgroups per CU (1024 queries, K = 100: 13.6 us with 1024, 8.3)
constexpr int kFoldSlots = 4096;                  // keys read at first: nlists * chunk at most
constexpr int kFoldLists = 1024;                  // lists per query at most
constexpr int kFoldCand = 2048;                   // candidates ranked at most; more (heavy ties in few lists) take the slow path

// Dynamic LDS: hist | ctl | stage (kFoldCand keys; first the groups' floor scores and the lists to read on in) | cand | sorted
__host__ __device__ inline size_t fold_lds_bytes(int K) {
    return kBins * sizeof(uint32_t) + align16(sizeof(Ctl)) + 2 * (size_t)kFoldCand * sizeof(uint64_t) + align16((size_t)K * sizeof(uint64_t));
}

// The fold for any K.  grid = (1, B).  The lists are sorted, so few keys decide: `need` lists whose key number `depth` is at
// least f hold need * depth >= K keys that are.  So the need-th largest of the lists' depth-th keys is a floor of the K-th
// best, and only keys that reach it are ranked: about 1.3 K of them.  The floor is found by comparing every list's score with
// every other's, so where far fewer lists are needed than there are, each of `groups` groups of lists puts forward its best
// only (512 lists of K = 15: 15.2 us for the kernel, with 64 groups 5).  A list's first `chunk` keys are read at once (chunk
// covers a list's share of the K best and what chance adds to it), lists that reach the floor with all of them are read on,
// chunk after chunk.  One round trip to memory, usually; reading everything instead took two launches for 256 lists of
// K = 100 (25,600 keys: sixteen folds of sixteen lists, then one: 12 us; this: 4 us).
template <int NT, bool STAMP = false>
__global__ __launch_bounds__(NT) void fold_lists_kernel(FoldArgs a) {
    constexpr int R = kFoldSlots / NT;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int n_cand, n_more[2];
    __shared__ uint32_t floor_score;
    uint32_t* hist = reinterpret_cast<uint32_t*>(smem);
    Ctl* ctl = reinterpret_cast<Ctl*>(smem + kBins * sizeof(uint32_t));
    uint64_t* stage = reinterpret_cast<uint64_t*>(smem + kBins * sizeof(uint32_t) + align16(sizeof(Ctl)));
    uint64_t* cand = stage + kFoldCand;
    uint64_t* sorted = cand + kFoldCand;
    uint32_t* heads = reinterpret_cast<uint32_t*>(stage);     // [kFoldLists], ordered as the scores they stand for
    int* more[2] = {reinterpret_cast<int*>(stage + kFoldLists), reinterpret_cast<int*>(stage + kFoldLists) + kFoldLists};
    static_assert(2 * kFoldLists * sizeof(int) <= (kFoldCand - kFoldLists) * sizeof(uint64_t), "room for both lists of lists");
    const int tid = threadIdx.x, lane = tid & (kWave - 1), q = blockIdx.y, K = a.K, nlists = a.nlists;
    uint64_t* const rec = STAMP ? a.stamps + ((size_t)q * (NT / kWave) + tid / kWave) * kStampSlots : nullptr;
    stamp<STAMP>(rec, kStampEntry, lane);
    const uint64_t* all = a.ws_keys + (size_t)q * nlists * K;
    const int cshift = 31 - __builtin_clz((uint32_t)a.chunk);   // (a power of two)
    auto emit = [&](int rank, uint64_t key) {
        a.out_ids[(size_t)q * K + rank] = id_of_key(key);
        a.out_scores[(size_t)q * K + rank] = score_of_key(key);
    };

    uint64_t keys[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * NT + tid, list = i >> cshift, pos = i & (a.chunk - 1);
        keys[r] = (list < nlists && pos < K) ? all[(size_t)list * K + pos] : 0ull;
    }
    if (tid == 0) { n_cand = 0; n_more[0] = n_more[1] = 0; floor_score = 0xFFFFFFFFu; }
    for (int g = tid; g < a.groups; g += NT) heads[g] = 0u;
    __syncthreads();                                          // (while the keys are under way)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * NT + tid, list = i >> cshift, pos = i & (a.chunk - 1);
        if (list < nlists && pos == a.depth - 1) atomicMax(&heads[list & a.group_mask], (uint32_t)(keys[r] >> 32));
    }
    __syncthreads();
    stamp<STAMP>(rec, kStampLoaded, lane);

    // ---- the need-th largest of the groups' scores: the smallest that fewer than `need` others beat (not that many lists so
    // long: zero, no floor)
    for (int part_of = tid; part_of < a.groups * 4; part_of += NT) {   // four lanes per group, each over a quarter of the others
        const int part = part_of & 3;
        const uint32_t mine = heads[part_of >> 2];
        uint32_t rank = 0;
        for (int u = part * 4; u < a.groups; u += 16) {
            const uint4 others = *reinterpret_cast<const uint4*>(heads + u);
            rank += (others.x > mine) + (others.y > mine) + (others.z > mine) + (others.w > mine);
        }
        rank += dpp_u32<kDppQuadSwap1>(0u, rank);
        rank += dpp_u32<kDppQuadSwap2>(0u, rank);
        if (part == 0 && rank < (uint32_t)a.need) atomicMin(&floor_score, mine);
    }
    __syncthreads();
    stamp<STAMP>(rec, kStampCut, lane);
    const uint64_t f = floor_score != 0u ? (uint64_t)floor_score << 32 : 1ull;   // (every key is at least 1)

    // ---- what reaches it
    auto take = [&](uint64_t key) {
        const bool in = key >= f;
        const uint64_t mask = __ballot(in);
        if (mask == 0) return;
        int base = 0;
        if (lane == __builtin_ctzll(mask)) base = atomicAdd(&n_cand, __popcll(mask));
        base = __builtin_amdgcn_readlane(base, __builtin_ctzll(mask));
        const int pos = base + __popcll(mask & ((1ull << lane) - 1ull));
        if (in && pos < kFoldCand) cand[pos] = key;
    };
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * NT + tid, list = i >> cshift, pos = i & (a.chunk - 1);
        take(keys[r]);
        if (keys[r] >= f && pos == a.chunk - 1 && a.chunk < K) more[0][atomicAdd(&n_more[0], 1)] = list;
    }
    __syncthreads();
    int n = n_more[0];
    for (int off = a.chunk, turn = 0; n != 0; off += a.chunk, turn ^= 1) {   // (the same n for the whole workgroup; ends at off >= K)
        const int slots = (n << cshift);
        for (int i0 = 0; i0 < slots; i0 += NT) {
            const int i = i0 + tid, pos = off + (i & (a.chunk - 1));
            const int list = i < slots ? more[turn][i >> cshift] : 0;
            const uint64_t key = (i < slots && pos < K) ? all[(size_t)list * K + pos] : 0ull;
            take(key);
            if (key >= f && (i & (a.chunk - 1)) == a.chunk - 1 && pos + 1 < K) more[turn ^ 1][atomicAdd(&n_more[turn ^ 1], 1)] = list;
        }
        __syncthreads();
        n = n_more[turn ^ 1];
        if (tid == 0) n_more[turn] = 0;
        __syncthreads();
    }
    stamp<STAMP>(rec, kStampCollected, lane);
    const int c = n_cand;
    if (c <= kFoldCand) {
        if (c > kRankByCount) {
            // by buckets over the candidates' own range
            float mn = __builtin_inff(), mx = -__builtin_inff(), lo, scale;
            for (int t = tid; t < c; t += NT) { const float v = score_of_key(cand[t]); mn = fminf(mn, v); mx = fmaxf(mx, v); }
            set_range<NT / kWave>(mn, mx, ctl, tid, lo, scale);
            if (!bucket_sort<NT, kFoldCand / NT>(cand, c, lo, scale, hist, tid)) {
                const int padded = pow2_at_least(c);
                for (int t = c + tid; t < padded; t += NT) cand[t] = 0ull;
                block_sort_desc<NT>(cand, padded, tid);
            }
            for (int t = tid; t < K; t += NT) emit(t, t < c ? cand[t] : 0ull);
        } else {
            const int c8 = (c + 7) & ~7;
            if (c + tid < c8) cand[c + tid] = 0ull;
            __syncthreads();
            rank_emit<NT>(cand, c, K, tid, emit);
        }
        stamp<STAMP>(rec, kStampSelected, lane);
        stamp<STAMP>(rec, kStampEnd, lane);
        return;
    }

    // ---- too many (a floor far below the K-th best: lists that share few of the best keys evenly): everything once more,
    // stage by stage
    __syncthreads();
    const long long nkeys = (long long)nlists * K;
    float mn = __builtin_inff(), mx = -__builtin_inff();
    for (long long i = tid; i < nkeys; i += NT) {
        const uint64_t key = all[i];
        if (key) { const float s = score_of_key(key); mn = fminf(mn, s); mx = fmaxf(mx, s); }
    }
    float lo, scale;
    set_range<NT / kWave>(mn, mx, ctl, tid, lo, scale);
    int keep = 0;                                             // best-so-far keys carried at the front of stage
    long long done = 0;
    while (done < nkeys) {
        long long n_in = nkeys - done;
        if (n_in > kFoldCand - keep) n_in = kFoldCand - keep;
        for (int t = tid; t < kFoldCand - keep; t += NT) stage[keep + t] = (t < n_in) ? all[done + t] : 0ull;
        __syncthreads();
        block_select<NT>(stage, kFoldCand, K, sorted, cand, kFoldCand, hist, ctl, tid);
        done += n_in;
        keep = K;
        if (done < nkeys) {
            for (int t = tid; t < K; t += NT) stage[t] = sorted[t];
            __syncthreads();
        }
    }
    for (int t = tid; t < K; t += NT) emit(t, sorted[t]);
}

// The fold for small K and few keys (nlists * K <= NT * R; the host's rule is fold_small_pays()): the keys go
// straight from memory to registers and through select_small_k(), the selection the short scan uses: per-wave floors
// by wave operations, one barrier, ranking by counting.  grid = (1, B).  A kernel of its own because this launch is all
// latency (a few thousand keys): its time is the two dependent memory round trips it cannot avoid (arguments, keys)
// plus its instruction count, and this one has a fifth of the general fold's instructions and a sixth of its barriers.
template <int NT, int R, bool STAMP = false>
__global__ __launch_bounds__(NT) void fold_small_kernel(const uint64_t* ws_keys, int* result_ids, float* result_scores, int nlists, int K,
                                                        uint64_t* stamps) {
    __shared__ SmallSelectLds<NT> sel;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), q = blockIdx.y;
    uint64_t* const rec = STAMP ? stamps + ((size_t)q * (NT / kWave) + tid / kWave) * kStampSlots : nullptr;
    stamp<STAMP>(rec, kStampEntry, lane);
    const int nkeys = nlists * K;
    const uint64_t* all = ws_keys + (size_t)q * nkeys;
    uint64_t keys[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = r * NT + tid;
        keys[r] = i < nkeys ? all[i] : 0ull;
    }
    small_select_clear<NT>(sel, tid);
    __syncthreads();
    float sc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) sc[r] = keys[r] != 0ull ? score_of_key(keys[r]) : empty_score();
    stamp<STAMP>(rec, kStampLoaded, lane);
    int* const out_ids = result_ids + (size_t)q * K;
    float* const out_scores = result_scores + (size_t)q * K;
    select_small_k<NT, R, STAMP>(sc, [&](int slot) -> uint32_t { return (uint32_t)id_of_key(keys[slot]); }, K, sel, tid,
                                 [&](int rank, uint64_t key) {
                                     out_ids[rank] = id_of_key(key);
                                     out_scores[rank] = score_of_key(key);
                                 }, rec);
    stamp<STAMP>(rec, kStampEnd, lane);
}
