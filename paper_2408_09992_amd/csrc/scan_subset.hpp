// Algorithm 1 with a candidate list V, for lists short enough that a workgroup's share fits its registers
// (scan_subset_kernel): lists of up to a couple of million candidates at batch 1.
// Part of kernels.hpp, which includes these parts inside namespace pqk in this order:
// common.hpp, subitem_scores.hpp, topk_parts.hpp, select_small.hpp, scan_single.hpp, scan_bytes.hpp, scan_short.hpp, scan_pair.hpp, scan_long.hpp, scan_subset.hpp,
// scan_batched.hpp, scan_filter.hpp, fold.hpp, comparison.hpp.
#pragma once

// Most 16-byte code vectors' worth of gathered rows a thread of the candidate-list kernel holds.
constexpr int kSubsetMaxVecs = 8;

// grid = (list blocks, B); one query per workgroup.  A thread holds R = U * (16 / M) candidates: slot s of thread t of
// workgroup g is position (s * blocks + g) * NT + t of the list (slot s of all workgroups together is one contiguous
// stretch of V: the ids are read coalesced).  Every id is requested first, then every row G[V[p]] (M bytes each,
// gathered where they lie: a random list costs a 32-byte sector per row), then the query's table goes to LDS; the rows
// of 16 / M candidates are packed into one code vector and scored by the scan's own routine (same lookups, same
// left-to-right sums), and the workgroup's K best come out of select_small_k(), keyed by ITEM id: ties go to the lower
// item id wherever it sits in the list.  The general kernel reads a row only when its turn comes and scores row after
// row; here all of a thread's rows are on their way at once, which is what a gather needs.
//   M: bytes of an item's row (4, 8 or 16); U: code vectors' worth of rows per thread (1 .. kSubsetMaxVecs)
// An id outside [0, n_items) is clamped to n_items - 1 (memory-safe; the result is then unspecified, as documented).
template <int M, int U, int NT>
__global__ __launch_bounds__(NT) void scan_subset_kernel(const uint8_t* codes, const int* subset, const float* S, void* out,
                                                         float* out_scores, uint32_t N, uint32_t n_items, int b, int K) {
    ScanArgs a;                                               // (plain arguments: see scan_short_kernel)
    a.codes = codes; a.subset = subset; a.S = S; a.N = N; a.n_items = n_items; a.m = M; a.b = b; a.K = K;
    a.ws_keys = static_cast<uint64_t*>(out); a.out_ids = out_scores != nullptr ? static_cast<int*>(out) : nullptr;
    a.out_scores = out_scores;
    constexpr int IPV = 16 / M, WPI = M / 4;                   // candidates per code vector, 4-byte words per row
    constexpr int R = U * IPV;
    static_assert(M == 4 || M == 8 || M == 16, "rows of 4, 8 or 16 bytes");
    static_assert(U >= 1 && U <= kSubsetMaxVecs, "vectors per thread");
    __shared__ __align__(16) float lut[M * kLutStride];
    extern __shared__ __align__(16) unsigned char smem[];     // what the selection needs, for this K
    const int tid = threadIdx.x;
    const int q = blockIdx.y, nblk = gridDim.x, blk = blockIdx.x;
    const uint32_t n = (uint32_t)a.N;                          // candidates in the list
    const uint32_t first = (uint32_t)blk * NT + (uint32_t)tid, stride = (uint32_t)nblk * NT;

    // ---- the ids (coalesced), then the rows they name
    uint32_t item[R];
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const uint32_t pos = first + (uint32_t)s * stride;
        item[s] = (uint32_t)a.subset[pos < n ? pos : n - 1];  // (past the end: a re-read, never scored)
    }
    // (up to rows of 8 bytes the query's table values are asked for between the ids and the rows, which wait for the ids: 1M candidates, m = 8, one query
    // 19.5 us with them after the rows, 18.7 so; 50,000, four queries 8.1 and 7.9; m = 16, whose table is larger: 200,000 11.7 and 11.9)
    const float* Sq = a.S + (size_t)q * M * b;
    constexpr int kPer = (M * kLutStride + NT - 1) / NT;
    float tv[kPer];
    auto ask_table = [&]() {
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int e = tid + i * NT, k = e / kLutStride, j = e % kLutStride;
            tv[i] = (e < M * kLutStride && j < b) ? Sq[k * b + j] : 0.0f;
        }
    };
    if constexpr (M <= 8) {
        ask_table();
        __builtin_amdgcn_sched_barrier(0);
    }
    uint32_t w[U][4];
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const uint32_t i = item[s] < a.n_items ? item[s] : a.n_items - 1;
        const uint32_t* row = reinterpret_cast<const uint32_t*>(a.codes + (size_t)i * M);
        if constexpr (M == 4) {
            w[s / IPV][s % IPV] = row[0];
        } else if constexpr (M == 8) {
            const uint2 x = *reinterpret_cast<const uint2*>(row);
            w[s / IPV][2 * (s % IPV)] = x.x; w[s / IPV][2 * (s % IPV) + 1] = x.y;
        } else {
            const uint4 x = *reinterpret_cast<const uint4*>(row);
            w[s][0] = x.x; w[s][1] = x.y; w[s][2] = x.z; w[s][3] = x.w;
        }
        item[s] = i;
    }
    static_assert(WPI * IPV == 4, "a code vector is four words");

    // ---- the query's table to LDS (rows padded with zeros to 256 entries), all values requested before the first store
    if constexpr (M <= 8) __builtin_amdgcn_sched_barrier(0);
    else ask_table();
#pragma unroll
    for (int i = 0; i < kPer; ++i)
        if (tid + i * NT < M * kLutStride) lut[tid + i * NT] = tv[i];
    if (K <= small_k_max(M)) small_select_clear<NT>(*reinterpret_cast<SmallSelectLds<NT>*>(smem), tid);
    else mid_select_clear<NT>(*reinterpret_cast<MidSelectLds<NT>*>(smem), tid);
    __syncthreads();

    // ---- Eq. 5 for every candidate this thread holds
    float sc[R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float part[IPV];
        score_vector<M, 1>(lut, w[u], part);
#pragma unroll
        for (int e = 0; e < IPV; ++e) {
            const int s = u * IPV + e;
            sc[s] = first + (uint32_t)s * stride < n ? part[e] : empty_score();
        }
    }

    // ---- the workgroup's K best, ranked, straight to the workspace or the result
    auto id_of = [&](int slot) -> uint32_t { return item[slot]; };
    auto emit = [&](int rank, uint64_t key) { emit_key(a, q, nblk, blk, rank, key); };
    if (K <= small_k_max(M)) select_small_k<NT, R>(sc, id_of, K, *reinterpret_cast<SmallSelectLds<NT>*>(smem), tid, emit);
    else select_mid_k<NT, R>(sc, id_of, K, *reinterpret_cast<MidSelectLds<NT>*>(smem), tid, emit);
}

// Most code vectors' worth of gathered rows a thread of the kernel below holds: up to 64 scores, of two queries each candidate.
__host__ __device__ constexpr int subset_pair_max(int m) { return m == 4 ? 8 : m == 8 ? 16 : 24; }
// its instances: 1, 2, 3, 4, 6, 8, 12, 16, 24
__host__ __device__ constexpr int subset_pair_instance(int vecs) {
    return vecs <= 4 ? vecs : vecs <= 6 ? 6 : vecs <= 8 ? 8 : vecs <= 12 ? 12 : vecs <= 16 ? 16 : 24;
}
__host__ __device__ constexpr bool subset_pair_has(int m, int u) { return u <= subset_pair_max(m) && subset_pair_instance(u) == u; }

// Candidate lists for several queries: as scan_subset_kernel, two queries per workgroup (grid.y = (B + 1) / 2), their tables' entries side
// by side in LDS as in scan_pair_kernel.  What bounds a list is the gathering of its rows, about one per clock and CU, and then the
// lookups: both are done once for two queries here.
// Rows are asked for behind the tables (see pair_tables()) but where a thread holds sixteen vectors: at m = 16 tables and rows together then take 132
// registers, and a compute unit has room for one workgroup instead of two (13,498 candidates, 899 queries 67.2 us, rows first 45.5; m = 8, 26,148, 491, K = 152 77.3
// and 74.3).
template <int M, int U, int NT>
__global__ __launch_bounds__(NT, 1) void scan_subset_pair_kernel(const uint8_t* codes, const int* subset, const float* S, void* out, float* out_scores,
                                                                 uint32_t N, uint32_t n_items, int b, int B, int K) {
    ScanArgs a;                                               // (plain arguments: see scan_short_kernel)
    a.codes = codes; a.subset = subset; a.S = S; a.N = N; a.n_items = n_items; a.m = M; a.b = b; a.K = K;
    a.ws_keys = static_cast<uint64_t*>(out); a.out_ids = out_scores != nullptr ? static_cast<int*>(out) : nullptr;
    a.out_scores = out_scores;
    constexpr int IPV = 16 / M, R = U * IPV;                   // candidates per code vector, per thread
    static_assert(subset_pair_has(M, U), "vectors per thread");
    extern __shared__ __align__(16) unsigned char smem[];
    float2* const lut = reinterpret_cast<float2*>(smem);
    auto& select = *reinterpret_cast<MidSelectLds<NT>(*)[2]>(smem + pair_table_bytes(M, b, 1));
    const int tid = threadIdx.x;
    const int q0 = blockIdx.y * 2, nblk = gridDim.x, blk = blockIdx.x;
    const bool two = q0 + 1 < B;
    const uint32_t n = (uint32_t)a.N;                          // candidates in the list
    const uint32_t first = (uint32_t)blk * NT + (uint32_t)tid, stride = (uint32_t)nblk * NT;

    // ---- the ids (coalesced), then the rows they name
    uint32_t item[R], w[U][4];
#pragma unroll
    for (int s = 0; s < R; ++s) {
        const uint32_t pos = first + (uint32_t)s * stride;
        item[s] = (uint32_t)a.subset[pos < n ? pos : n - 1];  // (past the end: a re-read, never scored)
    }
    auto fetch_rows = [&]() {
#pragma unroll
        for (int s = 0; s < R; ++s) {
            item[s] = item[s] < a.n_items ? item[s] : a.n_items - 1;
            load_row_words<M>(a.codes, item[s], &w[s / IPV][s % IPV * (M / 4)]);
        }
    };
    constexpr bool kTablesFirst = U != 16;
    if constexpr (!kTablesFirst) fetch_rows();
    pair_tables<M, 1, NT, kTablesFirst>(lut, a.S, q0, two, b, tid, fetch_rows);
    mid_select_clear<NT>(select[0], tid);
    mid_select_clear<NT>(select[1], tid);
    __syncthreads();

    // ---- Eq. 5 for every candidate this thread holds
    float sc[2][R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float p0[IPV], p1[IPV];
        pair_scores<M, 1, kLutStride>(lut, b, w[u], p0, p1);
#pragma unroll
        for (int e = 0; e < IPV; ++e) {
            asm volatile("" : "+v"(p0[e]), "+v"(p1[e]));      // (as in scan_pair_kernel: two vectors' lookups under way together)
            const bool have = first + (uint32_t)(u * IPV + e) * stride < n;
            sc[0][u * IPV + e] = have ? p0[e] : empty_score();
            sc[1][u * IPV + e] = have ? p1[e] : empty_score();
        }
        if (u + 2 < U) {
#pragma unroll
            for (int j = 0; j < 4; ++j) asm volatile("" : "+v"(w[u + 2][j]));
        }
    }
    auto emit = [&](int h, int rank, uint64_t key) {
        if (h == 0 || two) emit_key(a, q0 + h, nblk, blk, rank, key);
    };
    select_mid_k_pair<NT>(sc, [&](int slot) -> uint32_t { return item[slot]; }, K, select, tid, emit);
}
