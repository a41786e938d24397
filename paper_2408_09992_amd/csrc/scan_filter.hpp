// Eq. 5 + TopK for batches (filter_prepare_kernel, scan_filter_kernel): a scan of small-integer upper bounds finds the few
// items that can matter, and only those are scored exactly.
// Part of kernels.hpp, which includes these parts inside namespace pqk in this order:
// common.hpp, subitem_scores.hpp, topk_parts.hpp, select_small.hpp, scan_single.hpp, scan_bytes.hpp, scan_short.hpp, scan_pair.hpp, scan_long.hpp, scan_subset.hpp,
// scan_batched.hpp, scan_filter.hpp, fold.hpp, comparison.hpp.
//
// What bounds a batch is the LDS: random 16-byte gathers return 5 lane reads per clock and CU whatever they hold.  With
// fp32 table entries one of them serves four queries; with 8-bit entries it serves sixteen (16-bit: eight), and the four
// sums in a 32-bit word are made by ONE integer addition.  Two lanes that read a row of 32 bytes together, for 32 queries, get 5.9 reads each,
// and a quarter of the rows comes from device memory, through the L1, beside the LDS's: 7.4 together.  So:
//   - a table entry S[k][j] is replaced by a count of steps with base_k + count * step >= S[k][j].  The sum A of an item's
//     counts bounds its score from above: score <= sum(base) + A * step (+ the rounding of the fp32 chain, which `off`
//     below includes).  An item whose A is below T = floor((f - off) / step) scores below f: it is out.
//   - f is a floor of the query's K-th best score.  The first one comes from an exactly scored sample of the catalogue
//     (K of the sample's items reach it); the scan raises it as it finds better items.
//   - one 8-bit sum over a row is coarse: every count is rounded up.  So a sum is over four splits, whose counts are of an M / 4 th of a
//     step then, and sums are averaged, four fields by one v_lerp_u8: the bound is rounded up by two of some hundred steps whatever M
//     is.  Two items pass for every one that should, three or four at m = 16 and 32; at m = 64, and where there are few items per result,
//     16-bit fields are the better ones (one sum).  An exact score reads its table values from device memory, one lane per clock and CU.
//   - what is left is scored exactly, by the same left-to-right fp32 chain as everywhere, and only exact scores enter
//     lists, floors and results.  Bit for bit the same results as the other kernels, whatever the tables are.
// The time does depend on the tables: an item that passes costs as much as a hundred that do not.  Masked entries and, but in lists, queries
// of zeros (a padded batch) cost nothing extra, see filter_prepare_kernel; where most items pass all the same (a large entry
// that hardly any item has, scores that hardly differ in fp32) a query is given up and its share scanned exactly, four queries
// per LDS read.
// A sum starts at 128 - T (16-bit fields: 256 times that), so the top bit of their average says A >= T.  Fields never carry into each
// other: `step` is chosen so that the largest possible sum is at most T_first + 127, T never falls, and T is capped at 128
// (a lower T is always allowed).
// 50M items, m = 8, 32 queries: scan 280 us with one sum of whole steps and 16-bit counts in LDS to sort out what passed, 208 now; 20M, m = 16, 32
// queries, K = 10 and 100: whole calls 258 -> 198 and 470 -> 260; 3M, m = 32, 200 queries: 800 -> 432.
#pragma once

constexpr int kFilterThreads = kBigThreads;
constexpr int kFilterWaves = kFilterThreads / kWave;
constexpr int kFilterBins = 128;                  // histogram of exact scores per query, in units of T
constexpr int kFilterQueue = 3 * kWave / 2;       // a wave's queue of items to score exactly
constexpr int kFilterSpan = 127;                  // steps from the first T to the largest possible sum
// Steps from the first floor to the largest possible sum (a sum's counts and T are rounded), and where the first T of a query's own sample lies:
// the rest up to 128 is what it can rise by, and what lies further below it is looser.  Short rows have the floor near the largest sum.
__host__ __device__ constexpr float filter_room(int m) { return m == 4 ? 80.0f : m == 8 ? 90.0f : 110.0f; }
__host__ __device__ constexpr float filter_t0(int m) { return m == 4 ? 82.0f : m == 8 ? 98.0f : 100.0f; }
constexpr float kFilterUp = 2.5e-4f;              // steps an 8-bit count is rounded up by more than it must be, against the
constexpr float kFilterUp16 = 0.02f;              // rounding of its own computation; 256ths of one a 16-bit count is
constexpr float kFilterDown = 0.02f;              // steps T is rounded down by, likewise
constexpr int kHopeless = 256;
constexpr int kSampleBins = 256;                  // histogram of a sample's scores
constexpr int kSamplePasses = 8;                  // ... and the times its range is narrowed at most
constexpr int kFilterBest = 1280;                 // sample scores a query's parts leave at most

struct FilterQuery {                              // one query's bounds, written by filter_prepare_kernel
    float off, inv;                               // units of a score s: (s - off) * inv
    int t_first;                                  // T of the first part's own floor (+ kHopeless: nearly everything passes that)
    float floor;                                  // a score that K items reach
    __host__ __device__ bool flat() const { return inv == 0.0f && t_first > kFilterSpan; }   // every item scores the same, `off`: the result is the lowest ids
};

struct FilterArgs {
    const uint8_t* codes;
    const float* S;
    long long N;                // items scanned: the catalogue, or the candidate list's length
    int b, K, B;
    int cap;                    // keys of a query's list (a power of two)
    const int* subset;          // candidate list or nullptr
    uint32_t n_items;
    uint64_t* ws_keys;          // [B][nblk][K]
    int* out_ids;               // [B][K]: the result, when one workgroup scans everything for a query; nullptr: lists for the fold
    float* out_scores;
    uint8_t* counts;            // [B][pitch] a query's counts (two-byte sub-ids: of the splits that are looked up in LDS): bytes, or 16-bit words
    uint8_t* far;               // [tile][splits][stride][queries of a tile] counts of the splits looked up in device memory, a row per sub-id
    FilterQuery* query;         // [B]
    uint32_t* hist;             // [B][kFilterBins] exact scores found, by T above the first (cleared by filter_prepare_kernel)
    float* best;                // [B][parts][best_per_part] scores of sample items (parts > 1)
    long long entries;          // of a query's tables: M * 256, or M * b for two-byte sub-ids
    uint16_t* fine;             // [B][entries] 256ths of a step beside the bytes; nullptr: none
    uint32_t pitch;
    int far_splits, tile;       // splits looked up in device memory (the last ones), queries of a workgroup
    int wide;                   // 16-bit counts
    int sample;                 // units of a part's sample per round (code vectors, or items of more than 16 bytes; candidates of a list)
    int rounds;                 // ... and the rounds
    int parts, best_per_part;
    int patient;                // floors shared between workgroups rise so far that the sample gives no query up
    uint64_t* stamps;           // STAMP instances only
};

// Row geometry.  P: bytes of an item's row.  A lane's unit of work is kVecs 16-byte vectors = kItems items.
template <int M, int CW>
struct FilterShape {
    static constexpr int P = M * CW;
    static constexpr int kVecs = P >= 32 ? P / 16 : 1;
    static constexpr int kItems = kVecs * 16 / P;
    static constexpr int kWords = kVecs * 4;
    static constexpr int kSampleUnits = (P == 8 || P == 16 || P == 32) ? 2 : 1;   // ... of a part's sample per thread (vectors or wide items)
    static constexpr int kSampleItems = P >= 16 ? kSampleUnits : kSampleUnits * (16 / P);
    static constexpr int kSampleWords = P >= 16 ? kSampleUnits * P / 4 : kSampleUnits * 4;
};

// 8-bit sums hold the counts of four splits each: in the whole, as many sums of a step's M / 4 th parts as M / 4 are averaged, so that the bound of
// an item is rounded up by two of 118 steps on average whatever M is (one sum over all splits: by M / 2).
// Which sum a split belongs to: splits of neighbouring places go to different sums, forth and back, so that sums stay alike
// where splits differ in their spread.
__host__ __device__ constexpr int filter_sums(int m) { return m / 4; }
__host__ __device__ constexpr int filter_members(int m) { return m / filter_sums(m); }
__host__ __device__ constexpr int filter_member(int m, int sum, int i) { return i * filter_sums(m) + (i & 1 ? filter_sums(m) - 1 - sum : sum); }

// Splits whose tables stay in device memory, so that the L1's way to the lanes works beside the LDS's.  G lanes share an item.  Single lanes: an
// eighth of the splits, a row of 16 bytes per clock and CU beside the LDS's five (lists gather their rows that way, and two-byte sub-ids have more rows
// than the L1 holds: none).  Calls with none and with an eighth (us): m = 8, 1.28M items, 64 queries, K = 10 32.6 and 32.0, 1024, K = 100 296 and 290 (popular sub-ids,
// and Eq. 4 between the calls: 257 and 252 a step, in other runs within 1 %: exact scores come through the L1 too); 600,000, 700
// queries, K = 5 105.5 and 100.5; 600,000, 4096, K = 100 727 and 707; m = 16, 5M, 16, K = 10 48.1 and 45.9; 900,000, 150, K = 3 81.2 and 78.5.  Up to 1.6 % slower where
// much is scored exactly (m = 16, 500,000, 260, K = 4 77.5 and 78.8; m = 8, 200,000, 150, K = 50 32.0 and 32.4); where floors are shared, and for many results at m = 16, see
// filter_near_pays() and filter_near_pays16().
__host__ __device__ constexpr int filter_far_splits(int m, int words, bool w16, int lanes, bool subset = false, int cw = 1) {
    if (w16 || words < 4) return 0;
    if (lanes == 2) return m == 4 ? 0 : m == 8 ? 2 : 3;
    return m == 32 ? 4 : subset || cw == 2 || m == 4 ? 0 : m / 8;
}
// Splits that the tables in LDS have room for: single lanes of short rows keep room for all, which a second scan with exact tables uses.
__host__ __device__ constexpr int filter_table_splits(int m, int words, bool w16, int lanes) {
    return lanes == 1 && m <= 16 ? m : m - filter_far_splits(m, words, w16, lanes);
}

// Byte of a tile's rows in device memory ([splits][stride][queries]) where the part from query `first` on of sub-id `id`'s row begins, in the
// v-th of these splits.  A sub-id beyond the alphabet (two bytes hold more than there are rows) reads its last row: the rows lie in the
// caller's workspace, and no sub-id leads out of them.
__host__ __device__ constexpr uint32_t filter_far_at(uint32_t v, uint32_t id, uint32_t stride, uint32_t queries, uint32_t first) {
    return (v * stride + (id < stride ? id : stride - 1u)) * queries + first;
}

template <int M, int CW>
__device__ __forceinline__ uint32_t filter_sub_id(const uint32_t* w, int item, int k) {
    constexpr int P = M * CW;
    const int byte = item * P + k * CW;
    if constexpr (CW == 2) return (byte & 2) ? (w[byte >> 2] >> 16) : (w[byte >> 2] & 0xFFFFu);
    else return (w[byte >> 2] >> ((byte & 3) * 8)) & 0xFFu;
}

__host__ __device__ inline size_t filter_prepare_lds_bytes(long long entries, int m) {
    const size_t pieces = (size_t)m * (((size_t)entries / m + 4 * kWave - 1) / (4 * kWave));
    return align16((size_t)entries * sizeof(float)) + kSampleBins * sizeof(uint32_t) + align16(sizeof(Ctl)) + ((size_t)m + 1 + 3 * pieces) * sizeof(float);
}

// A cut through the sample's scores by their histogram: `reach` scores (0: there are fewer than asked for) exceed `cut`; the last of
// those asked for is in `bucket`, with `beyond` in higher ones.
struct SampleCut {
    float cut;
    int reach, beyond, bucket;
};
static_assert(kMaxWaves >= 12, "three of them in Ctl::wave_cnt");
__device__ __forceinline__ SampleCut sample_cut(const Ctl* ctl, int slot) {
    const int* c = ctl->wave_cnt + 4 * slot;
    return SampleCut{__int_as_float(c[0]), c[1], c[2], c[3]};
}
// one wave; lo and scale as in bucket_of()
__device__ __forceinline__ void find_sample_cut(const uint32_t* hist, int target, float lo, float scale, Ctl* ctl, int slot, int lane) {
    static_assert(kSampleBins == 4 * kWave, "four buckets per lane, lane 0 with the highest");
    const int base = kSampleBins - 4 * (lane + 1);
    const uint4 v = *reinterpret_cast<const uint4*>(hist + base);
    const uint32_t upto = wave_prefix_sum(v.x + v.y + v.z + v.w);
    const uint64_t has = __ballot(upto >= (uint32_t)target);
    const float ninf = -__builtin_inff();
    if (has != 0 ? lane == __builtin_ctzll(has) : lane == 0) {
        SampleCut c = {ninf, 0, 0, 0};
        if (has != 0) {
            uint32_t above = upto - (v.x + v.y + v.z + v.w);
            int i = 3;
            if (above + v.w < (uint32_t)target) { above += v.w; i = 2; }
            if (i == 2 && above + v.z < (uint32_t)target) { above += v.z; i = 1; }
            if (i == 1 && above + v.y < (uint32_t)target) { above += v.y; i = 0; }
            c.bucket = base + i;
            c.beyond = (int)above;
            c.reach = (int)(above + (i == 3 ? v.w : i == 2 ? v.z : i == 1 ? v.y : v.x));
            // a score of a lower bucket than that: every score of it or a higher one exceeds it
            c.cut = next_down(lo);                            // (all reach the lowest score)
            if (c.bucket > 0 && scale > 0.0f) {
                const float width = 1.0f / scale;
                float cut = lo + ((float)c.bucket - 0.5f) * width;
#pragma unroll 1
                for (int guard = 0; guard < 64 && bucket_of<kSampleBins>(cut, lo, scale) >= c.bucket; ++guard) cut -= width;
                if (bucket_of<kSampleBins>(cut, lo, scale) < c.bucket) c.cut = fmaxf(cut, c.cut);
            }
        }
        int* out = ctl->wave_cnt + 4 * slot;
        out[0] = __float_as_int(c.cut); out[1] = c.reach; out[2] = c.beyond; out[3] = c.bucket;
    }
}

// The sample.  grid = (parts, B).  Every part scores a sample of its own exactly, in rounds of kSampleItems per thread, and,
// when there are several, leaves its best scores; part 0 also sets the query's step and bases by the floor of its own sample
// and writes the table of counts.  (The scan takes the K-th best of all parts' scores as the first floor: at least as high
// as part 0's, so the fields' range holds.)  The more items the sample has, the fewer pass the floor it gives; a batch of
// few queries would leave most CUs idle with one part each (16 queries x 16 parts x 4096 items cost no more time than
// 16 x 4096), and a round more costs less than a part more, which loads the tables again.
// What it costs is latency: the tables' way from memory, then kSampleItems x M lookups per thread and round (4096 items at
// m = 8: 1.6 us), a histogram of the threads' best, the counts.
//   M, CW: splits, bytes per sub-id; SUB: the sample is taken from a candidate list
// Two workgroups per CU where the tables leave room (16 of 32 waves each: at most 64 vector and 80 scalar registers; with 88 scalar
// ones a CU held one workgroup, and 1024 queries at m = 8 took 31 us instead of 21).
// NT: threads.  512 where the queries alone are several workgroups per CU: four at a time then, and one's barriers pass in the others' work
// (1000 queries of 300,000 items at m = 8, K = 10: 95 -> 90 us a step).
template <int M, int CW, bool SUB, int NT>
__global__ __launch_bounds__(NT, M <= 16 ? 8 : 4) void filter_prepare_kernel(FilterArgs a) {
    using Sh = FilterShape<M, CW>;
    constexpr int NW = NT / kWave, P = Sh::P;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int q = blockIdx.y, part = blockIdx.x, b = a.b, K = a.K;
    const int stride = CW == 1 ? kLutStride : b;
    float* lut = reinterpret_cast<float*>(smem);
    uint32_t* hist = reinterpret_cast<uint32_t*>(smem + align16((size_t)a.entries * sizeof(float)));
    Ctl* ctl = reinterpret_cast<Ctl*>(hist + kSampleBins);
    float* bases = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(ctl) + align16(sizeof(Ctl)));   // [M]
    int* n_found = reinterpret_cast<int*>(bases + M);
    float* piece = reinterpret_cast<float*>(n_found + 1);     // [pieces of the tables][3]: max, min, sum
    const float* Sq = a.S + (size_t)q * M * b;

    // ---- the sample's rows: runs of units spread evenly over the catalogue (or the list), the parts' and rounds' interleaved.  (Runs of one, a line of memory
    // for every lane: 1024 queries, m = 8, four rounds, 25.7 us, of four 19.0; 32 queries, eight parts of three rounds 13.0 and 10.1; 64, four parts 7.9 and 6.4.)
    constexpr bool kByItem = SUB || P > 16;
    constexpr int kLoads = SUB ? Sh::kSampleItems : Sh::kSampleUnits;
    constexpr uint32_t kRun = SUB || P > 32 ? 1u : P == 32 ? 2u : 4u;   // units that follow each other in memory, 64 bytes: a line's neighbours come with it
    const uint32_t total = (uint32_t)(kByItem ? a.N : (a.N * P) / 16);
    const uint32_t n_sample = (uint32_t)a.sample < total ? (uint32_t)a.sample : total, every = total / n_sample;
    auto fetch = [&](int round, uint32_t (&w)[Sh::kSampleWords]) {
        const uint32_t slices = (uint32_t)(a.parts * a.rounds);
        const uint32_t shift = every * (uint32_t)(part * a.rounds + round) / slices;   // (every <= 2^21, or 1; slices <= 128)
#pragma unroll
        for (int u = 0; u < kLoads; ++u) {
            uint32_t i = (uint32_t)(u * NT + tid);
            i = i < n_sample ? i : n_sample - 1;
            i = (i & ~(kRun - 1u)) * every + shift * kRun + (i & (kRun - 1u));   // (within the units: shift < every, or 0 where every is 1)
            if constexpr (SUB) {
                uint32_t item = (uint32_t)a.subset[i];
                item = item < a.n_items ? item : a.n_items - 1;
                load_row_words<P>(a.codes, item, &w[u * P / 4]);
            } else if constexpr (P > 16) {
                load_row_words<P>(a.codes, i, &w[u * P / 4]);
            } else {
                const uint4 x = reinterpret_cast<const uint4*>(a.codes)[i];
                w[4 * u] = x.x; w[4 * u + 1] = x.y; w[4 * u + 2] = x.z; w[4 * u + 3] = x.w;
            }
        }
    };
    uint32_t w[Sh::kSampleWords];

    // ---- the query's tables to LDS, in pieces of 256 entries, their extremes on the way
    const int pieces = (stride + 4 * kWave - 1) / (4 * kWave);   // per split (one-byte sub-ids: one)
    auto load_piece = [&](int p, float (&v)[4]) {
        const int k = CW == 1 ? p : p / pieces, j0 = CW == 1 ? 0 : (p % pieces) * 4 * kWave;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = j0 + i * kWave + lane;
            v[i] = (p < M * pieces && j < b) ? Sq[(size_t)k * b + j] : 0.0f;
        }
    };
    auto keep_piece = [&](int p, const float (&v)[4]) {
        if (p >= M * pieces) return;
        const int k = CW == 1 ? p : p / pieces, j0 = CW == 1 ? 0 : (p % pieces) * 4 * kWave;
        float mx = -__builtin_inff(), mn = __builtin_inff(), sum = 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int j = j0 + i * kWave + lane;
            if (j < stride) lut[(size_t)k * stride + j] = v[i];
            if (j < b) { mx = fmaxf(mx, v[i]); mn = fminf(mn, v[i]); sum += v[i]; }
        }
        wave_minmax(mn, mx);
        sum = wave_sum_f32(sum);
        if (lane == 0) { piece[3 * p] = mx; piece[3 * p + 1] = mn; piece[3 * p + 2] = sum; }
    };
    constexpr int kAhead = CW == 1 ? (M + NW - 1) / NW : 4;   // pieces of a wave on their way together
    float v[kAhead][4];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) load_piece(wave + i * NW, v[i]);
    // (the sample's rows after the first pieces: loads return in order, and what is made of the pieces passes while the rows, which come from
    // further away, are on their way)
    fetch(0, w);                                              // (rounds >= 1)
    for (int i = tid; i < kSampleBins; i += NT) hist[i] = 0;
    if (tid == 0) *n_found = 0;
    if (part == 0 && tid < kFilterBins) a.hist[(size_t)q * kFilterBins + tid] = 0u;
    __builtin_amdgcn_sched_barrier(0);
    for (int p0 = wave; p0 < M * pieces;) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i) keep_piece(p0 + i * NW, v[i]);
        p0 += kAhead * NW;
        if (CW == 1 || p0 >= M * pieces) break;
#pragma unroll
        for (int i = 0; i < kAhead; ++i) load_piece(p0 + i * NW, v[i]);
    }
    __syncthreads();

    // ---- all rounds, scored: a thread keeps its best score (of its even and its odd items, when K is large).  At least K of
    // these exceed the cut, and hardly more of all scores do: they are a histogram's 1024 counts instead of thousands that
    // would have to be collected (64 queries, K = 120: 28 us, collecting and ranking, -> 10)
    constexpr int kPerLoad = Sh::kSampleItems / kLoads;
    auto have = [&](int e) { return (uint32_t)((e / kPerLoad) * NT + tid) < n_sample; };
    const float ninf = -__builtin_inff();
    float best[2] = {ninf, ninf};
    for (int round = 0; round < a.rounds; ++round) {
        float acc[Sh::kSampleItems];
#pragma unroll
        for (int e = 0; e < Sh::kSampleItems; ++e) {
#pragma unroll
            for (int k = 0; k < M; ++k) {
                const float v = lut[(size_t)k * stride + filter_sub_id<M, CW>(w, e, k)];
                acc[e] = k == 0 ? v : acc[e] + v;
            }
        }
        if (round + 1 < a.rounds) fetch(round + 1, w);
#pragma unroll
        for (int e = 0; e < Sh::kSampleItems; ++e) {
            asm volatile("" : "+v"(acc[e]));                  // (the lookups of all items under way together, whichever count)
            best[e & 1] = fmaxf(best[e & 1], have(e) ? acc[e] : ninf);
        }
    }
    const bool both = K > NT / 4 && Sh::kSampleItems > 1;
    if (!both) { best[0] = fmaxf(best[0], best[1]); best[1] = ninf; }
    // Cuts, from one histogram: several parts leave their best scores, those above the cut that so many exceed; part 0 goes on with
    // the cut that K exceed.  (Two waves look for them at the same time.)
    const int r = a.best_per_part;
    const bool several = a.parts > 1;
    float lo, scale;
    set_range<NW>(fminf(best[0] > ninf ? best[0] : -ninf, best[1] > ninf ? best[1] : -ninf), fmaxf(best[0], best[1]), ctl, tid, lo, scale);
    scale *= (float)kSampleBins / (float)kBins;
#pragma unroll
    for (int h = 0; h < 2; ++h)
        if (best[h] > ninf) atomicAdd(&hist[bucket_of<kSampleBins>(best[h], lo, scale)], 1u);
    // (meanwhile: the splits' extremes, lane k with split k, every wave for itself)
    const bool mine = lane < M;
    float s_mx = -__builtin_inff(), s_mn = __builtin_inff(), s_mean = 0.0f;
    for (int p = 0; p < pieces && mine; ++p) {
        const float* x = piece + 3 * (lane * pieces + p);
        s_mx = fmaxf(s_mx, x[0]); s_mn = fminf(s_mn, x[1]); s_mean += x[2];
    }
    if (!mine) s_mx = s_mn = 0.0f;
    s_mean = s_mean / (float)b;
    const float sum_max = wave_sum_f32(s_mx);
    const bool flat = __ballot(mine && s_mx != s_mn) == 0;    // every item has the same score (a query of zeros, as batches are padded with)
    __syncthreads();
    if (wave < 2) find_sample_cut(hist, wave == 0 ? K : r - r / 8, lo, scale, ctl, wave, lane);
    __syncthreads();
    // A score far from the others (an item with a masked sub-id, at -1e9) stretches the range until the buckets tell nothing apart:
    // while the one sought shares its bucket with many that are no better, that bucket alone is taken apart again.
    auto narrowed = [&](SampleCut c, int target) -> float {
        bool in0 = best[0] > ninf, in1 = best[1] > ninf;
        float from = lo, per = scale;
        int left = target;                                    // the left-th best of what is `in` is sought
#pragma unroll 1
        for (int pass = 0; pass < kSamplePasses && c.reach - left > target / 2 + kWave && per > 0.0f; ++pass) {
            left -= c.beyond;
            in0 = in0 && bucket_of<kSampleBins>(best[0], from, per) == c.bucket;
            in1 = in1 && bucket_of<kSampleBins>(best[1], from, per) == c.bucket;
            for (int i = tid; i < kSampleBins; i += NT) hist[i] = 0;   // (added to behind set_range()'s barrier)
            set_range<NW>(fminf(in0 ? best[0] : -ninf, in1 ? best[1] : -ninf), fmaxf(in0 ? best[0] : ninf, in1 ? best[1] : ninf), ctl, tid, from, per);
            per *= (float)kSampleBins / (float)kBins;
            if (in0) atomicAdd(&hist[bucket_of<kSampleBins>(best[0], from, per)], 1u);
            if (in1) atomicAdd(&hist[bucket_of<kSampleBins>(best[1], from, per)], 1u);
            __syncthreads();
            if (wave == 0) find_sample_cut(hist, left, from, per, ctl, 2, lane);
            __syncthreads();
            c = sample_cut(ctl, 2);
        }
        return c.cut;
    };
    const SampleCut first = sample_cut(ctl, 0), own = sample_cut(ctl, 1);
    float* const part_best = a.best + ((size_t)q * a.parts + part) * r;
    auto fill_best = [&]() { for (int t = *n_found + tid; t < r; t += NT) part_best[t] = ninf; };
    float cut = several ? own.cut : first.cut;
#pragma unroll 1
    for (int which = several ? 1 : 0;; --which) {
        const SampleCut c = which == 0 ? first : own;
        const int target = which == 0 ? K : r - r / 8;
        cut = c.cut;
        if (__builtin_expect(c.reach - target > target / 2 + kWave, 0)) cut = narrowed(c, target);
        if (which == 0) break;
        // this part's best scores, in any order (more than there is room for: as many as there is); fewer are filled up with -inf
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (best[h] > cut) {
                const int pos = atomicAdd(n_found, 1);
                if (pos < r) part_best[pos] = best[h];
            }
        }
        if (part != 0) {                                      // (the same for the whole workgroup)
            __syncthreads();
            fill_best();
            return;
        }
    }

    // ---- step and bases (lane k holds split k; from the clamping on the first wave alone: sixteen that all do the same share four SIMDs, and a
    // chain of dependent instructions takes each of them twice as long)
    // An item with an entry further than sum_max - cut below its split's largest scores below the cut whatever its others are: all
    // such entries count as that depth (more than they are: the bounds hold), and for the split's mean as three times as far from the
    // largest as its other entries (or the splits' on average) are.  Left as they are, one masked sub-id (-1e9) would
    // set step, bases and slack for all: 1.28M items, 64 queries with one masked sub-id each: 604 us (37 without it), now 36.
    // Only where a split's entries lie further from its largest than that, or twice as far as the splits' do on average: at m = 4 the
    // lowest entries of ordinary tables are that deep, and a second pass over the tables is 0.5 us.
    const float depth = sum_max - cut, deepest = s_mx - depth;
    float spread = wave_sum_f32(s_mx - s_mean);
    const bool clamped = __ballot(mine && s_mn < deepest && s_mx - s_mean > fminf(depth, spread * (2.0f / M))) != 0;   // (the same in every wave)
    if (__builtin_expect(clamped, 0)) {
        __syncthreads();
        for (int p = wave; p < M * pieces; p += NW) {
            const int k = CW == 1 ? p : p / pieces, j0 = CW == 1 ? 0 : (p % pieces) * 4 * kWave;
            const float least = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(deepest), __builtin_amdgcn_readfirstlane(k)));
            float sum = 0.0f, n = 0.0f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int j = j0 + i * kWave + lane;
                const float x = j < b ? lut[(size_t)k * stride + j] : -__builtin_inff();
                if (x >= least && j < b) { sum += x; n += 1.0f; }
            }
            sum = wave_sum_f32(sum);
            n = wave_sum_f32(n);
            if (lane == 0) { piece[3 * p + 1] = n; piece[3 * p + 2] = sum; }
        }
        __syncthreads();
        float sum = 0.0f, n = 0.0f;                           // the entries that count as they are: the largest at least
        for (int p = 0; p < pieces && mine; ++p) {
            n += piece[3 * (lane * pieces + p) + 1];
            sum += piece[3 * (lane * pieces + p) + 2];
        }
        const float near = mine ? s_mx - sum / n : 0.0f;
        // (... and further where most of a split's entries count so, by what keeps their items from passing in their numbers)
        const float most = (mine && (float)b > 2.0f * n) ? logf(((float)b - n) / n) : 0.0f;
        const float far = fmaxf(near, wave_sum_f32(near) * (1.0f / M)) * (3.0f + 0.18f * sqrtf((float)M) * most);
        if (mine) {
            s_mean = (sum + ((float)b - n) * (s_mx - fminf(far, depth))) / (float)b;
            s_mn = fmaxf(s_mn, deepest);
        }
        spread = wave_sum_f32(s_mx - s_mean);
    }
    constexpr int NA = filter_sums(M);
    if (__builtin_amdgcn_readfirstlane(wave) == 0) {
        const float sum_min = wave_sum_f32(s_mn), sum_abs = wave_sum_f32(fmaxf(fabsf(s_mx), fabsf(s_mn)));
        // what fp32 chains of M additions (scores, sums of bases) can be off by
        const float slack = 4.0f * (float)(M + 1) * 5.9604645e-8f * sum_abs;
        const float floor_s = clamped ? cut : fmaxf(cut, sum_min - slack);   // (at least K of the part's items exceed the cut)
        const float range = sum_max - floor_s + 2.0f * slack;
        // bases: the further a split's maximum lies above its mean, the more of the range it gets; what lies below the base
        // counts as the base (loose only for items that will rarely be near a floor)
        float step, inv, base, off, t_floor;
        auto place = [&](float room) {
            step = range / room;
            inv = 1.0f / step;
            if (!(step > 0.0f) || !(inv < 1.0e30f) || !(step < 1.0e30f)) { inv = 0.0f; step = 0.0f; }   // degenerate: T stays 0, every item is scored
            const float lambda = spread > 0.0f ? (sum_max - floor_s + filter_t0(M) * step) / spread : 0.0f;
            base = mine ? fmaxf(s_mn, s_mx - lambda * (s_mx - s_mean)) : 0.0f;
            off = wave_sum_f32(base) + slack;
        };
        auto first_t = [&]() {
            const float t = inv > 0.0f ? floorf((floor_s - off) * inv - kFilterDown) : 0.0f;
            t_floor = fminf(fmaxf(t, 0.0f), (float)(kFilterSpan + 1));
        };
        if (M >= 16 && a.wide) {
            place((float)(kFilterSpan - 3));
            first_t();
        } else {
            // A sum starts at 128 - T and must not run over: its four largest counts together are at most 127 + T.  The sum whose
            // splits spread most decides; the counts are nearly linear in the range's and T's steps.
            auto largest_sum = [&]() -> float {
                const float own = mine ? s_mx - base : 0.0f;
                float sum = 0.0f, least = 0.0f;
#pragma unroll
                for (int i = 0; i < filter_members(M); ++i) sum += __shfl(own, filter_member(M, lane & (NA - 1), i));
                wave_minmax(least, sum);
                return sum * inv * (float)NA + (float)filter_members(M) * (1.0f + 4.0f * kFilterUp);   // (counts rounded up)
            };
            float room = filter_room(M);
            place(room);
            first_t();
            float counts = largest_sum();
#pragma unroll 1
            for (int pass = 0; pass < 3 && counts > (float)kFilterSpan + t_floor; ++pass) {
                const float per = (counts - (float)filter_members(M)) / (room + filter_t0(M));
                room = fmaxf(((float)kFilterSpan - 5.0f + t_floor) / per - filter_t0(M), 8.0f);
                place(room);
                first_t();
                counts = largest_sum();
            }
            if (counts > (float)kFilterSpan + t_floor) {          // (splits that differ widely: these bases, a step with which a sum fits whatever T is)
                step *= counts / (float)(kFilterSpan - 5);
                inv = 1.0f / step;
                if (!(step < 1.0e30f)) { inv = 0.0f; step = 0.0f; }
                first_t();
            }
        }
        if (mine) bases[lane] = base;
        if (lane == 0) ctl->scale = inv;                      // (for all waves; the sample's ranges are done with)
        // How much of the sample would pass: scores within the roundings of their counts below the floor.  Where that is more than three
        // in ten, by the best of n scores of 64 threads, the scan gives the query up unless the parts together know better.
        // (Floors that few workgroups share over long shares rise by themselves, and how far nobody knows yet.)
        const float near = floor_s - step * (a.wide ? 0.5f : 2.5f);
        const int n = a.rounds * Sh::kSampleItems, pass = __popcll(__ballot(fmaxf(best[0], best[1]) >= near));
        const bool hopeless = !(inv > 0.0f) || (a.patient == 0 && (float)pass > (float)kWave * (1.0f - exp2f((float)n * -0.5146f)));   // 0.7 ^ n
        if (lane == 0) {
            const int t = (int)t_floor;
            a.query[q] = FilterQuery{off, inv, hopeless ? t + kHopeless : t, cut};
            if (__builtin_expect(flat && !SUB, 0)) {          // (no bound is reached, and the scan knows the result)
                float score = lut[0];
                for (int k = 1; k < M; ++k) score += lut[(size_t)k * stride];
                a.query[q] = FilterQuery{score, 0.0f, kFilterSpan + 1, cut};
            }
        }
    }
    __syncthreads();

    if (several) fill_best();
    const float inv = ctl->scale;
    const bool nothing = flat && !SUB;                        // (a flat query: nothing passes)
    uint32_t* const out = reinterpret_cast<uint32_t*>(a.counts + (size_t)q * a.pitch);
    if (M >= 16 && a.wide) {
        // ---- 16-bit counts, 256ths of a step, two entries per thread and store
        const float inv256 = nothing ? 0.0f : inv * 256.0f, up = nothing ? 0.0f : kFilterUp16;
        for (long long i = tid; i * 2 < a.entries; i += NT) { // (entries is a multiple of 16)
            uint32_t word = 0;
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint32_t e = (uint32_t)(i * 2 + c), k = e / (uint32_t)stride;
                const float x = ceilf((lut[e] - bases[k]) * inv256 + up);
                word |= (uint32_t)fminf(fmaxf(x, 0.0f), 65535.0f) << (c * 16);
            }
            out[i] = word;
        }
        return;
    }
    // ---- 8-bit counts, M / 4 ths of a step: four entries per thread and store (a pitch is a multiple of 16); two-byte sub-ids: of splits that
    // are looked up in device memory a byte of the tile's rows each.  (A tile's workgroups write bytes of the same lines, each its own.)
    const float per = nothing ? 0.0f : inv * (float)NA, up = nothing ? 0.0f : kFilterUp;
    auto count_of = [&](uint32_t e) -> uint32_t {
        const float x = ceilf((lut[e] - bases[e / (uint32_t)stride]) * per + up);
        return (uint32_t)fminf(fmaxf(x, 0.0f), 255.0f);
    };
    if constexpr (CW == 1 && (SUB ? M == 8 : M == 16)) {
        if (a.fine != nullptr) {                              // (and 16-bit counts beside them, from the same read of the table)
            uint2* const fine = reinterpret_cast<uint2*>(a.fine + (size_t)q * a.entries);
            const float inv256 = nothing ? 0.0f : inv * 256.0f, up16 = nothing ? 0.0f : kFilterUp16;
            for (uint32_t i = tid; i * 4 < (uint32_t)a.entries; i += NT) {
                const float4 x = reinterpret_cast<const float4*>(lut)[i];
                const float base_k = bases[i * 4 / kLutStride], v[4] = {x.x, x.y, x.z, x.w};
                uint32_t word = 0, words[2] = {0, 0};
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float over = v[c] - base_k;
                    word |= (uint32_t)fminf(fmaxf(ceilf(over * per + up), 0.0f), 255.0f) << (8 * c);
                    words[c / 2] |= (uint32_t)fminf(fmaxf(ceilf(over * inv256 + up16), 0.0f), 65535.0f) << (16 * (c & 1));
                }
                out[i] = word;
                fine[i] = make_uint2(words[0], words[1]);
            }
            return;                                           // (all splits are looked up in LDS)
        }
    }
    const uint32_t there = CW == 1 ? 0u : (uint32_t)a.far_splits * (uint32_t)stride, here = (uint32_t)(M * stride) - there;
    for (uint32_t i = tid; i * 4 < here; i += NT) {
        uint32_t word = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) word |= (i * 4 + c < here ? count_of(i * 4 + c) : 0u) << (8 * c);
        out[i] = word;
    }
    if constexpr (CW == 1) return;
    uint8_t* const row = a.far + (size_t)(q / a.tile) * there * a.tile + q % a.tile;
    const int pad = q == a.B - 1 ? a.tile - 1 - q % a.tile : 0;   // (queries that do not exist count nothing)
    for (uint32_t i = tid; i < there; i += NT) {
        uint8_t* const at = row + (size_t)i * a.tile;
        at[0] = (uint8_t)count_of(here + i);
        for (int c = 1; c <= pad; ++c) at[c] = 0;
    }
}

__host__ __device__ constexpr size_t filter_state_bytes(int queries) {   // everything but the tables, the lists and the queues
    return (size_t)queries * (kFilterBins * sizeof(uint32_t) + sizeof(uint64_t) + 3 * sizeof(uint32_t) + sizeof(FilterQuery)) + 64;
}
// `lanes`: that share an item; `stride`: table entries of a split
__host__ __device__ constexpr size_t filter_table_bytes(int m, long long stride, int words, bool w16, int lanes) {
    return (size_t)filter_table_splits(m, words, w16, lanes) * stride * words * 4 * lanes;
}
// `fine`: 16-bit counts beside the bytes
__host__ __device__ constexpr size_t filter_lds_bytes(int m, long long stride, int words, bool w16, int lanes, int cap, bool fine = false) {
    const int queries = words * (w16 ? 2 : 4) * lanes;
    return align16(filter_table_bytes(m, stride, words, w16, lanes)) + (fine ? (size_t)m * stride * queries * sizeof(uint16_t) : 0) + (size_t)queries * cap * sizeof(uint64_t) +
           (size_t)kFilterWaves * kFilterQueue * sizeof(uint64_t) + align16(filter_state_bytes(queries));
}

template <int W> struct FilterWord;
template <> struct FilterWord<1> { typedef uint32_t type; };
template <> struct FilterWord<2> { typedef uint2 type; };
template <> struct FilterWord<4> { typedef uint4 type; };

// The scan.  grid = (item blocks, tiles of QT queries).  M, CW, SUB as above; W: 32-bit words of a lane's table entry (1, 2, 4);
// W16: 16-bit fields.  G lanes (1 or 2) share an item, each with W * 4 (or 2) of the QT queries.
// Dynamic LDS: tables (two-byte sub-ids) | lists [QT][cap] | queues [waves][kFilterQueue] | hist [QT][kFilterBins] | thr | state words.
// SHARE: the workgroups of a query share their floors (a choice at run time would make the loop wait for all of a wave's loads).
// STAMP: measurement instance that also records wall-clock stamps per wave.
// FINE: 16-bit counts in LDS beside the bytes (one-byte sub-ids): what the bytes let pass is looked up there, nine 2-byte lanes per clock,
// before it is scored exactly, one lane per clock: of three or four that pass at m = 16, one is left.  Half the queries per LDS read pay
// for it there, see filter_fine_pays() (120,000 items, 400 queries, K = 60: a call 84 -> 74 us); lists of m = 8 have room for sixteen.
// NEAR: all splits in LDS where others keep some in device memory.
template <int M, int CW, int W, bool W16, bool SUB, int G, bool SHARE, bool STAMP = false, bool FINE = false, bool NEAR = false>
__global__ __launch_bounds__(kFilterThreads) void scan_filter_kernel(FilterArgs a) {
    using Sh = FilterShape<M, CW>;
    using Word = typename FilterWord<W>::type;
    constexpr int NT = kFilterThreads, NW = kFilterWaves, P = Sh::P, NI = Sh::kItems;
    constexpr int F = W16 ? 2 : 4, QL = W * F, QT = QL * G;   // fields per word, queries per lane and per tile
    constexpr int PER = kWave / G;                            // items a wave looks up side by side
    constexpr int V = NEAR ? 0 : filter_far_splits(M, W, W16, G, SUB, CW);   // splits looked up in device memory, the last ones
    constexpr int T = filter_table_splits(M, W, W16, G);      // ... that the tables in LDS have room for
    static_assert(T >= M - V, "room for the splits looked up in LDS");
    constexpr int NA = W16 ? 1 : filter_sums(M);              // sums of a field
    constexpr int QW = (QT + NW - 1) / NW;                    // queries that a wave looks after
    constexpr int EW = T * G >= M ? W : W / 2;          // queries of a second scan: exact tables in the counts' place
    // Reads of device memory are under way a unit ahead: pairs of lanes, and single ones whose units are an item each.  (Two items, m = 8: a unit more that a
    // wave holds costs more at the end; 64 queries 32.3 us with, 31.9 without; 1024, K = 100 293 and 290; m = 16, 16 queries of 5M 45.7 and 46.0.)
    constexpr bool AHEAD = V > 0 && Sh::kWords == 4 && NI * V * W <= 16 && (G == 2 || NI == 1);
    constexpr int D = G == 2 ? 4 : AHEAD ? 3 : 2;             // units whose codes a wave holds or has asked for
    constexpr int XS = AHEAD ? (D & 1 ? D : 2) : 1;           // units whose rows of device memory it does
    constexpr uint32_t TOP = W16 ? 0x80008000u : 0x80808080u;
    static_assert(W16 ? (M >= 16 && G == 1) : (G == 1 || (G == 2 && W == 4 && QT == 32)), "16-bit fields, or pairs of lanes");
    static_assert(!FINE || (!W16 && G == 1 && CW == 1 && V == 0), "fine counts: beside bytes");
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int half = G == 1 ? 0 : lane & 1;                   // this lane's part of a row
    const int nblk = gridDim.x, tile = blockIdx.y, blk = blockIdx.x, q0 = tile * QT, K = a.K, b = a.b, cap = a.cap;
    uint64_t* const rec = STAMP ? a.stamps + (((size_t)tile * nblk + blk) * NW + wave) * kStampSlots : nullptr;
    stamp<STAMP>(rec, kStampEntry, lane);
    const int nq = a.B - q0 < QT ? a.B - q0 : QT;
    const int stride = CW == 1 ? kLutStride : b;
    __shared__ __align__(16) uint32_t tab_static[CW == 1 ? T * kLutStride * W * G : 4];
    uint32_t* const tab = CW == 1 ? tab_static : reinterpret_cast<uint32_t*>(smem);
    const uint32_t here = (uint32_t)((M - V) * stride);       // entries of a query in LDS
    uint16_t* const fine = reinterpret_cast<uint16_t*>(smem);                     // FINE: [QT][M * 256]
    uint64_t* const lists = reinterpret_cast<uint64_t*>(smem + (CW == 1 ? (FINE ? (size_t)QT * M * kLutStride * sizeof(uint16_t) : 0) : align16((size_t)here * W * G * 4)));
    uint64_t* const queue = lists + (size_t)QT * cap + (size_t)wave * kFilterQueue;
    uint32_t* const hist = reinterpret_cast<uint32_t*>(lists + (size_t)QT * cap + (size_t)NW * kFilterQueue);
    uint64_t* const thr = reinterpret_cast<uint64_t*>(hist + QT * kFilterBins);   // a pruned list's K-th best key
    uint32_t* const cnt = reinterpret_cast<uint32_t*>(thr + QT);                  // keys in the list (or asked for)
    uint32_t* const lock = cnt + QT;
    FilterQuery* const par = reinterpret_cast<FilterQuery*>(lock + QT);
    uint32_t* const start = reinterpret_cast<uint32_t*>(par + QT);                // [G][W] the fields' start values: 128 - T, or 256 times that
    uint32_t* const next_unit = start + 8;
    uint32_t* const given_up = next_unit + 1;                                     // queries the bounds are no use for, as bits of a mask of hits
    uint32_t* const passed = given_up + 1;                                        // [QT] items whose bounds reached the floor; top bit: given up

    // a query's bit in a mask of hits: field f of word j is bit f * 8 (or 16) + j; the second lane's words follow the first's
    auto bit_of = [](int q) -> int { return W16 ? (q & 1) * 16 + (q >> 1) : (q & 3) * 8 + (q >> 2); };
    auto query_of = [](int bit) -> int { return W16 ? (bit & 15) * 2 + (bit >> 4) : (bit & 7) * 4 + (bit >> 3); };

    // ---- units of work: a wave's share (PER x kVecs vectors), the workgroups' interleaved one by one (whole rounds of a
    // workgroup's waves left some with a twentieth more than others: 5M items at m = 16, 256 workgroups)
    const uint32_t total = (uint32_t)((P <= 16 && !SUB) ? (a.N * P) / 16 : a.N);  // whole vectors, or items / candidates
    constexpr uint32_t kPerLane = (P <= 16 && !SUB) ? Sh::kVecs : NI;             // ... per lane and unit
    // (`beside`: items side by side, PER as long as G lanes share one, or a whole wave's)
    constexpr std::integral_constant<int, PER> kShared = {};
    constexpr std::integral_constant<int, kWave> kOwn = {};
    auto share_of = [&](auto beside) -> uint32_t {            // this workgroup's units
        constexpr uint32_t kPerUnit = decltype(beside)::value * kPerLane;
        const uint32_t all = (total + kPerUnit - 1) / kPerUnit;
        return (uint32_t)blk < all ? (all - blk + nblk - 1) / nblk : 0;
    };
    const uint32_t units = share_of(kShared);
    const uint32_t last = total - 1;
    auto first_of = [&](auto beside, uint32_t u) -> uint32_t {   // the lane's first element of unit u; the others follow at `beside`
        return (u * (uint32_t)nblk + (uint32_t)blk) * (decltype(beside)::value * kPerLane) + (uint32_t)(decltype(beside)::value == kWave ? lane : lane / G);
    };
    auto fetch_ids = [&](auto beside, uint32_t u, uint32_t (&id)[NI]) {   // candidate lists: the items' ids
        if constexpr (SUB) {
            const uint32_t p0 = first_of(beside, u);
#pragma unroll
            for (int e = 0; e < NI; ++e) {
                const uint32_t p = p0 + e * decltype(beside)::value;
                const uint32_t item = (uint32_t)a.subset[p < last ? p : last];
                id[e] = item < a.n_items ? item : a.n_items - 1;
            }
        }
    };
    auto fetch = [&](auto beside, uint32_t u, const uint32_t (&id)[NI], uint32_t (&w)[Sh::kWords]) {   // branch-free: clamped past the end
        const uint32_t p0 = first_of(beside, u);
        if constexpr (SUB) {
#pragma unroll
            for (int e = 0; e < NI; ++e) load_row_words<P>(a.codes, id[e], &w[e * P / 4]);
        } else {
            constexpr int kEach = P > 16 ? P / 16 : 1;        // vectors that follow each other
#pragma unroll
            for (int v = 0; v < Sh::kVecs / kEach; ++v) {
                const uint32_t p = p0 + v * decltype(beside)::value;
                const uint4* const at = reinterpret_cast<const uint4*>(a.codes) + (size_t)(p < last ? p : last) * kEach;
#pragma unroll
                for (int i = 0; i < kEach; ++i) {
                    const uint4 x = at[i];
                    uint32_t* const o = &w[4 * (v * kEach + i)];
                    o[0] = x.x; o[1] = x.y; o[2] = x.z; o[3] = x.w;
                }
            }
        }
    };
    // element e of unit u: the item (or its place in the list), or -1u past the end
    auto element_of = [&](auto beside, uint32_t u, int e) -> uint32_t {
        const uint32_t p0 = first_of(beside, u);
        if constexpr (SUB || P > 16) {
            const uint32_t p = p0 + e * decltype(beside)::value;
            return p <= last ? p : ~0u;
        } else {
            constexpr int IPV = 16 / P;
            const uint32_t p = p0 + (e / IPV) * decltype(beside)::value;
            return p <= last ? p * IPV + e % IPV : ~0u;
        }
    };
    auto item_at = [&](uint32_t element) -> uint32_t {
        if constexpr (SUB) {
            const uint32_t item = (uint32_t)a.subset[element];
            return item < a.n_items ? item : a.n_items - 1;
        } else {
            return element;
        }
    };

    // ---- the tile's counts on their way, then the first units' codes (loads return in order, and codes may come from
    // far away: asked for first, they held the tables up by 5 us on an 80 MB catalogue), then the tables: rows of counts,
    // one per query, become entries of QL fields per lane (transposed in registers, N entries of one lane's queries at a time).  One-byte
    // sub-ids: those of the splits looked up in device memory too, which every workgroup of the tile writes, the same bytes at the same place, and
    // reads behind its own barrier (made by the sample's kernels, a byte of a row from each of a tile's queries, they cost 1024 queries 20 us)
    constexpr int N_ = W16 ? 2 : 4;                           // counts of a 32-bit word
    const uint32_t stored = CW == 1 ? (uint32_t)(M * stride) : here;              // entries of a query's row of counts
    const uint32_t pieces = (stored + N_ - 1) / N_ * G;       // (rows are padded to whole words)
    const uint32_t* const rows = reinterpret_cast<const uint32_t*>(a.counts + (size_t)q0 * a.pitch);
    auto fetch_counts = [&](uint32_t i, uint32_t (&in)[QL]) {
        const uint32_t at = i < pieces ? i / G : 0u;
        const int first = (int)(i % G) * QL;
#pragma unroll
        for (int q = 0; q < QL; ++q) in[q] = rows[(size_t)(first + q < nq ? first + q : 0) * (a.pitch / 4) + at];
    };
    uint32_t first_in[QL];
    fetch_counts(tid, first_in);
    constexpr int kFineRow = M * kLutStride / 8, kFineVecs = FINE ? QT * kFineRow / NT : 1;   // 16-byte pieces of a query's fine counts, of a thread
    uint32_t fine_in[kFineVecs][4];                           // (words: an array of uint4 stays in scratch memory)
    if constexpr (FINE) {
        static_assert(QT * kFineRow % NT == 0, "whole pieces");
#pragma unroll
        for (int i = 0; i < kFineVecs; ++i) {
            const int at = i * NT + tid, q = at / kFineRow;
            const uint4 x = reinterpret_cast<const uint4*>(a.fine)[(size_t)(q0 + (q < nq ? q : 0)) * kFineRow + at % kFineRow];
            fine_in[i][0] = x.x; fine_in[i][1] = x.y; fine_in[i][2] = x.z; fine_in[i][3] = x.w;
        }
    }
    FilterQuery my_par[QW];                                   // (a wave per query below, or two queries)
#pragma unroll
    for (int i = 0; i < QW; ++i) my_par[i] = a.query[q0 + (wave + i * NW < nq ? wave + i * NW : 0)];
    // (several parts: their best scores, where a few registers hold them)
    constexpr int kFew = 4;
    const int n_best = a.parts * a.best_per_part;
    float my_best[QW][kFew];
#pragma unroll
    for (int i = 0; i < QW; ++i)
#pragma unroll
        for (int j = 0; j < kFew; ++j)
            my_best[i][j] = a.parts > 1 && j * kWave + lane < n_best ? a.best[(size_t)(q0 + (wave + i * NW < nq ? wave + i * NW : 0)) * n_best + j * kWave + lane] : -__builtin_inff();
    uint32_t w[D][Sh::kWords], unit[D], inext[NI];            // slot i: a unit's codes
#pragma unroll
    for (int i = 0; i < D - 1; ++i) {
        unit[i] = (uint32_t)(i * NW + wave);
        fetch_ids(kShared, unit[i], inext);
        fetch(kShared, unit[i], inext, w[i]);
    }
    for (int i = tid; i < QT * cap; i += NT) lists[i] = 0ull;
    for (int i = tid; i < QT * kFilterBins; i += NT) hist[i] = 0u;
    if constexpr (FINE) {
#pragma unroll
        for (int i = 0; i < kFineVecs; ++i) reinterpret_cast<uint4*>(fine)[i * NT + tid] = make_uint4(fine_in[i][0], fine_in[i][1], fine_in[i][2], fine_in[i][3]);
    }
    for (uint32_t i = tid; i < pieces; i += NT) {             // entries N_ * (i / G) .. of the queries of lane i % G
        uint32_t in[QL];
        if (i == (uint32_t)tid) {
#pragma unroll
            for (int q = 0; q < QL; ++q) in[q] = first_in[q];
        } else {
            fetch_counts(i, in);
        }
        const int first = (int)(i % G) * QL;
        if (nq < QT) {
#pragma unroll
            for (int q = 0; q < QL; ++q) in[q] = first + q < nq ? in[q] : 0u;
        }
        uint32_t out[N_][W];                                  // [entry][word of the entry]
#pragma unroll
        for (int j = 0; j < W; ++j) {
            if constexpr (W16) {
                out[0][j] = __builtin_amdgcn_perm(in[2 * j + 1], in[2 * j], 0x05040100u);
                out[1][j] = __builtin_amdgcn_perm(in[2 * j + 1], in[2 * j], 0x07060302u);
            } else {                                          // four by four bytes
                const uint32_t a01 = __builtin_amdgcn_perm(in[4 * j + 1], in[4 * j], 0x05010400u), b01 = __builtin_amdgcn_perm(in[4 * j + 1], in[4 * j], 0x07030602u);
                const uint32_t a23 = __builtin_amdgcn_perm(in[4 * j + 3], in[4 * j + 2], 0x05010400u), b23 = __builtin_amdgcn_perm(in[4 * j + 3], in[4 * j + 2], 0x07030602u);
                out[0][j] = __builtin_amdgcn_perm(a23, a01, 0x05040100u);
                out[1][j] = __builtin_amdgcn_perm(a23, a01, 0x07060302u);
                out[2][j] = __builtin_amdgcn_perm(b23, b01, 0x05040100u);
                out[3][j] = __builtin_amdgcn_perm(b23, b01, 0x07060302u);
            }
        }
#pragma unroll
        for (int c = 0; c < N_; ++c) {
            Word x;
            if constexpr (W == 1) x = out[c][0];
            else if constexpr (W == 2) x = make_uint2(out[c][0], out[c][1]);
            else x = make_uint4(out[c][0], out[c][1], out[c][2], out[c][3]);
            const uint32_t e = i / G * N_ + c;
            if (e < here) reinterpret_cast<Word*>(tab)[e * G + i % G] = x;
            else if constexpr (V > 0 && CW == 1) reinterpret_cast<Word*>(a.far + (size_t)tile * ((size_t)V * stride * QT))[(e - here) * G + i % G] = x;
        }
    }
    constexpr uint32_t kLost = 0x80000000u;                   // in passed[]
    // (words that other waves write meanwhile: relaxed accesses)
    auto set_t = [&](int q, int t) {
        const int s = kFilterSpan + 1 - t;
        if constexpr (W16) lds_poke(reinterpret_cast<uint16_t*>(start) + q, (uint16_t)(s << 8));
        else lds_poke(reinterpret_cast<uint8_t*>(start) + q, (uint8_t)s);
    };
    auto t_of = [&](int q) -> int {
        if constexpr (W16) return kFilterSpan + 1 - (int)(lds_peek(reinterpret_cast<uint16_t*>(start) + q) >> 8);
        else return kFilterSpan + 1 - (int)lds_peek(reinterpret_cast<uint8_t*>(start) + q);
    };
    auto units_of_score = [&](float s, const FilterQuery& p) -> int {
        const float x = floorf((s - p.off) * p.inv - kFilterDown);
        return (int)fminf(fmaxf(x, 0.0f), (float)(kFilterSpan + 1));
    };
    if (tid < QT) { thr[tid] = 0ull; cnt[tid] = 0u; lock[tid] = 0u; }
    if (tid == 0) { *next_unit = (D - 1) * NW; *given_up = 0u; }
    uint32_t all_hopeless = 0;                                // bit i: this wave's query wave + i * NW is given up at once
#pragma unroll
    for (int i_own = 0; i_own < QW; ++i_own) {
        if (wave + i_own * NW >= QT) break;
        // a wave per query: the first T (queries that do not exist: start 0, counts 0: never at the top bit)
        const int q = wave + i_own * NW;
        FilterQuery p = q < nq ? my_par[i_own] : FilterQuery{0.0f, 0.0f, kFilterSpan + 1, 0.0f};
        bool hopeless = p.t_first >= kHopeless;
        if (hopeless) p.t_first -= kHopeless;
        if (q < nq && a.parts > 1) {
            // the K-th best of the parts' scores, to 16 bits of its order-preserving image: K of them reach it
            const int n = n_best;
            const float* v = a.best + (size_t)(q0 + q) * n;
            uint32_t at = 0;
            auto search = [&](auto per_lane) {
                constexpr int R = decltype(per_lane)::value;
                uint32_t o[R];
#pragma unroll
                for (int i = 0; i < R; ++i) o[i] = i * kWave + lane < n ? orderable_bits(R <= kFew ? my_best[i_own][i < kFew ? i : 0] : v[i * kWave + lane]) : 0u;
                for (uint32_t bit = 0x80000000u; bit >= 0x10000u; bit >>= 1) {
                    const uint32_t t = at | bit;
                    int c = 0;
#pragma unroll
                    for (int i = 0; i < R; ++i) c += __popcll(__ballot(o[i] >= t));
                    if (c >= K) at = t;
                }
            };
            if (n <= kWave) search(std::integral_constant<int, 1>());
            else if (n <= 4 * kWave) search(std::integral_constant<int, 4>());
            else search(std::integral_constant<int, kFilterBest / kWave>());
            const float f = float_of_orderable(at);
            if (f == f && f > -__builtin_inff()) {
                const int t = p.inv > 0.0f ? units_of_score(f, p) : 0;
                hopeless = hopeless && t <= p.t_first;
                p.t_first = t > p.t_first ? t : p.t_first;
                p.floor = fmaxf(p.floor, f);
            }
        }
        if (lane == 0) {
            par[q] = p;
            set_t(q, p.t_first);
            passed[q] = 0u;
        }
        all_hopeless |= (uint32_t)hopeless << i_own;
    }
    stamp<STAMP>(rec, kStampRequested, lane);
    __syncthreads();
    stamp<STAMP>(rec, kStampTables, lane);

    // Floors.  Every exact score that enters a list is counted in its query's histogram, and wave q looks after query q: now
    // and then it asks for the counters and one unit later reads off the highest T that K of the counted scores reach.
    // SHARE: the histogram is in device memory and counts for all workgroups that serve the query: the K-th best of all
    // their shares together is a far higher floor than one share's own.  For a few workgroups with long shares (serving:
    // four per query, K = 100: scan 373 -> 238 us).  Where many workgroups share a query their updates of the same counters
    // are served one by one, and a wave's loads wait behind its updates: the histogram is the workgroup's own then, in LDS
    // (256 workgroups, 20 units per wave: 46 us, 64 with a shared one).
    static_assert(kFilterBins == 2 * kWave, "two counters per lane");
    unsigned long long seen[QW] = {};                         // this lane's two counters of a query as asked for
    int until_look = 1, look_gap = 2;                         // groups of units until the next request; the gap grows by a quarter
    bool asked = false;
    auto look = [&]() {
        if (wave >= nq) return;
        if (asked) {
            asked = false;
#pragma unroll
            for (int i = 0; i < QW; ++i) {
                const int q = wave + i * NW;
                if (i > 0 && q >= nq) break;
                const uint32_t h0 = (uint32_t)seen[i], h1 = (uint32_t)(seen[i] >> 32);
                const int top = kFilterBins - 1 - 2 * lane;   // lane 0 owns the highest two
                const uint32_t upto = wave_prefix_sum(h0 + h1);
                const uint64_t has = __ballot(upto >= (uint32_t)K);
                if (has != 0) {
                    const int owner = __builtin_ctzll(has);
                    const int bin = __builtin_amdgcn_readlane(upto - h0 >= (uint32_t)K ? top : top - 1, owner);
                    const int t = par[q].t_first + bin < kFilterSpan + 1 ? par[q].t_first + bin : kFilterSpan + 1;
                    if (lane == 0 && t > t_of(q)) set_t(q, t);
                }
            }
        }
        if (--until_look <= 0) {
            const int at = kFilterBins - 2 - 2 * lane;
#pragma unroll
            for (int i = 0; i < QW; ++i) {
                const int q = wave + i * NW;
                if (i > 0 && q >= nq) break;
                if constexpr (SHARE) seen[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(a.hist + (size_t)(q0 + q) * kFilterBins + at),
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                else seen[i] = lds_peek(reinterpret_cast<const unsigned long long*>(hist + q * kFilterBins + at));
            }
            asked = true;
            look_gap += (look_gap + 3) >> 2;
            until_look = look_gap < 16 / D ? look_gap : 16 / D;
        }
    };

    // One wave makes room in query q's full list, which it has locked: keys below the present floor go; if that is not
    // enough the list is sorted and its K best stay.  Every slot has been handed out, and whoever was handed one writes it
    // without waiting for anything, so the wait for the last of them ends.
    auto make_room = [&](int q) {
        uint64_t* const list = lists + (size_t)q * cap;
        for (int t = lane; t < cap; t += kWave)
            while (lds_peek(list + t) == 0ull) __builtin_amdgcn_s_sleep(1);
        const int tq = t_of(q);
        const FilterQuery p = par[q];
        int kept = 0;
        for (int base = 0; base < cap; base += kWave) {       // in place: a chunk is in registers before its survivors
            const uint64_t key = list[base + lane];           // are written at or below its start
            const bool take = units_of_score(score_of_key(key), p) >= tq;
            const uint64_t mask = __ballot(take);
            wave_sync();
            if (take) list[kept + __popcll(mask & ((1ull << lane) - 1ull))] = key;
            kept += __popcll(mask);
            wave_sync();
        }
        if (kept > cap / 2 && kept > K + K / 4) {
            const uint64_t kth = sort_wave_list(list, cap, kept, K, lane);
            kept = K;
            if (lane == 0) lds_poke(thr + q, kth);
        }
        for (int t = kept + lane; t < cap; t += kWave) list[t] = 0ull;
        wave_sync();
        if (lane == 0) lds_poke(cnt + q, (uint32_t)kept);
        wave_sync();
    };

    // Tables whose bounds say little (a large entry that hardly any item has stretches the steps; scores that hardly differ in
    // fp32; ties) let most items through, and each of them costs what a hundred others do.  A query that has let pass a quarter
    // of the items so far, and by then so many of the whole share that they have cost about what scanning it exactly
    // costs (a twelfth; a quarter of wide rows, a twentieth with shared floors; half that while its floor has not risen), or that
    // the sample has found hopeless, is given up (counted from
    // where a wave has scored a dozen batches more than it has seen units, so that ordinary tables pay nothing): its counts
    // go to zero, so that nothing passes any more, and when the others are done its share is scanned again from the start
    // with exact scores, W queries at a time (below).
    // 1.28M items, m = 8, 64 queries with such an entry each, K = 10: 117 us instead of 808 (37 without it); 1024, K = 100: 2.5 ms
    // instead of 9.6.  (Given up at once, shared floors' queries with heavy-tailed tables took 1.3 ms instead of 0.5.)
    uint32_t batches = 0, units_seen = 0, gone = 0;           // batches scored, units seen; queries given up, as far as this wave has looked
    const uint32_t give_up_from = units * (PER * NI) / (M >= 32 ? 4u : SHARE ? 20u : 12u);
    auto give_up = [&](int q) {
        const uint32_t bit = 1u << bit_of(q);
        uint32_t before = 0;
        if (lane == 0) before = atomicOr(given_up, bit);
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)before) & bit) return;
        if (lane == 0) {
            (void)atomicOr(&passed[q], kLost);
            set_t(q, kFilterSpan + 1);                        // (as for a query that does not exist; nothing relies on it)
        }
        const uint32_t keep = W16 ? ~(0xFFFFu << (q & 1) * 16) : ~(0xFFu << (q & 3) * 8);
#pragma unroll 1
        for (uint32_t i = lane; i < here; i += kWave) atomicAnd(&tab[i * (W * G) + q / F], keep);
    };

    auto count_passed = [&](int n0) {                         // queue entries [n0, n0 + 64), which have been scored
        const int q = (int)(queue[n0 + lane] >> 32);
        // (units begun: those handed out less what the waves hold)
        const uint32_t out = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_peek(next_unit)), begun = out > (D + 2) * NW ? out - (D + 1) * NW : NW;
        const uint32_t line = begun * (PER * NI / 4);
        // (a floor that has not risen by a step yet is less likely to)
        const uint32_t from = t_of(q) == par[q].t_first ? give_up_from / 2 : give_up_from;
        uint64_t over = __ballot(atomicAdd(&passed[q], 1u) > (line > from ? line : from));
#pragma unroll 1
        while (over != 0) {
            const int qo = __builtin_amdgcn_readlane(q, __builtin_ctzll(over));
            over &= ~__ballot(q == qo);
            give_up(qo);
        }
        wave_sync();
        gone = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_peek(given_up));
    };

    // Scores queue entries [n0, n0 + n), n <= 64, exactly, one per lane, and puts what reaches its query's floor into the
    // query's list.
    constexpr int kAsked = M < 16 ? M : 16;                   // table values under way together
    // `again`: in a query's second scan
    auto process = [&](auto again, int n0, int n) {
        wave_sync();
        bool live = lane < n;
        const uint64_t entry = live ? queue[n0 + lane] : 0ull;
        const int q = (int)(entry >> 32);
        const uint32_t item = item_at((uint32_t)entry);
        uint32_t row[P / 4];
        load_row_words<P>(a.codes, item, row);
        if constexpr (FINE && !decltype(again)::value) {
            uint32_t sum = 0;
#pragma unroll
            for (int k = 0; k < M; ++k) sum += fine[(uint32_t)(q * M + k) * kLutStride + filter_sub_id<M, CW>(row, 0, k)];
            live = live && sum >= (uint32_t)t_of(q) << 8;
        }
        const float* Sq = a.S + (size_t)(q0 + q) * M * b;
        float acc = 0.0f;
        auto score = [&]() {
#pragma unroll
        for (int k0 = 0; k0 < M; k0 += kAsked) {
            float v[kAsked];
#pragma unroll
            for (int k = 0; k < kAsked; ++k) {
                const uint32_t g = filter_sub_id<M, CW>(row, 0, k0 + k);
                v[k] = Sq[(size_t)(k0 + k) * b + (g < (uint32_t)b ? g : (uint32_t)b - 1u)];   // (never outside the tables)
            }
#pragma unroll
            for (int k = 0; k < kAsked; ++k) acc = k0 + k == 0 ? v[0] : acc + v[k];
        }
        };
        if (!FINE || live) score();
        const FilterQuery p = par[q];
        const int t = units_of_score(acc, p);
        const uint64_t key = make_key(acc + 0.0f, item);
        const bool want = live && t >= t_of(q) && key > lds_peek(thr + q);
        if (want) {
            int bin = t - p.t_first;
            bin = bin < 0 ? 0 : (bin > kFilterBins - 1 ? kFilterBins - 1 : bin);
            // (a shared histogram is not cleared for the second scan: no item may be counted twice)
            if (decltype(again)::value && SHARE) {}
            else if (SHARE) (void)__hip_atomic_fetch_add(a.hist + (size_t)(q0 + q) * kFilterBins + bin, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            else atomicAdd(&hist[q * kFilterBins + bin], 1u);
        }
        // Who still has a key to place is kept as a mask in scalar registers, never as a flag per lane that goes round the
        // loop: the compiler then lets lanes that are done skip ahead and parks them outside, and the loop's steps for the
        // whole wave (lane 0 takes the lock, all lanes tidy the list) run without them.
        uint64_t left = __ballot(want);
        while (left != 0) {
            bool full = false;
            if ((left >> lane) & 1ull) {
                const uint32_t pos = atomicAdd(&cnt[q], 1u);
                full = pos >= (uint32_t)cap;
                if (!full) lds_poke(lists + (size_t)q * cap + pos, key);
            }
            left &= __ballot(full);
            if (left == 0) break;
            // a list is full: the wave that gets its lock makes room, the others try again
            const int qf = __builtin_amdgcn_readlane(q, __builtin_ctzll(left));
            uint32_t got = 1u;
            if (lane == 0) got = atomicExch(&lock[qf], 1u);
            got = (uint32_t)__builtin_amdgcn_readfirstlane((int)got);
            if (got == 0u) {
                const uint32_t now = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds_peek(cnt + qf));
                if (now >= (uint32_t)cap) make_room(qf);
                wave_sync();
                if (lane == 0) lds_poke(lock + qf, 0u);
            } else {
                __builtin_amdgcn_s_sleep(2);
            }
            wave_sync();
            left &= __ballot(key > lds_peek(thr + q));
        }
        wave_sync();
        // (while much is scored, as in the first units of a long scan, floors move fast: look every time)
        until_look = 0;
        look();
    };

    if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)all_hopeless) != 0, 0)) {
#pragma unroll 1
        for (int i = 0; i < QW; ++i)
            if ((__builtin_amdgcn_readfirstlane((int)all_hopeless) >> i) & 1) give_up(wave + i * NW);
    }

    // ---- stream
    int queued = 0;                                           // entries in this wave's queue
    uint32_t s[W];                                            // the fields' start values
    auto read_start = [&]() {
        if constexpr (W == 1) s[0] = lds_peek(start);         // (fields other waves may be raising: any value read is a floor)
        else {
#pragma unroll
            for (int j = 0; j < W; j += 2) {
                const unsigned long long x = lds_peek(reinterpret_cast<const unsigned long long*>(start) + (half * W + j) / 2);
                s[j] = (uint32_t)x; s[j + 1] = (uint32_t)(x >> 32);
            }
        }
        if constexpr (G == 1) {
#pragma unroll
            for (int j = 0; j < W; ++j) s[j] = (uint32_t)__builtin_amdgcn_readfirstlane((int)s[j]);
        }
    };
    // where a lane's part of a sub-id's row begins (pairs, one-byte sub-ids: one dot product of bytes, 32 g + 16 half)
    auto row_at = [&](const uint32_t* w, int e, int k) -> uint32_t {
        if constexpr (G == 2 && CW == 1) {
            const int byte = e * P + k;
            return __builtin_amdgcn_udot4(w[byte >> 2], (uint32_t)QT << ((byte & 3) * 8), (uint32_t)(half * QL), false);
        } else {
            return filter_sub_id<M, CW>(w, e, k) * (W * G * 4) + (uint32_t)(half * W * 4);
        }
    };
    const uint8_t* const far = V == 0 ? nullptr : a.far + (size_t)tile * ((size_t)V * stride * QT);
    auto fetch_far = [&](const uint32_t* w, Word (&x)[NI][V > 0 ? V : 1]) {
#pragma unroll
        for (int e = 0; e < NI; ++e)
#pragma unroll
            for (int v = 0; v < V; ++v) {
                // (one-byte sub-ids: a row for each of 256, and the address as in LDS)
                const size_t at = CW == 1 ? (size_t)v * stride * QT + row_at(w, e, M - V + v)
                                          : filter_far_at((uint32_t)v, filter_sub_id<M, CW>(w, e, M - V + v), (uint32_t)stride, QT, (uint32_t)(half * QL));
                x[e][v] = *reinterpret_cast<const Word*>(far + at);
            }
    };
    auto add_word = [](uint32_t (&sum)[W], const Word& x) {
        if constexpr (W == 1) sum[0] += x;
        else if constexpr (W == 2) { sum[0] += x.x; sum[1] += x.y; }
        else { sum[0] += x.x; sum[1] += x.y; sum[2] += x.z; sum[3] += x.w; }
    };
    // a unit's hits: per item a mask of the queries whose field has its top bit set
    auto scan_unit = [&](uint32_t u, const uint32_t (&w)[Sh::kWords], const Word (&x)[NI][V > 0 ? V : 1], uint32_t (&hits)[NI]) {
        uint32_t sum[NI][W];
        uint32_t any = 0;
#pragma unroll
        for (int e = 0; e < NI; ++e) {
            auto entry = [&](int k) -> Word {
                return *reinterpret_cast<const Word*>(reinterpret_cast<const uint8_t*>(tab) + (size_t)k * stride * (W * G * 4) + row_at(w, e, k));
            };
            if constexpr (NA == 1) {
#pragma unroll
                for (int j = 0; j < W; ++j) sum[e][j] = s[j];
                constexpr int STEP = M < 8 ? M : 8;
#pragma unroll
                for (int k0 = 0; k0 < M; k0 += STEP) {
                    Word v[STEP];
#pragma unroll
                    for (int k = k0; k < k0 + STEP; ++k) v[k - k0] = k < M - V ? entry(k) : x[e][k < M - V ? 0 : k - (M - V)];
#pragma unroll
                    for (int k = 0; k < STEP; ++k) add_word(sum[e], v[k]);
                }
            } else {
                // sums of four, averaged two by two: rounded up, but the last: it reaches 128 where all sums' total reaches NA * 128
                uint32_t level[6][W];
#pragma unroll
                for (int g0 = 0; g0 < NA; g0 += 2) {
                    Word v[2][filter_members(M)];
#pragma unroll
                    for (int g = 0; g < 2; ++g)
#pragma unroll
                        for (int i = 0; i < filter_members(M); ++i) {
                            const int k = filter_member(M, g0 + g, i);
                            v[g][i] = k < M - V ? entry(k) : x[e][k < M - V ? 0 : k - (M - V)];
                        }
                    uint32_t two[2][W];
#pragma unroll
                    for (int g = 0; g < 2; ++g) {
#pragma unroll
                        for (int j = 0; j < W; ++j) two[g][j] = s[j];
#pragma unroll
                        for (int i = 0; i < filter_members(M); ++i) add_word(two[g], v[g][i]);
                    }
                    // pairs of finished averages become one of the next level
#pragma unroll
                    for (int j = 0; j < W; ++j) {
                        uint32_t avg = __builtin_amdgcn_lerp(two[0][j], two[1][j], NA == 2 ? 0u : 0x01010101u);
#pragma unroll
                        for (int l = 1; (1 << l) < NA; ++l) {
                            if (((g0 >> l) & 1) == 0) { level[l][j] = avg; break; }
                            avg = __builtin_amdgcn_lerp(level[l][j], avg, (2 << l) == NA ? 0u : 0x01010101u);
                        }
                        if (g0 + 2 == NA) sum[e][j] = avg;
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < W; ++j) any |= sum[e][j];
        }
        const bool some = __ballot((any & TOP) != 0u) != 0;
#pragma unroll
        for (int e = 0; e < NI; ++e) hits[e] = 0;
        if (some) {
#pragma unroll
            for (int e = 0; e < NI; ++e) {
#pragma unroll
                for (int j = 0; j < W; ++j) hits[e] |= ((sum[e][j] & TOP) >> (W16 ? 15 : 7)) << j;
                hits[e] <<= half * W;
                if (V > 0) hits[e] &= ~gone;                  // (rows in device memory are not cleared when a query is given up)
                if (element_of(kShared, u, e) == ~0u) hits[e] = 0;
            }
        }
        return some;
    };
    if (units != 0) {
        // Groups of D units: looked up one after the other, their hits queued together.  A unit's codes are asked for D - 1 units
        // ahead, its rows in device memory one.
        int pending = 0;                                      // lane 0: the counter request in flight
        // (an increment that the compiler's combining of lanes' additions leaves alone: that waits for the answer at once)
        auto request = [&]() { if (lane == 0) pending = (int)__builtin_amdgcn_atomic_inc32(next_unit, ~0u, __ATOMIC_RELAXED, "workgroup"); };
        auto requested = [&]() -> uint32_t { return (uint32_t)__builtin_amdgcn_readfirstlane(pending); };
        request();
        uint32_t un = requested();
        request();
        fetch_ids(kShared, un, inext);
        Word x[XS][NI][V > 0 ? V : 1];
        static_assert(!AHEAD || D >= 3, "a unit's codes are here when its rows are asked for, a unit ahead");
        if constexpr (AHEAD) fetch_far(w[0], x[0]);
        while (unit[0] < units) {                             // (slot 0 holds the oldest; loads past the end are clamped and never count)
            look();
            read_start();
            uint32_t hits[D][NI], in_group[D];
            bool some = false;
#pragma unroll
            for (int i = 0; i < D; ++i) {
                if constexpr (AHEAD) fetch_far(w[(i + 1) % D], x[(i + 1) % D % XS]);
                else if constexpr (V > 0) fetch_far(w[i], x[0]);
                const int into = (i + D - 1) % D;
                unit[into] = un;
                fetch(kShared, un, inext, w[into]);
                un = requested();
                request();
                fetch_ids(kShared, un, inext);
                in_group[i] = unit[i];
                if (unit[i] < units) {
                    some = scan_unit(unit[i], w[i], x[i % XS], hits[i]) || some;
                } else {
#pragma unroll
                    for (int e = 0; e < NI; ++e) hits[i][e] = 0;
                }
            }
            units_seen += D;
            if (some) {
                // into the queue, every lane's hits in its turn: ranks from a prefix sum, and as many at a time as there is room for
                uint32_t mine = 0;
#pragma unroll
                for (int i = 0; i < D; ++i)
#pragma unroll
                    for (int e = 0; e < NI; ++e) mine += __popc(hits[i][e]);
                const uint32_t upto = wave_prefix_sum(mine);
                const uint32_t all = (uint32_t)__builtin_amdgcn_readlane((int)upto, kWave - 1);
                uint32_t rank = upto - mine, queued_to = 0;   // this lane's next hit; hits queued so far
                while (queued_to < all) {
                    const uint32_t room = (uint32_t)(kFilterQueue - queued), limit = queued_to + room < all ? queued_to + room : all;
                    uint64_t* const at = queue + queued - (int)queued_to;
#pragma unroll
                    for (int i = 0; i < D; ++i)
#pragma unroll
                        for (int e = 0; e < NI; ++e) {
                            while (hits[i][e] != 0u && rank < limit) {
                                const int q = query_of(__builtin_ctz(hits[i][e]));
                                at[rank] = ((uint64_t)q << 32) | element_of(kShared, in_group[i], e);
                                hits[i][e] &= hits[i][e] - 1u;
                                ++rank;
                            }
                        }
                    queued += (int)(limit - queued_to);
                    queued_to = limit;
                    while (queued >= kWave) {
                        queued -= kWave;
                        process(std::false_type(), queued, kWave);
                        if (__builtin_expect(++batches > units_seen + 12u, 0)) count_passed(queued);   // (as long as that is not so, nothing is counted)
                    }
                }
            }
        }
    }
    if constexpr (P < 16 && !SUB) {
        // the fewer than 16 / P items after the last whole code vector: straight to the queue of one wave of block 0
        const uint32_t first_left = total * (16 / P), n_left = (uint32_t)a.N - first_left;
        if (blk == 0 && wave == 0 && n_left != 0) {
#pragma unroll 1
            for (int q = 0; q < nq; ++q) {
                if ((uint32_t)lane < n_left) queue[queued + lane] = ((uint64_t)q << 32) | (first_left + (uint32_t)lane);
                queued += (int)n_left;
                if (queued >= kWave) {
                    queued -= kWave;
                    process(std::false_type(), queued, kWave);
                }
            }
        }
    }
    stamp<STAMP>(rec, kStampStreamed, lane);
#pragma unroll 1
    while (queued != 0) {
        const int n = queued < kWave ? queued : kWave;
        queued -= n;
        process(std::false_type(), queued, n);
    }
    stamp<STAMP>(rec, kStampOffered, lane);
    __syncthreads();

    // ---- the queries that were given up, EW at a time: lists, counters and floors as at the start, exact tables in the counts'
    // place, an item per lane; what exceeds a query's floor and its list's K-th best key goes through the queue like any hit
    // (with a pair of lanes to an item, both loading its codes: 50M items, m = 8, 32 queries, an entry that five items have: 2009 us, now 1416)
    const uint32_t units_again = share_of(kOwn);
    uint32_t todo = (uint32_t)__ballot(lane < QT && (lds_peek(passed + (lane < QT ? lane : 0)) & kLost) != 0u);
    while (__builtin_expect(todo != 0, 0)) {
        int qs[EW];
#pragma unroll
        for (int j = 0; j < EW; ++j) {
            qs[j] = todo != 0 ? __builtin_ctz(todo) : -1;
            todo &= todo - 1u;
            const int q = qs[j];
            if (q < 0) continue;
            for (int i = tid; i < cap; i += NT) lists[(size_t)q * cap + i] = 0ull;
            if (tid < kFilterBins) hist[q * kFilterBins + tid] = 0u;
            if (tid == 0) { thr[q] = 0ull; cnt[q] = 0u; set_t(q, par[q].t_first); }
        }
        for (uint32_t i = tid; i < (uint32_t)(M * stride); i += NT) {
            const uint32_t k = i / (uint32_t)stride, g = i - k * (uint32_t)stride;
#pragma unroll
            for (int j = 0; j < EW; ++j)
                tab[i * EW + j] = qs[j] >= 0 && g < (uint32_t)b ? __float_as_uint(a.S[((size_t)(q0 + qs[j]) * M + k) * b + g]) : 0u;
        }
        if (tid == 0) *next_unit = NW;
        uint32_t u = wave;
        uint32_t wa[Sh::kWords], wb[Sh::kWords];
        fetch_ids(kOwn, u, inext);
        if constexpr (P <= 16) fetch(kOwn, u, inext, wa);
        __syncthreads();
        float first_floor[EW];
#pragma unroll
        for (int j = 0; j < EW; ++j) first_floor[j] = par[qs[j] < 0 ? 0 : qs[j]].floor;
        queued = 0;
        bool done = units_again == 0;
        while (!done) {
            // (the next unit's codes on their way while this one is scored)
            int pending = 0;
            if (lane == 0) pending = (int)atomicAdd(next_unit, 1u);
            const uint32_t un = (uint32_t)__builtin_amdgcn_readfirstlane(pending);
            fetch_ids(kOwn, un, inext);
            if constexpr (P <= 16) fetch(kOwn, un, inext, wb);
            // scores that matter: above the sample's floor and the list's K-th best (none yet: key 0, whose score is a NaN and loses)
            float floor[EW];
#pragma unroll
            for (int j = 0; j < EW; ++j) floor[j] = score_of_key(lds_peek(thr + (qs[j] < 0 ? 0 : qs[j])));
#pragma unroll
            for (int j = 0; j < EW; ++j) floor[j] = qs[j] < 0 ? __builtin_nanf("") : fmaxf(floor[j], first_floor[j]);
            uint32_t hits[NI];                                // per item bit j: query qs[j]
            if (u < units_again) {
#pragma unroll
                for (int e = 0; e < NI; ++e) {
                    float acc[EW];
                    // (a few lookups on their way together: few registers, and sixteen waves hide each other's waits)
                    constexpr int kTogether = P <= 16 && M >= 8 ? 8 : 4;
                    auto add = [&](const uint32_t* row, int base, int k0, bool first) {   // sub-ids base + k0 .., of which `row` starts with `base`
                        using Exact = typename FilterWord<EW>::type;
                        Exact v[kTogether];
#pragma unroll
                        for (int k = k0; k < k0 + kTogether; ++k) v[k - k0] = reinterpret_cast<const Exact*>(tab)[(base + k) * stride + filter_sub_id<M, CW>(row, 0, k)];
#pragma unroll
                        for (int k = 0; k < kTogether; ++k) {
                            float x[EW];
                            if constexpr (EW == 1) x[0] = __uint_as_float(v[k]);
                            else if constexpr (EW == 2) { x[0] = __uint_as_float(v[k].x); x[1] = __uint_as_float(v[k].y); }
                            else { x[0] = __uint_as_float(v[k].x); x[1] = __uint_as_float(v[k].y); x[2] = __uint_as_float(v[k].z); x[3] = __uint_as_float(v[k].w); }
#pragma unroll
                            for (int j = 0; j < EW; ++j) acc[j] = first && k == 0 ? x[j] : acc[j] + x[j];
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    };
                    if constexpr (P <= 16) {
#pragma unroll
                        for (int k0 = 0; k0 < M; k0 += kTogether) add(&wa[e * P / 4], 0, k0, k0 == 0);
                    } else {                                  // wide rows: piece by piece from memory
                        const uint32_t at = element_of(kOwn, u, e);
                        const uint4* const row = reinterpret_cast<const uint4*>(a.codes + (size_t)item_at(at != ~0u ? at : 0u) * P);
                        constexpr int kPer = 16 / CW;         // sub-ids of a piece
#pragma unroll
                        for (int j = 0; j < EW; ++j) acc[j] = -0.0f;   // (-0 + x is x, whatever x)
#pragma unroll 1
                        for (int i = 0; i < P / 16; ++i) {
                            const uint4 x = row[i];
                            const uint32_t piece_words[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                            for (int k0 = 0; k0 < kPer; k0 += kTogether) add(piece_words, i * kPer, k0, false);
                        }
                    }
                    hits[e] = 0;
#pragma unroll
                    for (int j = 0; j < EW; ++j) hits[e] |= (uint32_t)(acc[j] >= floor[j]) << j;
                    if (__ballot(hits[e] != 0u) != 0) {
                        const uint32_t at = element_of(kOwn, u, e), item = at != ~0u ? item_at(at) : ~0u;
#pragma unroll
                        for (int j = 0; j < EW; ++j)
                            if (item == ~0u || make_key(acc[j] + 0.0f, item) <= lds_peek(thr + (qs[j] < 0 ? 0 : qs[j]))) hits[e] &= ~(1u << j);
                    }
                }
            } else {
                done = true;
#pragma unroll
                for (int e = 0; e < NI; ++e) hits[e] = 0;
                if constexpr (P < 16 && !SUB) {               // the items after the last whole code vector (at most 3 of EW queries)
                    const uint32_t first_left = total * (16 / P), n_left = (uint32_t)a.N - first_left;
                    if (blk == 0 && wave == 0 && n_left != 0) {
#pragma unroll
                        for (int j = 0; j < EW; ++j) {
                            if (qs[j] < 0) continue;
                            if ((uint32_t)lane < n_left) queue[queued + lane] = ((uint64_t)qs[j] << 32) | (first_left + (uint32_t)lane);
                            queued += (int)n_left;
                        }
                    }
                }
            }
            for (;;) {
                uint32_t mask = 0, item = 0, left = 0;
#pragma unroll
                for (int e = 0; e < NI; ++e) left |= hits[e];
                const uint64_t who = __ballot(left != 0u);
                if (who == 0 && !(done && queued != 0)) break;
                const bool full = queued + __popcll(who) > kFilterQueue;
                if (!full) {
                bool taken = false;
#pragma unroll
                for (int e = 0; e < NI; ++e) {
                    const bool here = !taken && hits[e] != 0u;
                    mask = here ? hits[e] : mask;
                    item = here ? element_of(kOwn, u, e) : item;
                    hits[e] = here ? hits[e] & (hits[e] - 1u) : hits[e];
                    taken = taken || here;
                    asm volatile("" : "+v"(hits[e]));
                }
                int q = 0;
#pragma unroll
                for (int j = 0; j < EW; ++j) q = (mask & (0u - mask)) == (1u << j) ? qs[j] : q;
                if (taken) queue[queued + __popcll(who & ((1ull << lane) - 1ull))] = ((uint64_t)q << 32) | item;
                queued += __popcll(who);
                }
                if (full || queued >= kWave || who == 0) {
                    const int n = queued < kWave ? queued : kWave;
                    queued -= n;
                    process(std::true_type(), queued, n);
                }
            }
            look();
            u = un;
#pragma unroll
            for (int i = 0; i < Sh::kWords; ++i) wa[i] = wb[i];
        }
        __syncthreads();
    }

    // ---- a wave per query: keys that reach the final floor, ranked by counting, straight to the workspace
#pragma unroll 1
    for (int q = wave; q < nq; q += NW) {
        uint64_t* const list = lists + (size_t)q * cap;
        const int tq = t_of(q);
        const FilterQuery p = par[q];
        const int n = (int)cnt[q] < cap ? (int)cnt[q] : cap;
        int kept = 0;
        for (int base = 0; base < n; base += kWave) {
            const uint64_t key = base + lane < n ? list[base + lane] : 0ull;
            const bool take = key != 0ull && units_of_score(score_of_key(key), p) >= tq;
            const uint64_t mask = __ballot(take);
            wave_sync();
            if (take) list[kept + __popcll(mask & ((1ull << lane) - 1ull))] = key;
            kept += __popcll(mask);
            wave_sync();
        }
        auto out = [&](int t, uint64_t key) {
            if (a.out_ids != nullptr) {
                a.out_ids[(size_t)(q0 + q) * K + t] = id_of_key(key);
                a.out_scores[(size_t)(q0 + q) * K + t] = score_of_key(key);
            } else {
                a.ws_keys[((size_t)(q0 + q) * nblk + blk) * K + t] = key;
            }
        };
        if (!SUB && p.flat()) {
            for (int t = lane; t < K; t += kWave) out(t, blk == 0 ? make_key(p.off + 0.0f, (uint32_t)t) : 0ull);
        } else if (kept > 3 * kWave) {                               // (counting costs kept^2 / 64: 192 keys as much as a sort of 256)
            sort_wave_list(list, cap, kept, K, lane);
            for (int t = lane; t < K && t < kept; t += kWave) out(t, list[t]);
            for (int t = kept + lane; t < K; t += kWave) out(t, 0ull);
            kept = 0;
        } else {
            for (int t = kept + lane; t < K; t += kWave) out(t, 0ull);
        }
        const int n8 = (kept + 7) & ~7;                       // (cap is a multiple of 8)
        if (kept + lane < n8) list[kept + lane] = 0ull;
        wave_sync();
        for (int t = lane; t < kept; t += kWave) {
            const uint64_t mine = list[t];
            uint32_t rank = 0;
            for (int u = 0; u < n8; u += 8) {
                const ulonglong2 p0 = *reinterpret_cast<const ulonglong2*>(list + u), p1 = *reinterpret_cast<const ulonglong2*>(list + u + 2);
                const ulonglong2 p2 = *reinterpret_cast<const ulonglong2*>(list + u + 4), p3 = *reinterpret_cast<const ulonglong2*>(list + u + 6);
                rank += (uint32_t)((p0.x > mine) + (p0.y > mine) + (p1.x > mine) + (p1.y > mine) + (p2.x > mine) + (p2.y > mine) +
                                   (p3.x > mine) + (p3.y > mine));
            }
            if (rank < (uint32_t)K) out((int)rank, mine);
        }
    }
    if (wave < nq) stamp<STAMP>(rec, kStampSelected, lane);
    stamp<STAMP>(rec, kStampEnd, lane);
}
