// PQTopK scoring for gfx950 (MI355X): kernels and the C ABI declared in include/pqtopk.h.
//
// Path (paper Section 3): pq_subitem_scores() builds the sub-id score matrix S (Eq. 4); pq_score_topk() streams the
// codebook G once, turns every item's m sub-ids into a score by m table lookups in LDS (Eq. 5), and keeps only the
// K best <id, score> pairs (Algorithm 1, V = I).  Item scores never reach memory.
//
// Total order used everywhere: a 64-bit key  (orderable(score) << 32) | ~id.  A larger key is a better item:
// higher score first, lower id between equal scores.  Keys of distinct items are distinct, key 0 means "empty".
//
// Shape of pq_score_topk(): one scan launch, then a small fold launch (none when one workgroup per query does).  The scans, by
// what they are for:
//   scan_short_kernel (scan_short.hpp; scan_subset_kernel for candidate lists): a workgroup's share fits its registers as scores, up to
//     64 per thread: single queries over up to 8M items, batches over small catalogues.  The K best are selected from there.
//   scan_pair_kernel (scan_pair.hpp): the same for two queries per workgroup: a few queries, or many over small catalogues.
//   scan_long_kernel (scan_long.hpp): a single query over more, in segments of registers.
//   scan_filter_kernel (scan_filter.hpp; filter_prepare_kernel before it takes a sample for the first floors and makes the tables):
//     batches.  Upper bounds of 8 or 16 bits for up to 32 queries are summed with one LDS read per sub-id; only what reaches
//     a query's floor is scored exactly.
//   scan_topk_tiled_kernel (scan_batched.hpp; m = 8 or 16): large batches over catalogues too small for bounds to pay, four queries per
//     16-byte LDS read.
//   scan_topk_kernel (scan_single.hpp): everything else: any row length, tables that do not fit LDS, the longest single-query scans
//     (sixteen copies of the tables, per-wave lists, floors from a running histogram).
//   fold_lists_kernel or fold_small_kernel (fold.hpp; one workgroup per query) reduces the workgroups' lists to the final sorted K.
// Floors and histograms only ever prune; every decision that picks a winner compares full keys, so the result is
// exact for any input, including heavy ties (which merely take slower paths).
//
// This file holds the host side (plans, launches, the extern "C" entry points).  The device code is in the .hpp parts
// that kernels.hpp gathers in namespace pqk; the large scan kernels are compiled in the inst_*.hip translation units
// and only launched from here.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <tuple>

#include "pqtopk.h"
#include "pqtopk_measure.h"
#include "kernels.hpp"

// Built-in scratch of pq_score_topk_static(): device memory, one copy per GPU, held until the process ends.  Host code
// never uses this name as an address (it is a handle for hipGetSymbolAddress(), see static_scratch() below).
// Behind the bytes that decide what is taken there is room for the rows of counts that a batch's scan looks up in device memory: with these
// among the 8 MiB, batches that otherwise fit were scanned without bounds (102,314 items, m = 8, 3141 queries, K = 2: 416 us instead of 97;
// 699,551, 2485, K = 18 1427 and 321).  A query has at most 768 bytes of rows beside at least five times as many others.
constexpr size_t kStaticScratchBytes = PQ_STATIC_SCRATCH_BYTES, kStaticRowsBytes = PQ_STATIC_SCRATCH_BYTES / 4;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes + kStaticRowsBytes];

namespace {

using namespace pqk;

// ---------------------------------------------------------------------------------------------------------------
// host side

thread_local char g_hip_error[256] = "no HIP error recorded";

// pq_measure_force_general(): bit 0 keeps calls off the short and long scans and off those by pairs of queries, bit 1 off fold_small_kernel, bit 2
// Eq. 4 off the matrix cores, bit 3 off the scans by upper bounds; bit 4 on them wherever they can; bit 5 spreads short candidate lists
// over the chip; bit 6: longer single queries always in segments; bit 7: scans by upper bounds by pairs of lanes wherever these fit; bit 8: batches by
// pairs of queries wherever these fit; bit 9 keeps single queries off the scan by one-byte bounds; bit 10: on it wherever it fits (0: the product's choice)
std::atomic<int> g_force_general{0};

int record_hip(hipError_t e) {
    if (e == hipSuccess) return PQ_OK;
    (void)hipGetLastError();                                 // (reported here: not a second time by whoever asks next)
    strncpy(g_hip_error, hipGetErrorString(e), sizeof(g_hip_error) - 1);
    g_hip_error[sizeof(g_hip_error) - 1] = 0;
    return PQ_ERR_HIP;
}

int next_pow2(int x) {
    int p = 1;
    while (p < x) p <<= 1;
    return p;
}

// Keys per wave list: a power of two (the overflow path sorts it) with room for K kept keys plus a wave's worth of
// new ones, and at least K / 4: a list that holds K of its `cap` keys for good is sorted every cap - K appends
// (K = 448 in 512 slots sorted every 64 keys: twice as slow as K = 449 in 1024).
int list_capacity(int K) {
    const int spare = K / 4 > kWave ? K / 4 : kWave;
    const int cap = next_pow2(K + spare);
    return cap < 128 ? 128 : cap;
}

struct ScanPlan {
    int copies;      // single-query kernel: copies of the score tables in LDS (1 or kTableCopies)
    bool tiled;      // batched kernel: kQ queries per workgroup
    bool big;        // single-query kernel: kBigThreads threads per workgroup, one workgroup per CU
    int nblk;        // item blocks per query
    bool direct;     // nblk is 1 and the scan writes the result itself
    int cap;         // keys per wave list
    int candmax;     // keys of the candidate array
    size_t scan_dyn_lds;     // dynamic LDS of the scan launch
    size_t scan_lds;         // dynamic + the static score tables of the vector kernels
    size_t fold_lds;
    bool vec;
    bool glut;       // two-byte sub-ids: the m x b table does not fit LDS and is read from device memory
    bool short_scan; // scan_short_kernel: every workgroup's share fits its registers, K small
    int short_units; // ... units (code vectors, or items for m = 32, 64) a thread holds
    bool bytes;      // scan_bytes_kernel: one query's long catalogue by one-byte upper bounds
    bool long_scan;  // scan_long_kernel: one query's catalogue in segments
    bool pair_scan;  // scan_pair_kernel: as the short scan, two queries per workgroup (short_units: what a thread holds)
    bool short_subset; // scan_subset_kernel: a candidate list whose share per thread fits its registers, K small
    bool subset_pair;  // scan_subset_pair_kernel: the same, two queries per workgroup
    int subset_vecs;   // ... code vectors' worth of gathered rows a thread holds
    bool filter;       // filter_prepare_kernel + scan_filter_kernel: a batch scanned by integer upper bounds
    int f_words;       // ... 32-bit words of a table entry
    bool f_w16;        // ... 16-bit fields (8-bit otherwise)
    bool f_fine;       // ... 16-bit counts beside 8-bit fields
    bool f_near;       // ... all splits in LDS
    int f_queries;     // ... queries per workgroup
    int f_cap;         // ... keys of a query's list
    int f_lanes;       // ... lanes that share an item (1 or 2)
    size_t f_pitch;    // ... bytes of a query's counts that go to LDS
    int f_far;         // ... splits whose counts stay in device memory (f_near: none)
    int f_stride;      // ... table entries of a split
    bool f_share;      // ... the workgroups of a query share their floors
    bool f_patient;    // ... which rise so far that the sample gives no query up
    int f_prepare;     // ... threads of a workgroup that takes a part of the sample
    int f_sample;      // ... units of a part's sample
    int f_rounds;      // ... rounds of a part's sample
    int f_parts;       // ... parts of the sample
    int f_best;        // ... scores a part leaves (several parts)
    long long f_entries;  // ... table entries
    int f_batch;       // ... queries scanned together (larger batches in turns, so that the tables of counts stay bounded)
};

// What make_plan() may choose from.
enum { kNoFilter = 1, kNoLong = 2, kNoPair = 4, kNoBytes = 8 };

bool is_vec_m(int m) { return m == 1 || m == 2 || m == 4 || m == 8 || m == 16 || m == 32 || m == 64; }

bool is_vec_m16(int m) { return m == 4 || m == 8 || m == 16; }   // 16-bit sub-ids: rows of 8, 16 or 32 bytes

// With a multiple of 8 blocks per query, block x of every query runs on XCD x % 8 and the queries share that XCD's L2
// (worth about 5 %): taken when it costs at most a sixteenth of the blocks.
long long xcd_aligned(long long nb, int B) {
    return (B > 1 && (nb & 7) * 16 <= nb) ? (nb & ~7LL) : nb;
}

// Item blocks per query when B single-query scans run side by side on `slots` workgroup slots (CUs times resident
// workgroups) and B is too large for eight blocks each: as many as fill the slots once, or a few times over when one
// filling would leave many idle.  Cost of a choice: (fillings) x (a block's share of the query's streaming time, which
// the table lookups bound at 9.1 per clock and CU, plus some 8 us per workgroup for tables, first cut and selection).
long long blocks_for_many_queries(long long slots, long long B, long long rounds, double lookups_per_query) {
    const double stream_us = lookups_per_query / (9.1 * 2400.0);
    long long best_nb = 1;
    double best_us = 0.0;
    for (int fill = 1; fill <= 8; ++fill) {
        long long nb = slots * fill / B;
        if (nb > rounds) nb = rounds;
        if (nb < 1) nb = 1;
        const long long fillings = (B * nb + slots - 1) / slots;
        const double us = (double)fillings * (stream_us / (double)nb + 8.0);
        if (fill == 1 || us < best_us) { best_us = us; best_nb = nb; }
    }
    return best_nb;
}

// Lookups (B * N * m) from which the batched kernel beats B single-query scans side by side.  Measured on catalogues
// of 3e5 to 2e7 items: its fixed costs (about 15 us of tables, first cuts and final merge, more with K) are paid back
// from 2e8 lookups on at K = 10.  At m = 8 the side-by-side scans run with replicated tables as long as their lists
// leave room for them (K <= 64) and then stay ahead up to 8e8 lookups; for K > 128 their shared floors do.
double tiled_min_lookups(int m, int K) {
    if (m == 8) {
        if (K <= 12) return kTiledMinLookups * (1.0 + K / 400.0);
        if (K <= 64) return 8.5e8;
        if (K <= 128) return 3.5e8;
        return 9.0e8;
    }
    return K <= 128 ? kTiledMinLookups * (1.0 + K / 400.0) : 5.0e8;
}

// Units (code vectors; items of 32 bytes and more) per thread up to which one workgroup scans a query's whole catalogue and
// writes the result: the scan takes up to 3 us longer than spread over the chip, the fold's launch (3 us of host time, 3.7 us
// from the scan's end to the result) is saved.
constexpr long long kDirectUnits(int row) { return row <= 16 ? 8 : row == 32 ? 4 : 2; }

// Where one workgroup takes all N candidates of a query's list and writes the result itself.  A compute unit gathers about one row
// per clock, whatever its length, and looks up m entries for it: a candidate costs m + 8 here.  Spread over the chip this passes, but
// the fold's launch (3 us of host time) comes on top, and so do the tables that every workgroup loads, the more of the chip B queries
// fill.  Calls back to back, where the host's time is hidden (bench.py --rules; one workgroup and spread, us): m = 4, B = 1, K = 10:
// 4800 candidates 6.0 and 6.3, 7700 8.0 and 6.3, 9600 8.8 and 6.4; B = 30, K = 40: 5700 6.8 and 9.2, 11,400 10.9 and 10.0; B = 100,
// K = 200: 15,600 17.9 and 18.5; m = 8, B = 1: 3600 5.7 and 6.1, 7200 8.7 and 6.3 (K = 300: 10.9 and 10.5).  The line lies where one
// launch less still pays for a program that the host's time bounds: at B = 1 up to 2.4 us of the GPU's time above the other side.
bool subset_direct_pays(long long N, int m, int B) {
    if (N * m > kDirectUnits(16) * 16LL * kThreads) return false;
    return N * (m + 8) <= (112LL << 10) + 720LL * B;
}

// Bytes of codes from which one query's catalogue is scanned by one-byte bounds (scan_bytes_kernel): before that its sample, counts and lists per wave
// weigh more than the lookups and the uneven rounds that it saves.  Popular sub-ids (codes by Zipf(1.1)) collide less in exact tables, so the lines of long rows and many results lie where these
// gain too.  Calls without and with (us; uniform codes from several catalogues in turn, so that no cache holds them; Zipf: one catalogue), just below the lines and further on:
// m = 4: 8M items, K = 10 16.4 and 17.2, 11M 19.5 and 18.8, Zipf 19.4 and 18.6, K = 100 25.4 and 25.8, 17.5M 32.3 and 30.1, K = 512 14M 39.1 and 45.0, 22M 56.3 and 52.3;
// m = 8: 5M, K = 10 17.7 and 18.0, 6.5M 22.7 and 19.8, Zipf 20.2 and 19.2, K = 100 10M 31.1 and 31.2, 13.8M 36.7 and 35.4, Zipf 35.7 and 34.7, K = 256 13.8M 41.6 and 41.9, 17.5M 48.5 and 46.8, Zipf 47.5 and 46.2,
// K = 512 13.8M 46.8 and 54.5, 22.5M 68.9 and 66.9, Zipf 67.1 and 65.4;
// m = 16: Zipf, K = 10 6M 23.7 and 24.4, 6.5M (no longer the short kernel) 29.4 and 25.5, uniform 7M 33.6 and 27.3; K = 100 8M 35.3 and 35.8, 9M 39.9 and 38.4, uniform 43.9 and 39.6; K = 256 14M 56.2 and 56.8, 16M
// 61.4 and 61.3, uniform 66.4 and 61.9;
// m = 32: Zipf, K = 10 4M 29.1 and 29.2, 4.5M (likewise) 34.7 and 31.6, uniform 4.7M 39.5 and 34.1; K = 100 4.7M 44.8 and 39.1, uniform 3.2M 33.9 and 34.2; K = 256 8M 57.9 and 61.5, 10M 72.1 and 70.7, uniform 78.8 and 71.9;
// m = 64: Zipf, K = 10 9M 104.0 and 107.8, 20M 219 and 222, 40M 429 and 424, uniform 9M 112.6 and 108.8, 40M 443 and 424; K = 100 and 256 alike.
// Two bytes: what they gain is the memory's rate (units of one vector, 6.3 TB/s instead of 5.9), the less the larger the tables that come first, and nothing while the last-level cache holds the
// codes (in brackets: one catalogue over and over).  m = 4, b = 1500: 14M, K = 10 29.1 and 29.1, 19M (33.4 and 33.9), 30M (46.9 and 45.1); b = 3500: 30M 50.3 and 49.1 (47.1 and 47.2), 60M 89.8 and 85.4; m = 8, b = 1024:
// 12.5M 40.8 and 41.4 (38.3 and 39.7), 16M 50.1 and 50.3 (46.6 and 48.7), 19M 56.2 and 55.2, 45M 126.4 and 120.5; b = 1500: 20M 61.3 and 60.2 (60.1 and 59.8), 30M 88.5 and 85.0; m = 16, b = 300: 4M 29.2 and 31.5, 5M (no
// longer the short kernel) 37.4 and 36.6, K = 100 46.0 and 41.0; b = 800: 10M, K = 10 62.9 and 63.5, 15M 88.7 and 89.6.  Zipf codes give the same there.
bool bytes_pay(long long N, int m, int b, int K, int cw) {
    const double bytes = (double)N * m * cw;
    if (cw == 2) return m * b <= 9000 ? bytes >= (m == 4 ? 2.0e8 : m == 8 ? 3.0e8 : 1.5e8) : m < 16 && bytes >= 4.5e8;
    switch (m) {
        case 4: return bytes >= (K <= 16 ? 4.4e7 : K <= 256 ? 7.0e7 : 9.0e7);
        case 8: return bytes >= (K <= 16 ? 5.2e7 : K <= 128 ? 1.1e8 : K <= 256 ? 1.4e8 : 1.8e8);
        case 16: return bytes >= (K <= 16 ? 1.0e8 : K <= 128 ? 1.4e8 : 2.5e8);
        case 32: return bytes >= (K <= 16 ? 1.35e8 : K <= 128 ? 1.5e8 : 3.2e8);
        case 64: return bytes >= 2.5e9;
        default: return false;
    }
}

// Where one query's catalogue is scanned in segments (scan_long_kernel) and not by the general kernel's per-wave lists: while the first
// cut, the lists' merge and the sorting of full lists weigh more than the general kernel's twice as many waves.  Both sides
// around the lines (bench.py --rules; segments and general, us): m = 4, K = 10: 16M items 22.2 and 22.8, 18M 24.6 and 23.8 (K = 257 on
// 40M: 73 and 56, on the wrong side of its line); m = 8: 19M 34.9 and 36.2 at K = 10, 40.6 and 51.2 at K = 80; 21M 37.7 and 38.2, 44.2
// and 54.2 (the line in K could lie lower); 42M at K = 128 79.8 and 87.1, at 257 96.5 and 95.6; m = 16: within 4 % at K = 10 and 31,
// 16M at K = 80 61 and 67; m = 32, 12M: 86.8 and 91.6 at K = 129; m = 64: 5M 85.2 and 79.5 at K = 257; two bytes, m = 4: 13M 26.9 and
// 29.9 at K = 10, 40M at K = 256 88 and 83; m = 8: 40M 113 and 121; m = 16: within 3 %.
bool long_scan_pays(long long N, int m, int K, int cw) {
    if (cw == 2) return m == 4 ? K <= 256 || N <= 12000000 : m == 8 || (m == 16 && K > 256);
    switch (m) {
        case 4: return K > 256 || N <= 17000000;
        case 8: return K > 256 || N <= 20000000 || (K > 80 && (K <= 128 || N <= 40000000));
        case 16: return K > 80 || (K >= 32 && N <= 17000000);
        case 32: return K > 128;
        case 64: return K > 256;
        default: return false;
    }
}

// Where two queries per workgroup (scan_pair_kernel) beat one: half the lookups, for a second selection (and twice the lists), which
// costs the more the more results there are.  Around the lines (us, without Eq. 4; one and two): m = 8, 1.28M items, 2 queries (20M
// lookups): K = 12 12.6 and 11.4, K = 48 13.0 and 13.9; 4 queries (41M): K = 48 17.1 and 16.2, 64 17.6 and 16.9, 100 19.1 and 20.2;
// m = 16, 300,000, 12 (58M): K = 100 22.4 and 20.7; m = 4, 1M, 6 (24M): K = 12 12.8 and 13.9; 236,127, 34 (32M): K = 59 21.6 and 17.2;
// m = 64, 400,000, 4 (102M): K = 400 31.7 and 28.3, 83,912, 15 (81M): K = 152 27.4 and 30.8.  A single workgroup per query leaves no lists
// to fold: with 22,906 items, m = 8, 170 queries 13.0 and 11.7, 14,183 10.2 and 12.8 (m = 64: 3400 14.5 and 16.5).  The general kernel
// is the slower one wherever shares fit (m = 8, 37,863, 170, K = 23: 20.4 and 15.2; two bytes, 42,619, 357, K = 434: 237 and 69), but for
// many results of more queries than compute units, over more blocks than one (m = 16, 28,254, 455, K = 157: 53.6 and 62.0).
constexpr double kPairLookupsPerUs = 20000.0;         // a CU's
bool pair_pays(const ScanPlan& p, long long N, int B, int m, int K) {
    double least = 2.0e7;
    if (p.short_scan) {
        if (p.nblk == 1 && B <= kAssumedCUs && N * m < (m >= 32 ? 300000 : 160000)) return false;
        least = K <= 12 ? (m >= 32 ? 3.0e7 : 2.0e7) : K <= 32 ? 3.0e7 : K <= 64 ? 4.0e7 : m >= 32 ? 1.0e8 : 6.0e7;
        if (m == 4) least *= 1.5;
    }
    return (double)B * (double)N * m >= least;
}
double filter_min_lookups(int m, int K, int B, bool subset, int cw);
// ... and beat the scan by bounds, which has its sample and tables to make first: m = 8, 200,000 items, 44 queries (71M lookups) 21.6 and 17.9,
// 45,066, 226 (81M) 20.5 and 18.0, 420,542, 50 (168M) 37.8 and 65.3; m = 16, 64,130, 110 (113M) 24.9 and 21.3, 43,359, 620 (430M) 78.7 and 70.6,
// 85,925, 175 (241M) 37.0 and 42.7; m = 8, 28,000, 512, K = 50 63.9 and 31.6, K = 10 26.0 and 26.3, 36,000, 900, K = 50 80.5 and 64.9, 48,000 79.2 and 85.3; m = 64, 61,190, 78 (305M) 55.8 and 43.4; m = 4, 2.6M, 7 (73M) 17.0 and 20.5.
// Lists: the rows that are gathered, once per pair and at most, against once per sixteen queries. By bounds and by pairs: m = 8, 17,851 candidates, 158
// queries 22.7 and 16.1, 100,000, 100 25.7 and 42.3, 900,000, 4 38 and 26, 6 39 and 53, 2M, 2 60 and 46, 4 60 and 82; m = 4, 900,000, 4 36 and 23, 2M, 4 55 and 73;
// m = 16, 400,000, 4 28 and 18, 6 28 and 31, 900,000, 4 37 and 42, 2M, 2 58 and 49.
// Few results: m = 16 with more than 24 vectors to a thread (`held`; one workgroup to a compute unit), 40,000 items, 450 queries, K = 5 41.1 and 45.2, 650 49.5 and 67.1, 800,
// K = 16 60.4 and 87.7, 35,000, 600, K = 2 41.5 and 59.5, K = 20 71.1 and 62.0; m = 32, 30,000, 530, K = 2 70.5 and 84.8, 800, K = 5 96 and 119, 450, K = 5 66.8 and 60.8, 650,
// K = 10 94.6 and 88.6, 40,000, 800, K = 10 114 and 149.
bool pair_beats_bounds(long long N, int B, int m, int K, bool subset, int cw, int held) {
    const double all = (double)B * (double)N * m, least = filter_min_lookups(m, K, B, subset, cw);
    if (subset) return N * ((B + 1) / 2) <= (m == 16 && B > 2 ? 1000000 : 2100000);
    if (cw == 1 && m == 16 && B > kAssumedCUs && held > 24 && K <= (N >= 38000 ? 20 : 4) && N >= 33000) return false;
    if (cw == 1 && m == 32 && B > 2 * kAssumedCUs && K <= 10 && N >= (K <= 5 ? 26000 : 36000)) return false;
    return m > 4 && (all < 1.35 * least || N < (m > 8 ? 48000 : K >= 32 ? 40000 : 24000));
}
// Workgroups whose last round would leave more than a quarter of the compute units' time idle (10,045 candidates, m = 16, 538 queries: 269
// workgroups 54.4 us, by the general kernel 40.0; 17,113, 531: 532 69.7 and 58.2; 16,000, 700: 700 42.2 and 57.1).
// (`idle`: per cent.)  More than 512 queries with rows of 16 bytes, at 16,000 candidates and more, from an eighth on: 17,780, 652, K = 1 (15 %) 66.9 and 57.4
// (59,869, 262, K = 118, as much idle, 105 and 127).
bool last_round_empty(long long groups, int idle = 25) {
    const long long rounds = (groups + kAssumedCUs - 1) / kAssumedCUs;
    return rounds > 1 && 100 * groups < (100 - idle) * rounds * kAssumedCUs;
}
// Candidate lists by two queries per workgroup (scan_subset_pair_kernel; us, without): instead of the general kernel, m = 8: 11,583 candidates, 172
// queries, K = 48 32.6 and 16.8; 100,000, 30, K = 300 48.1 and 23.8; m = 16: 17,825, 162 29.7 and 19.6, 76,492, 296, K = 422 198 and 169, 5086,
// 146 (12M lookups) 17.2 and 21.0; m = 4: 159,107, 30 35.2 and 20.6, 32,174, 786, K = 150 146 and 125.  Instead of one query per workgroup,
// m = 4: 77,144, 35 20.5 and 16.2, 12,846, 230 18.7 and 17.2, 99,700, 12 (5M) 13.7 and 13.4; m = 8: 148,492, 7 13.8 and 13.2, 20,032, 68, K = 137
// 19.5 and 21.8.
bool subset_pair_pays(const ScanPlan& p, long long N, int B, int m) {
    return !(p.short_subset && m > 4) && (double)B * (double)N * m >= (p.short_subset ? 1.0e7 : 1.5e7);
}

// `generic`: plan for the generic kernel whatever m is (candidate-list scans use it: their rows are gathered)
// `cw`, `b`: bytes per sub-id (1 or 2) and, for two-byte sub-ids, the alphabet size (it sizes the tables in LDS)
size_t workspace_bytes(const ScanPlan& p, int B, int K);
void plan_filter(ScanPlan& p, long long N, int B, int m, int K, bool subset, int cw, int b);

ScanPlan make_plan(long long N, int B, int m, int K, bool generic = false, int cw = 1, int b = kLutStride, int without = 0) {
    ScanPlan p;
    const int row = m * cw;                                    // bytes of an item's row
    size_t lut_floats = cw == 1 ? (size_t)m * kLutStride : (size_t)m * b;
    p.cap = list_capacity(K);
    p.candmax = next_pow2(2 * K);
    if (p.candmax < 512) p.candmax = 512;
    // two-byte sub-ids whose table leaves no room in LDS (even for one 1024-thread workgroup): lookups go to memory
    p.glut = cw == 2 && scan_lds_bytes(lut_floats, p.cap, p.candmax, K, kMaxWaves) > kMaxLdsBytes;
    if (p.glut) lut_floats = 0;
    p.vec = !generic && (cw == 1 ? is_vec_m(m) : is_vec_m16(m)) && N * row >= 16;   // (one whole code vector at least)
    const long long units = (p.vec && row <= 16) ? (N * row) / 16 : N;   // whole code vectors (the few items after them are extra)
    const long long per_round = (long long)kThreads * (p.vec ? vec_per_thread(row) : kGenericItemsPerThread);
    long long rounds = (units + per_round - 1) / per_round;
    const double lookups = (double)N * m;                           // table lookups of one query's scan
    long long most = (kBlocksPerCU * (long long)kAssumedCUs) / B;   // workgroups over the whole grid
    if (most < 8) most = blocks_for_many_queries(kBlocksPerCU * (long long)kAssumedCUs, B, rounds, lookups);
    long long nblk = rounds < most ? rounds : most;
    long long one_per_cu = kAssumedCUs / B;                    // a short scan is spread evenly: one workgroup per CU, which
    if (one_per_cu < 8) one_per_cu = 8;                        // then takes two or three (possibly ragged) rounds
    if (rounds > one_per_cu && rounds <= most) nblk = one_per_cu;
    if (nblk < 1 || (rounds <= kRing && N >= K)) nblk = 1;    // (what one workgroup holds in registers: no fold)
    nblk = xcd_aligned(nblk, B);
    p.nblk = (int)nblk;
    p.copies = 1;
    // A long scan for few queries is bound by LDS bank conflicts of the random lookups: with kTableCopies copies of
    // the tables, lanes l and l' collide only if l % kTableCopies == l' % kTableCopies.  Worth its LDS and fill time
    // only when every workgroup streams many rounds; one workgroup per CU then (the tables take 128 KB at m = 8).
    if (cw == 1 && p.vec && m <= 8) {
        const long long big_round = (long long)kBigThreads * vec_per_thread(m);
        const long long big_rounds = (units + big_round - 1) / big_round;
        long long nb = kAssumedCUs / B;                        // one workgroup (of kBigThreads) per CU over the whole grid
        if (nb < 8) nb = blocks_for_many_queries(kAssumedCUs, B, big_rounds, lookups);
        const size_t dyn = scan_lds_bytes((size_t)m * kLutStride * kTableCopies, p.cap, p.candmax, K, kMaxWaves);
        if (big_rounds >= kTableCopiesMinRounds * nb && dyn <= kMaxLdsBytes) {
            p.copies = kTableCopies;
            p.nblk = (int)nb;
        }
    }
    // A scan whose tables leave room for only one 512-thread workgroup per CU (generic: m > 36 or so; m = 64; large
    // alphabets of two-byte sub-ids) runs 1024-thread workgroups instead, one per CU: the same tables then serve
    // sixteen waves, which is what hides the latency of the row loads.  Only when there is more than one workgroup's
    // worth of work per CU.
    p.big = p.copies > 1;
    if (!p.vec || m == 64 || cw == 2) {
        const size_t small = scan_lds_bytes(lut_floats, p.cap, p.candmax, K, kWaves);
        const size_t big = scan_lds_bytes(lut_floats, p.cap, p.candmax, K, kMaxWaves);
        const long long big_round = (long long)kBigThreads * (p.vec ? vec_per_thread(row) : kGenericItemsPerThread);
        const long long big_rounds = (units + big_round - 1) / big_round;
        long long nb = kAssumedCUs / B;
        if (nb < 8) nb = blocks_for_many_queries(kAssumedCUs, B, big_rounds, lookups);
        if (2 * small > kMaxLdsBytes && big <= kMaxLdsBytes && rounds > nb) {
            if (big_rounds < nb) nb = big_rounds;
            nb = xcd_aligned(nb, B);
            p.big = true;
            p.nblk = (int)nb;
        }
    }
    const bool static_lut = p.vec && p.copies == 1 && cw == 1;   // tables in the kernel's static LDS array
    const size_t lut_dyn = p.copies > 1 ? lut_floats * p.copies : (static_lut ? 0 : lut_floats);
    p.scan_dyn_lds = scan_lds_bytes(lut_dyn, p.cap, p.candmax, K, p.big ? kMaxWaves : kWaves);
    p.scan_lds = p.scan_dyn_lds + (static_lut ? lut_floats * sizeof(float) : 0);
    p.tiled = false;
    // (a small batch over a small catalogue is faster as B single-query scans side by side: the batched kernel's
    // fixed costs, about 15 us of table fill, first-round cuts and final merge, are not yet paid back)
    const bool small_job = B <= 2 || (double)B * (double)N * m <= tiled_min_lookups(m, K);
    if (cw == 1 && !generic && !small_job && (m == 8 || m == 16) && N * m >= 16) {   // batched kernel, if its tables and lists fit in LDS
        const size_t dyn = tiled_lds_bytes(p.cap, p.candmax, K);
        const size_t all = dyn + (size_t)kQ * m * kLutStride * sizeof(float);
        if (all <= kMaxLdsBytes) {
            p.tiled = true;
            p.scan_dyn_lds = dyn;
            p.scan_lds = all;
            const long long tiles = (B + kQ - 1) / kQ;
            const long long t_round = (long long)kThreads * kTileVecs;
            const long long t_rounds = (units + t_round - 1) / t_round;
            // Item blocks per tile: as many as fill the CUs once, or twice or three times over when a single filling
            // would leave many CUs idle (96 tiles: 2 blocks = 192 workgroups, 5 blocks = 480).  The LDS is the bound, so
            // L workgroups on a CU take L times a workgroup's streaming time, plus fixed costs per workgroup (tables,
            // first-round cuts, final merge; measured: 28 us, and 20 + 0.75 K us for every further workgroup on the CU;
            // streaming: 1.3 ns per code vector and tile).
            const double stream_us = 1.3e-3 * (double)units;
            double best_us = 0.0;
            long long nb = 1;
            for (int fill = 1; fill <= 3; ++fill) {
                long long cand = ((long long)kAssumedCUs * fill) / tiles;
                if (cand > t_rounds) cand = t_rounds;
                if (cand < 1) cand = 1;
                const long long per_cu = (tiles * cand + kAssumedCUs - 1) / kAssumedCUs;   // workgroups on the busiest CU
                const double us = (double)per_cu * stream_us / (double)cand + 28.0 + (20.0 + 0.75 * K) * (double)(per_cu - 1);
                if (fill == 1 || us < best_us) { best_us = us; nb = cand; }
            }
            p.nblk = (int)nb;
        }
    }
    p.fold_lds = fold_lds_bytes(K);
    // Single-query scans (one query per workgroup row) whose share per thread fits a few registers run
    // the short kernel: scores stay in registers, one selection, a few KB of code.  Its grid is spread as thin as the
    // CUs allow (one workgroup per CU over all queries): a workgroup's time is the lookups of its share plus a fixed
    // selection, so the fewer units a thread holds the better, and the small fold takes the 256 lists in its stride.
    p.short_scan = false;
    p.short_units = 0;
    // (two-byte sub-ids: when the table fits LDS beside the selection's few KB)
    const size_t table16 = cw == 2 ? align16((size_t)m * b * sizeof(float)) : 0;
    auto select_lds = [](bool small) { return small ? sizeof(SmallSelectLds<kThreads>) : sizeof(MidSelectLds<kThreads>); };
    const bool short16 = cw == 2 && table16 + select_lds(K <= small_k_max(row)) <= kMaxLdsBytes;
    if ((cw == 1 || short16) && p.vec && !generic && !p.tiled) {
        long long nb = kAssumedCUs / B;
        if (nb < 1 || units <= kDirectUnits(row) * (long long)kThreads) nb = 1;
        const long long thin = (units + kThreads - 1) / kThreads;          // workgroups if every thread held one unit
        if (nb > thin) nb = thin;
        const long long per_slot = (long long)kThreads * nb;               // units one slot of all threads covers
        const long long slots = (units + per_slot - 1) / per_slot;
        const int instance = slots <= 48 ? short_instance((int)slots, cw == 1 ? short_held_units(m) : short16_held_units(m)) : 0;
        const size_t select = select_lds(short_selects_small(K, instance, row));
        if (slots <= (cw == 1 ? short_max_units(m) : short16_max_units(m)) && table16 + select <= kMaxLdsBytes) {
            // (one-byte sub-ids: the general kernel takes the same grid when the measurement hook keeps a call off the
            // short one; two-byte sub-ids: its plan stays as it is)
            const bool forced = (g_force_general.load(std::memory_order_relaxed) & 1) != 0;
            if (cw == 1 || !forced) {
                p.nblk = (int)nb;
                p.copies = 1;
                p.big = false;
            }
            if (cw == 1) {
                p.scan_dyn_lds = scan_lds_bytes(0, p.cap, p.candmax, K, kWaves);
                p.scan_lds = p.scan_dyn_lds + lut_floats * sizeof(float);
            }
            if (!forced) {
                p.short_scan = true;
                p.short_units = (int)slots;
                p.glut = false;
                p.scan_dyn_lds = select + table16;
                p.scan_lds = select + (cw == 1 ? lut_floats * sizeof(float) : table16);
            }
        }
    }
    // Longer catalogues of a single query are scanned in segments, one workgroup per CU.  So are any queries whose tables of two-byte
    // sub-ids fit LDS beside one candidate array but not beside a list per wave: the general kernel looks them up in device memory
    // then, one lane per clock and CU (K = 512: one query, m = 4, b = 8192, 29M items 370 us, in segments 74; m = 8, b = 4096, 64 queries of
    // 300,000 items 521 and 74, 400 of 100,000 1103 and 154; K = 120: m = 16, b = 2048, one query, 8M 274 and 53; 400 of 100,000 2166 and 217).
    p.long_scan = false;
    if (!(without & kNoLong) && !p.short_scan && p.vec && !generic && !p.tiled && (B == 1 || p.glut) &&
        !(g_force_general.load(std::memory_order_relaxed) & 1) &&
        (p.glut || long_scan_pays(N, m, K, cw) || ((g_force_general.load(std::memory_order_relaxed) & 64) && (cw == 2 || m >= 4)))) {
        const size_t table = cw == 1 ? lut_floats * (m <= 8 ? kTableCopies : 1) * sizeof(float) : table16;
        if (table + sizeof(LongSelectLds<kLongThreads>) <= kMaxLdsBytes) {
            const long long per_segment = (long long)kLongThreads * (row <= 16 ? kLongScores * row / 16 : kLongScores);
            p.long_scan = true;
            p.glut = false;
            p.nblk = B == 1 ? kAssumedCUs : (int)blocks_for_many_queries(kAssumedCUs, B, (units + per_segment - 1) / per_segment, lookups);
            p.copies = cw == 1 && m <= 8 ? kTableCopies : 1;
            p.big = true;
            p.scan_dyn_lds = sizeof(LongSelectLds<kLongThreads>) + table16;
            p.scan_lds = sizeof(LongSelectLds<kLongThreads>) + table;
        }
    }
    // Long catalogues of a single query: one-byte bounds first.
    p.bytes = false;
    if (!(without & kNoBytes) && B == 1 && p.vec && !generic && m >= 4 && !(g_force_general.load(std::memory_order_relaxed) & (1 | 64 | 512)) &&
        (bytes_pay(N, m, b, K, cw) || (g_force_general.load(std::memory_order_relaxed) & 1024))) {
        const size_t dyn = scan_lds_bytes(0, p.cap, p.candmax, K, kMaxWaves), tables = bytes_table_bytes(m, b, cw), all = dyn + tables + 2 * kMaxWaves * sizeof(float) + (m > kMaxWaves ? 2 * (m - kMaxWaves) * sizeof(float) : 0);
        if (all + 64 <= kMaxLdsBytes) {
            p.bytes = true;
            p.short_scan = p.long_scan = p.glut = false;
            p.nblk = kAssumedCUs;
            p.copies = 1;
            p.big = true;
            p.scan_dyn_lds = dyn + (cw == 2 ? tables : 0);
            p.scan_lds = all;
        }
    }
    // Candidate lists (the `generic` plans) of rows of 4, 8 or 16 bytes, short enough for a thread to
    // hold its share: every row of a thread is requested at once and the selection comes straight from registers.
    // Same thin grid as the short scan.
    p.short_subset = false;
    p.subset_vecs = 0;
    if (generic && cw == 1 && (m == 4 || m == 8 || m == 16) && !(g_force_general.load(std::memory_order_relaxed) & 1)) {
        long long nb = kAssumedCUs / B;
        if (nb < 1 || (subset_direct_pays(N, m, B) && !(g_force_general.load(std::memory_order_relaxed) & 32))) nb = 1;
        const long long thin = (N + kThreads - 1) / kThreads;              // workgroups if every thread held one candidate
        if (nb > thin) nb = thin;
        const long long per_thread = (N + kThreads * nb - 1) / (kThreads * nb);
        const long long vecs = (per_thread * m + 15) / 16;
        if (vecs <= kSubsetMaxVecs) {
            p.short_subset = true;
            p.subset_vecs = (int)vecs;
            p.nblk = (int)nb;
            p.copies = 1;
            p.big = false;
            p.scan_dyn_lds = select_lds(K <= small_k_max(m));
            p.scan_lds = (size_t)m * kLutStride * sizeof(float) + p.scan_dyn_lds;
        }
    }
    // A few queries over catalogues that fit registers: two queries per workgroup.
    p.pair_scan = false;
    const int forced = g_force_general.load(std::memory_order_relaxed);
    if (!(without & kNoPair) && B >= 2 && m >= 4 && p.vec && !generic && !(forced & 1) &&
        ((forced & 256) || pair_pays(p, N, B, m, K))) {
        const long long pairs = (B + 1) / 2, per = (long long)kThreads * pair_max_units(row);
        const long long least = (units + per - 1) / per, thin = (units + kThreads - 1) / kThreads;
        const size_t lds = pair_table_bytes(m, b, cw) + 2 * sizeof(MidSelectLds<kThreads>);
        if (least <= kAssumedCUs && lds <= kMaxLdsBytes) {
            // as many workgroups as fill the chip once to four times: a workgroup's share takes 5 us beside its lookups, lists 3 us to fold
            long long nb = 0;
            double best_us = 0.0;
            for (int fill = 0; fill <= 4; ++fill) {
                long long c = fill == 0 ? least : (long long)kAssumedCUs * fill / pairs;
                c = c < least ? least : c > thin ? thin : c > kAssumedCUs ? kAssumedCUs : c;
                const double us = (double)((pairs * c + kAssumedCUs - 1) / kAssumedCUs) * (5.0 + lookups / (double)c / kPairLookupsPerUs) + (c > 1 ? 3.0 : 0.0);
                if (nb == 0 || us < best_us) { best_us = us; nb = c; }
            }
            const bool alone = p.short_scan && p.nblk == 1;   // otherwise: one workgroup per query, without lists
            p.pair_scan = B <= kAssumedCUs || nb <= cw || K <= (m <= 16 && B > 2 * kAssumedCUs && nb > 2 ? 16 : 128);
            // More than 512 queries take several rounds of workgroups.  Pairs and without (us): a workgroup each, the last round far from full, m = 8, 17,000 items, K = 150, 600
            // queries 46.5 and 39.0, 900 (full) 47.4 and 51.9; m = 16, 9000, K = 150, 720 37.3 and 27.1; m = 8, 5000, K = 2, 600 9.4 and 8.6; m = 32, 5000, K = 150, 900 45.9 and
            // 36.3, 12,000, 650, K = 100 65.2 and 55.8.  m = 16 from 25 vectors to a thread on, one workgroup to a compute unit, in four rounds: 30,000 items, 800, K = 10 70.7 and
            // 57.1, K = 100 90.6 and 77.1 (22,000, two to a compute unit 42.8 and 46.0)
            const long long held = (units + kThreads * nb - 1) / (kThreads * nb);
            if (B > 2 * kAssumedCUs) {
                if (alone && nb == 1 && last_round_empty(pairs) && (K > 128 || (K <= 10 && N * m < 60000))) p.pair_scan = false;
                if (alone && m == 32 && K > (nb == 1 ? 128 : 64)) p.pair_scan = false;
                if (cw == 1 && m == 16 && held > 24 && pairs * nb > 3 * kAssumedCUs) p.pair_scan = false;
            }
            // Two bytes, more than one round of workgroups, instead of the general kernel: m = 4, 35,673 items, 358 queries, K = 146 49.2 and 34.2; 75,948, 152, K = 135 39.8 and 34.5; m = 8,
            // 25,444, 439, K = 152 56.4 and 38.5; 350,142, 250, K = 196 (nine rounds) 203 and 153, 416,818, 253, K = 292 (eleven) 245 and 200 (136,065, 75, K = 265, two, 39.7 and 41.6);
            // m = 4, 66,572, 426, K = 4 (four) 49.7 and 37.2, 46,702, 483, K = 6 (three) 38.4 and 29.7
            if (cw == 2 && !p.short_scan && !p.long_scan && !p.glut && pairs * nb > kAssumedCUs) {
                if (K > 100 && (K <= 200 || pairs * nb > 4 * kAssumedCUs)) p.pair_scan = false;
                if (m == 4 && K <= 32 && pairs * nb > 2 * kAssumedCUs) p.pair_scan = false;
            }
            // m = 4, instead of the general kernel with one or two workgroups per query, where lists are long (pairs and without, us): K = 130, 250 queries, 33,000 items 29.8 and 18.4, 90,000 54.2
            // and 28.9, 170, 60,000 30.3 and 23.3, 90, 90,000 29.4 and 25.9; K = 100, 250, 43,000 25.5 and 19.5, 430, 60,000 58.4 and 43.5, 340, whose last round is two thirds
            // empty, 43,000 29.5 and 36.9; K = 70, 250, 43,000 20.6 and 18.7, 170, 33,000 (even); K = 182, 158, 68,000 24.1 and 25.7; two bytes: K = 100, 430, 90,000 81.5 and
            // 55.6, K = 40, 430, 43,000 36.4 and 31.8, 340 31.1 and 36.0
            if (m == 4 && p.nblk <= 2 && !p.short_scan && !p.long_scan && !p.glut) {
                const int last = B % kAssumedCUs;
                const bool idle = B > kAssumedCUs && last > 0 && last <= kAssumedCUs * 2 / 5;
                if (p.nblk == 2 ? K > 110 && K <= 150 : K > (B > 200 && B <= kAssumedCUs ? 64 : 80) && !(idle && cw == 1 && N < 50000) && !(K > 150 && B <= 200 && N < 80000)) p.pair_scan = false;
                if (cw == 2 && K > 32 && pairs * nb > 2 * kAssumedCUs && !idle) p.pair_scan = false;
            }
            // ... and of the short one: 29,000, 832, K = 81 52.8 and 43.1, 24,000, 1000, K = 100 44.6 and 39.4, K = 70 36.1 and 37.2; a workgroup each, 15,000, 1016, K = 22 18.7
            // and 17.0, 10,000, 787, K = 2 10.5 and 11.8
            if (m == 4 && p.short_scan && B > 2 * kAssumedCUs && (nb > 1 ? K > 75 : B > 3 * kAssumedCUs && N >= 14000 && K >= 20)) p.pair_scan = false;
            p.pair_scan = p.pair_scan || (forced & 256);
            // (one workgroup to a compute unit: 718 queries of 4500 items, two bytes, m = 16, b = 619 17.1 us without, 19.6)
            if (!(forced & 256) && p.short_scan && 2 * lds > kMaxLdsBytes && last_round_empty(pairs * nb)) p.pair_scan = false;
            // (rows of 4 bytes, lists to fold: 3M items, 5 queries, K = 80 28.4 us without, 31.2)
            if (!(forced & 256) && m == 4 && K > 64 && nb > 128) p.pair_scan = false;
            if (p.pair_scan) {
                p.tiled = p.short_scan = p.long_scan = false;
                p.glut = false;
                p.nblk = (int)nb;
                p.copies = 1;
                p.big = false;
                p.short_units = (int)((units + kThreads * nb - 1) / (kThreads * nb));
                p.scan_dyn_lds = p.scan_lds = lds;
            }
        }
    }
    p.subset_pair = false;
    if (B >= 2 && generic && cw == 1 && (m == 4 || m == 8 || m == 16) && !(forced & 1) && ((forced & 256) || subset_pair_pays(p, N, B, m))) {
        const long long pairs = (B + 1) / 2, per = (long long)kThreads * subset_pair_max(m) * 16 / m;
        const long long least = (N + per - 1) / per, thin = (N + kThreads - 1) / kThreads;
        long long nb = kAssumedCUs / pairs;
        // (twice as many workgroups as compute units where their shares are long: 42,189 candidates, m = 8, 134 queries 37.2 and 30.6 us,
        // 17,825, m = 16, 162 21.6 and 19.6, 24,629, 67 17.9 and 19.0)
        if (N * (m + 8) >= 120000 * (nb < 1 ? 1 : nb)) nb = 2 * kAssumedCUs / pairs;
        nb = nb < least ? least : nb > thin ? thin : nb;
        if (nb < 1) nb = 1;
        if (least <= kAssumedCUs && ((forced & 256) || !last_round_empty(pairs * nb, m == 16 && N >= 16000 && B > 2 * kAssumedCUs ? 12 : 25))) {
            p.subset_pair = true;
            p.short_subset = false;
            p.subset_vecs = (int)(((N + kThreads * nb - 1) / (kThreads * nb) * m + 15) / 16);
            p.nblk = (int)nb;
            p.copies = 1;
            p.big = false;
            p.scan_dyn_lds = p.scan_lds = pair_table_bytes(m, b, 1) + 2 * sizeof(MidSelectLds<kThreads>);
        }
    }
    p.filter = false;
    const bool pair_first = (p.pair_scan || p.subset_pair) && !(forced & (16 | 128)) && ((forced & 256) || pair_beats_bounds(N, B, m, K, p.subset_pair, cw, p.short_units));
    if (!(without & kNoFilter) && !pair_first) {
        ScanPlan f = p;
        plan_filter(f, N, B, m, K, generic, cw, b);
        // (the whole batch's tables at most 32 KB per result and 1 MB: a single result of each query is not worth larger ones)
        const size_t others = f.filter ? (size_t)(B - f.f_batch) * ((size_t)f.f_entries * sizeof(uint16_t) + sizeof(FilterQuery) + kFilterBins * sizeof(uint32_t)) : 0;
        if (f.filter && workspace_bytes(f, B, K) + others <= ((size_t)B * K << 15) + (1u << 20)) p = f;
    }
    p.direct = p.nblk == 1;
    return p;
}

// Tables of counts the workspace holds at most: 1024 queries' at m = 64 or over 32768 two-byte entries, 16384 queries' at m = 8.
// So many fill the chip several times over; a batch larger still takes turns with the same workspace.
constexpr size_t kFilterTableBytes = 64u << 20;

// LDS reads a CU returns per clock when every lane reads at random: of 4-, 8- and 16-byte words.
constexpr double kGather4 = 8.7, kGather8 = 8.5, kGather16 = 5.0;
// ... and of 16-byte words with an eighth of the splits read from device memory (5 reads from LDS for seven splits of eight: 5.7; with its fixed costs a whole
// call at m = 8, 50M items, 40 queries, comes to 5.4, at m = 16, 16M, to 5.1), and by pairs of lanes that read a row of 32 bytes together,
// a quarter of the splits from device memory (7.0 and 6.1).  33 to 48 queries of long scans are two tiles of pairs or three of single lanes
// (us): m = 8, K = 10, 10M 97.9 and 90.4, 50M 372 and 363; m = 16, 2.2M 69.5 and 58.2, 16M 272 and 246.
constexpr double kGather16Far = 5.7, kGatherPairs = 7.4;

// Eight queries to a workgroup instead of sixteen single lanes at m = 8 and 16, an eighth of whose splits comes from device memory: the reads alone
// speak for sixteen, but a workgroup of eight has half to look after and to select for, which is 1 to 3 us of a call and decides where the last of the
// sixteens is hardly half full: 17 to 24 queries, and 33 to 40 over shorter scans.  Calls with sixteen and eight (us): m = 8, 20 queries, 700,000 items, K = 10 22.4 and
// 20.0, 1.3M 24.9 and 23.0, K = 128 36.6 and 34.2, 5M, K = 10 42.5 and 39.1, 7.5M, K = 200 77.9 and 73.9, 20M 145 and 158; 36 queries, 700,000 24.2 and 22.3, 1.3M 28.9 and 27.2, 3.5M 44.5
// and 43.1, K = 40 50.5 and 50.6, 5.2M 64.6 and 67.0, K = 200 87.9 and 99.8; m = 16, 20 queries, 600,000, K = 10 26.2 and 24.5, 3.7M 57.6 and 52.9, 10M, K = 40 122 and 115;
// 36, 250,000, K = 10 24.3 and 22.1, 2.6M, K = 50 71.8 and 71.2, 3.7M, K = 40 91.9 and 90.5, 5.8M, K = 200 (all splits in LDS) 167 and 178.  Long scans for more than 128 results fill
// their lists, sixteen's most: 36, K = 200, m = 8, 14M 179 and 190, 20M 268 and 234, 50M 509 and 483; m = 16, 9M 285 and 229, 20M 464 and 436.
// In costs as below, three eights for two sixteens are 1.01 of these, five for three 1.12, seven for four 1.17.
double half_tiles_within(long long N, int m, int K) { return N <= 4000000 || (K > 128 && N * m >= 130000000) ? 1.15 : 1.02; }

// Whether the workgroups of a query, `each` queries to one, share its floors: few of them, `least` rounds of codes each (see shares() below).
bool few_share(long long N, int B, int row, int each, int least) {
    const long long blocks = kAssumedCUs / ((B + each - 1) / each), rounds = N * row / (16LL * kFilterThreads);
    return blocks > 1 && ((blocks <= 16 && rounds / blocks >= least) || (blocks <= 32 && rounds / blocks >= 32));
}

// Lookups (B * N * m) from which a batch is scanned by upper bounds: the sample, the tables and one launch more (some 12 us
// together) are then paid back; longer rows cost more to prepare, the most at m = 64 with many results.  Two queries fill half a
// word's fields; more than 256 make the sample take turns on the CUs, which costs two-byte sub-ids with their larger tables most.
// Candidate lists gain earlier: the rows are gathered once per sixteen queries, not once per query.
// At four fifths and five fourths of the lines (bench.py --rules; by bounds and without, us): B = 4, K = 10: m = 4 17.8 and 19.2, 19.4 and
// 22.6; m = 8 19.6 and 19.8, 21.7 and 23.8; m = 16 21.6 and 22.6, 26.4 and 33.3; m = 32 (B = 8) 29.4 and 29.8, 32.3 and 44.8; m = 64
// (B = 8) 37.1 and 41.4, 41.6 and 62.0; lists, m = 8: 33.2 and 32.0, 38.9 and 43.7; two bytes, m = 8: 25.8 and 24.2, 28.5 and 30.5.
// The shape that loses most by its line: a list of 68,750, m = 4, B = 64: 23.4 and 30.8, scanned without.
double filter_min_lookups(int m, int K, int B, bool subset, int cw) {
    if (subset) return m <= 8 ? 2.2e7 : 4.5e7;
    double least = m == 4 ? 6.0e7 : m == 8 ? 6.5e7 : m == 16 ? 1.0e8 : m == 32 ? (K <= 64 ? 1.6e8 : 2.1e8) : K <= 64 ? 2.4e8 : K <= 128 ? 3.2e8 : 4.0e8;
    if (B == 2) least *= 1.5;
    if (cw == 2) least *= (m == 16 ? 1.3 : 1.0) * (B > 256 ? 2.5 : 1.0);
    return least;
}
// ... and the items per result: with fewer, a sample that is an eighth of them gives too low a floor, and what passes it is
// scored exactly (from tables in device memory: two-byte sub-ids' are large).  The more queries there are, the less the scans
// side by side leave idle.  (m = 16 with sixteen-bit fields, more than 256 queries: against the batched kernel.)
// Two bytes, m = 16 (by bounds and without, us; 16 bits): 390 queries of 350,000 items, b = 300, K = 200 203 and 472, 580 of 63,000, K = 39 89 and 143; 8 bits, b = 1900:
// 900 of 350,000, K = 200 810 and 1342, 390 668 and 599.
// At four fifths and five fourths of the lines (bench.py --rules; by bounds and without, us): m = 8, B = 64, K = 300: 40.9 and 44.2, 41.1 and
// 54.5; B = 512, K = 100: 81.0 and 60.1, 70.2 and 87.4; K = 200: 196 and 169, 221 and 251; m = 16, B = 512, K = 100: 118 and 159 (it
// could lie lower), 147 and 219; m = 32, B = 64, K = 100: 41.8 and 44.2, 47.4 and 59.9; lists, m = 8, B = 64, K = 300: 43 and 68, 46 and 93
// (likewise); two bytes, m = 8, B = 64, K = 100: 36.3 and 37.1, 40.2 and 47.1.
// The catalogue itself has at least eight items per table entry, 3.5 with long rows (m = 64, 100 queries of 60,000 items, K = 10: 87 ->
// 60 us).
long long filter_min_items_per_result(long long N, int m, int K, int B, bool subset, bool w16, int cw) {
    if (m == 16 && w16 && B > 256) return subset ? 600 : cw == 2 ? 1000 : 2000;
    if (subset) return K > 128 ? 350 : 150;
    if (cw == 2) return m == 16 && B > 512 ? 1000 : 2000;
    if (m >= 32) return N < 5LL * m * kLutStride ? 2000 : 1000;
    // (K > 128, more than 256 queries, with eight queries to a workgroup and shared floors and without bounds: m = 8, 512, 150,000 items, K = 250 94 and
    // 130, 900, 90,000, K = 150 103 and 155; m = 4, 900, 150,000, K = 250 109 and 168; floors not shared: m = 8, 300, 150,000, K = 250 147 and 115, K = 150
    // 78 and 107; m = 4, 512, 187,500, K = 150 99 and 87)
    if (B > 256 && K > 128) return m <= 8 && few_share(N, B, m, 8, 14) ? 600 : m == 8 ? 1000 : 1300;
    // (m = 4 over 512 queries: 1000, 24,000 items, K = 40 63.2 and 37.3, 800, 32,500, K = 58 73 and 62; 33,000, K = 40 42.9 and 62)
    return B <= 256 ? (K > 128 ? 800 : 500) : K > (m == 4 && B > 512 ? 31 : 64) ? 800 : 500;
}

// Lookups (B * N * m) from which a batch is scanned by pairs of lanes (see plan_filter()).
double filter_pair_lookups(int m, int K, int B) {
    return B > 128 && !(m == 8 && B <= 256) ? 5.5e9 : (m == 4 ? 2.0e9 : 1.4e9) * (K > 32 ? 1.5 : 1.0);
}

// Where 16-bit counts lie in LDS beside the bytes (m = 16; eight queries to a workgroup instead of sixteen): where many items are scored
// exactly for each that is streamed, which is so the more queries and results and the fewer items there are.  Calls with sixteen queries and bytes alone (K > 32: or
// 16-bit fields, or by pairs) and with eight and both, as their ratio, at 50,000, 150,000, 350,000, 700,000 and 2M items: 1000 queries, K = 2 1.00 1.05 1.03 0.88
// 0.74, K = 6 1.44 1.22 1.34 1.06 0.82, K = 20 1.89 1.58 1.32 1.16 1.01; 400 queries, K = 2 0.95 0.96 1.03 0.99 0.85, K = 4 1.02 1.04 1.10 1.03 0.83, K = 20 1.23 1.70 1.46 1.29
// 1.07; 220 queries, K = 6 0.94 0.88 1.09 1.00 0.89, K = 20 1.00 1.03 1.09 1.03 0.98; 130 queries, K = 6 1.00 0.98 0.98 1.13 1.05, K = 20 1.00 1.03 1.05 1.08 1.04; 100
// queries, K = 20 1.01 1.03 1.03 0.98 1.08, K = 40 0.99 1.07 1.05 1.05 1.07.  (Many items: sixteen or, by pairs of lanes, 32 queries to a workgroup.)  With few items per
// result, floors that are not shared and lists to fold other kernels are ahead: 400 queries, 60,000 items, K = 60 55 us by pairs of queries, 81 with counts.
bool filter_fine_pays(long long N, int m, int K, int B, bool subset, int cw) {
    if (m != 16 || cw != 1 || subset || K > 256 || K < (B > 700 ? 2 : B >= 400 ? 4 : 5)) return false;
    if (N >= 100000LL * K && (double)B * (double)N * m >= 0.6 * filter_pair_lookups(m, K, B)) return false;
    if (N < 2000LL * K && !few_share(N, B, m, 8, 12)) return false;
    if (B >= 400) return true;
    if (B >= 250) return N >= (K <= 10 ? 140000 : 60000);
    if (K <= 16) return B >= 130 && (double)B * (double)N >= 4.6e7;   // (130 queries, 250,000 items, K = 12: 43.9 without, 49.6 with)
    return N >= 100000 && B >= (K <= 32 ? 130 : 81);
}

// Where single lanes look all splits up in LDS.  m = 8, floors shared: over short shares with many results, which score so much exactly,
// through the L1 too, that an eighth of the lookups comes in its way.  Calls with an eighth through the L1 and with none (rounds of codes of a workgroup; us):
// 330,000 items, 512 queries (20), K = 6 54.5 and 53.3; 400,000, 512 (24) 58.8 and 58.5; 180,000, 1000 (22) 63.8 and 62.7; 700,000, 512 (42), K = 20 90.0 and 91.9;
// 1M, 512 (61), K = 45 122.7 and 126.2; 600,000, 700 (58), K = 5 100.5 and 105.5; 800,000, 1000 (98), K = 70 194.1 and 195.7; 1.28M, 1024 (156), K = 100 290 and 296.
// Floors that are not shared: from 512 queries on (whose shares are short then, and whose samples are by half a workgroup) from 16 results on.  80,000 items, 512 queries, K = 10
// 32.8 and 33.0, K = 16 35.2 and 34.4, K = 30 42.3 and 39.9, K = 100 73.6 and 67.9; 60,000, 2500, K = 30 109.5 and 104.0; 130,000, 4000, K = 100 318.9 and 308.6.  (100,000 items, 400
// queries, K = 100 57.3 and 57.4; 120 queries 28.2 and 29.7.)
bool filter_near_pays(long long rounds, int K, int queries, bool shared) { return (shared || (queries >= 2 * kAssumedCUs && K >= 16)) && (double)rounds < 28.0 + 0.7 * K; }
// m = 16, where such shares have 16-bit counts beside the bytes: many results of a query whose floors are not shared, for the items that there are or for its
// workgroups `nb`, each of which looks for as many.  With an eighth through the L1 and with none (us), 800,000 items, 64 queries, K = 100 58.6 and 57.9, 300,000, 64, K = 20 30.9
// and 30.5, 500,000, 60, K = 10 33.1 and 33.4, 5M, 16, K = 10 45.9 and 48.1; tables that let more pass lose more (2M, 48, K = 100: heavy tails 145 and 131).
// Long shares, as a ratio, 5M, 12M and 20M items: 256 workgroups K = 130 0.99 0.96 0.97, K = 256 1.01 0.98 1.04; 128 K = 130 0.97 0.96 1.00, K = 200 1.02 1.01 1.06; 85 K = 100
// 1.01 1.00 1.01, K = 130 1.04 1.03 1.04, K = 200 1.08 1.10 1.09; 64 K = 100 1.00 0.97 0.97, K = 130 1.04 1.00 1.00, K = 200 1.07 1.06 1.04; 51 K = 64 1.00 0.98 0.96, K = 100 1.08 1.03 1.00.
bool filter_near_pays16(long long N, int K, long long nb) { return N < 30000LL * K || (K >= (nb <= 56 ? 90 : 125) && 5LL * K >= 7 * nb); }

// Whether a batch is scanned by upper bounds (scan_filter.hpp), and how.
size_t workspace_bytes(const ScanPlan& p, int B, int K);
void plan_filter(ScanPlan& p, long long N, int B, int m, int K, bool subset, int cw, int b) {
    const int force = g_force_general.load(std::memory_order_relaxed);
    if (force & 8) return;
    const bool rows = (cw == 1 && !subset) ? (m == 4 || m == 8 || m == 16 || m == 32 || m == 64) : (m == 4 || m == 8 || m == 16);
    if (!rows || N * m * cw < 16) return;
    const long long entries = (long long)m * (cw == 1 ? kLutStride : b);
    // Fields: eight bits, or sixteen, which halve the queries of an LDS read but let hardly anything pass that should not: at m = 64, and
    // with few items per result, where more is scored than the reads save.  Calls of 16 bits and 8 (us): m = 32, K = 20: 48 queries, 300,000
    // items 44.3 and 47.7, 600,000 65.5 and 59.9; 200 queries 125 and 181, 202 and 231; K = 10, 600,000 195 and 170; K = 100, 600,000: 224
    // and 268; m = 16, K = 100: 200 queries, 300,000 items 85 and 132, 600,000 123 and 157, 300 queries, 600,000 196 and 203; 100 queries,
    // 600,000 (8) 74; lists, m = 16, K = 100: 200 queries, 200,000 candidates 94 and 144, 1M 223 and 241; 64 queries, 1M 96 and 90.
    bool w16 = m == 64;
    if (m == 32) w16 = N < (long long)K * (K > 64 ? 10000 : B > 150 ? 40000 : 13000);
    if (m == 16 && cw == 1) w16 = subset ? K > 32 || (B > 256 && N < 20000LL * K) : K > 32 && B > 128 && N < 8000LL * K;
    // Two bytes, m = 16, more than 32 results (23 from 257 queries on, 17 from 601): with eight or four queries of 16 bits, up to a line of items per result, which lies lower where workgroups of 8 bits have no more
    // queries and where there are few queries; with two, for 65 to 256 queries of many results or where no four of 8 bits have room.  Calls of 16 bits and 8 (us): b = 300,
    // 350,000 items: 170 queries, K = 40 86 and 84, K = 100 98 and 122, 390, K = 40 148 and 182, K = 100 171 and 306, 900, K = 40 353 and 285, K = 100 409 and 469; 1M, 390, K = 40
    // 314 and 265, K = 100 336 and 399; 63,000, 600, K = 31 95 and 118, 56,000, 940, K = 19 107 and 142; eight queries of either, 1M, 900, K = 400
    // 1168 and 1324, 550,000, 490, K = 149 278 and 261; four and eight, 2.6M, 250, K = 409 590 and 489; four, b = 1000, 1M, 390, K = 200 588 and 717; 128 queries, 320,000, K = 67 72 and 65; b = 1000
    // (four), 1M, 170, K = 100 273 and 289, 900, K = 100 974 and 1444, 40, K = 100 94 and 77; b = 1900 (two), 1M, 170, K = 200 414 and 520, 390, K = 100 925 and 704, 900, K = 400
    // 2331 and in segments 3648.
    if (m == 16 && cw == 2 && K > (B > 600 ? 17 : B > 256 ? 23 : 32) && 2 * K <= 1024) {
        auto queries = [&](bool wide) {
            for (int w = 4; w >= 1; w >>= 1)
                if (filter_lds_bytes(m, entries / m, w, wide, 1, K <= 64 ? 128 : next_pow2(2 * K)) <= kMaxLdsBytes) return w * (wide ? 2 : 4);
            return 0;
        };
        const int of16 = queries(true), of8 = queries(false);
        const long long line = B <= 128 ? 4000 : of16 == of8 ? (of16 == 8 ? 2800 : 5500) : K > 256 ? 3500 : B > 600 && K < 64 ? 7000 : 10500;
        w16 = !of8 || (N < line * K && (of16 >= 4 || (B > 64 && B <= 256 && K >= 100)));
    }
    const bool fine = filter_fine_pays(N, m, K, B, subset, cw);
    if (fine) w16 = false;
    if (!(force & 16) && (B < 2 || (double)B * (double)N * m < filter_min_lookups(m, K, B, subset, cw) || 2 * N < (m >= 32 ? 7 : 16) * entries ||
                          N < (fine ? (B > 700 ? 1000 : 450) : filter_min_items_per_result(N, m, K, B, subset, w16, cw)) * K))
        return;
    if (filter_prepare_lds_bytes(entries, m) > kMaxLdsBytes) return;
    const int stride = (int)(entries / m);
    const int fields = w16 ? 2 : 4;
    // Keys of a query's list: twice K, 128 at least (64 for K = 12: full lists are tidied so often that half a million items, m = 4, 300 queries
    // take 45 us, with 128 43), but where that does not fit and K is small.
    const int roomy = 2 * K < 128 ? 128 : next_pow2(2 * K);
    int cap = roomy;
    // Words of a lane's table entry, lanes that share an item: what reads least of the LDS's time.
    // Pairs of lanes read a third more per clock, but a workgroup has twice the queries to prepare, to look after and to select for, and reads
    // of device memory come in the way of the exact scores': for long scans of few results, where floors are not shared the longest.
    // Calls by single lanes and by pairs (us; m = 8, K = 10): 32 queries, 3M items 36.4 and 37.8, 8M 62.9 and 57.2, 20M 124 and 99; 64 queries, 1M
    // 31.2 and 34.3, 3M 53.9 and 51.2, 8M 108 and 88; 200, 1M 66 and 62, 8M 298 and 246; 500, 1M 112 and 123, 3M 269 and 260; K = 100:
    // 32 queries, 8M 75 and 75, 20M 144 and 126; 200, 3M 154 and 220.  m = 4: 64 queries, 8M 66 and 64, 20M 126 and 120; 500, 3M 160 and 145.
    // m = 16: 32, 3M 56.5 and 54.6, 8M 111 and 97; 200, 1M 105 and 114.  Lists: m = 4, 500 queries, 200,000 candidates 77 and 64, 1M 178 and 130.
    const bool pairs = subset ? m == 4 && B >= 400 && N >= 150000 : (double)B * (double)N * m >= filter_pair_lookups(m, K, B) && (K <= 32 || B <= 128);
    // Eight queries to a workgroup instead of sixteen: half as many workgroups share a query, and below some number they share its floors, where
    // much is scored exactly and the streaming that doubles is not the most of it.  Calls with sixteen and eight (us): m = 8, K = 200: 130
    // queries, 1M items (floors not shared, shared) 154 and 77, 300,000 (neither) 53 and 65; 300, 300,000 147 and 78; K = 60: 200 queries, 1M
    // 84 and 71, 130, 3M 114 and 107; 300, 500,000 (both shared) 75 and 68, 2M 147 and 166; K = 100, 600, 500,000 125 and 118, 1.28M 227 and 228;
    // m = 4, 130 queries, 3M, K = 100 138 and 88 (with shared floors already 16 are better); two bytes, m = 8, 260 queries, 300,000, K = 20 87 and 75.
    const double scanned = (double)B * (double)N;
    const int row_bytes = m * cw;
    const bool eight = !subset && !w16 && !(force & 128) && (m == 4 || m == 8) && few_share(N, B, row_bytes, 8, 14) && K >= (m == 8 && cw == 2 ? 10 : 50) &&
                       (!few_share(N, B, row_bytes, 16, 12) || (m == 8 && scanned <= (cw == 2 ? 3.5e8 : K > 128 ? 6.0e8 : K >= 90 ? 4.0e8 : 2.2e8)));
    double best_cost = 0.0, rate = 0.0;
    int words = 0, lanes = 1;
    for (int w = 8; w >= (w16 && m == 16 && cw == 1 ? 4 : w16 && m == 32 ? 2 : 1); w >>= 1) {   // (8: four words for each of two lanes)
        const int l = w == 8 ? 2 : 1, each = w == 8 ? 4 : w;
        if (fine && w != 2) continue;
        if (l == 2 && (w16 || (subset && m != 4) || !(pairs || (force & 128)))) continue;
        if ((m >= 32 && l == 2) || (m == 64 && each == 4)) continue;
        const int c = K <= 16 && filter_lds_bytes(m, stride, each, w16, l, roomy, fine) > kMaxLdsBytes ? 64 : roomy;
        if (filter_lds_bytes(m, stride, each, w16, l, c, fine) > kMaxLdsBytes) continue;
        if (w > 2 && eight) continue;
        const long long tiles = (B + w * fields - 1) / (w * fields);
        const double r = l == 2 ? kGatherPairs : each == 4 ? (filter_far_splits(m, 4, w16, 1, subset, cw) > 0 ? kGather16Far : kGather16) : each == 2 ? kGather8 : kGather4;
        const double cost = (double)tiles * l / r;
        const double within = each == 2 && words == 4 && lanes == 1 && m <= 16 && filter_far_splits(m, 4, w16, 1, subset, cw) > 0 ? half_tiles_within(N, m, K) : 1.0;
        if (words == 0 || cost < best_cost * within) { words = each; lanes = l; cap = c; best_cost = cost; rate = r; }
        if (l == 2 && (force & 128)) break;
    }
    if (words == 0) return;
    const int row = m * cw, queries = words * fields * lanes;
    // (lists of m = 8 whose floors are shared have 16-bit counts beside the bytes, see below)
    const bool fine_list = subset && m == 8 && words == 4 && filter_lds_bytes(m, stride, words, w16, lanes, cap, true) <= kMaxLdsBytes;
    const long long together = (long long)(kFilterTableBytes / ((size_t)entries * (fine || fine_list ? 3 : 2))), turns = (B + together - 1) / together;
    const int batch = turns == 1 ? B : (int)std::min<long long>(((B + turns - 1) / turns + 31) & ~31LL, B);
    const long long tiles = (batch + queries - 1) / queries;
    const bool by_vector = row <= 16 && !subset;
    const long long units = by_vector ? N * row / 16 : N;
    const int vecs = row >= 32 ? row / 16 : 1;
    const long long per_round = (long long)kFilterThreads / lanes * (by_vector ? vecs : vecs * 16 / row);
    const long long rounds = (units + per_round - 1) / per_round;
    // Item blocks per tile: one workgroup per CU, or a few one after the other when one filling would leave CUs idle.
    const double stream_us = (double)N * m * lanes / (rate * 2400.0);
    const double gather_us = subset && m == 4 ? (double)N / 2400.0 : 0.0;   // (a row per clock, longer than four lookups take)
    // Workgroups of a query share their floors where they are few and their shares long, a round being a unit of every wave (one word:
    // batches of a few queries, but at m = 64 and with large alphabets, whose tables leave room for no more beside many results: two bytes, m = 4, b = 6000, 140 queries, 1M
    // items, K = 131 141 and 98).  K = 100, not shared and shared (us): m = 4, 200 queries, 8M items 236 and 179; m = 8, 3M 193 and 154; m = 16,
    // 3M 427 (16-bit fields) and 275; K = 3, m = 4, 373 queries, 731,549 items 47.4 and 52.3.
    // More than sixteen update one histogram too often for few results, and at m = 64, where 16-bit fields let little pass, for some more: m = 64, 40
    // queries, 1M items, K = 5 143 and 161, 10 147 and 162, 50 229 (1.5M) and 215; 32, 1.5M, K = 5 159 and 182; 56, 2M, K = 20 367 and 342, 52, 1.5M (77 rounds), K = 9 265 and 256; m = 4, 130,
    // 4M, K = 3 71.3 and 73.5, 200, K = 10 106 and 94; m = 8, 250, 1.5M, K = 1 69 and 79, 3 75 and 80; m = 16, 180, 700,000, K = 1 71 and 78, 220, 700,000, K = 2
    // 83 and 79; m = 32, 180, 1.5M, K = 3 235 and 221.  m = 64, shares of few rounds: 64 queries, 200,000 items (12 rounds), K = 10 69 and 87, K = 100 93
    // and 116, 450,000 (27) 149 and 153; 100, 300,000 (29) 212 and 192.
    // Two bytes, K = 6: m = 8, b = 1500, 60, 2M (61 rounds) 57 and 72, 100, 1M (51) 58 and 67, 2M (102) 84 and 86, 4M (205) 130 and 126; m = 4, b = 4000, 60, 4M (61) 66 and 77;
    // K = 20: 60, 2M 66 and 69, 100, 2M 100 and 92.
    // ... but by five workgroups: 170, 140,000 (27), K = 10 141 and 144, K = 120 292 and 208; 190, 110,000 (21), K = 60 197 and 192.  One word, two bytes: m = 4, b = 6000, 130, 340,000 (24),
    // K = 13 51 and 60, K = 30 72 and 62, 700,000 (49), K = 4 59 and 75, 300 (114), K = 4 119 and 107; by seventeen, m = 8, b = 3000, 60, 700,000, K = 30 62 and 76, K = 60 74 and 75,
    // m = 16, b = 1600, K = 60 107 and 112.
    const bool narrow = cw == 2 && words == 1;
    auto shares = [&](long long blocks) {
        if (blocks <= 1 || blocks > 32 || !(words > 1 || m == 64 || cw == 2)) return false;
        const long long each = rounds / blocks;
        if (blocks > 16) {
            const int few = cw == 2 && each < 110 ? (narrow ? 64 : 12) : m <= 8 ? 4 : m <= 32 ? 1 : each < 60 ? 16 : 8;
            return each >= 32 && K > few;
        }
        return each >= (K <= 4 ? (narrow ? 100 : 30) : m == 64 ? (blocks <= 6 ? 20 : 28) : narrow && K <= 16 ? 28 : 12);
    };
    long long nb = 1;
    double best_us = 0.0;
    for (int fill = 1; fill <= 4; ++fill) {
        long long cand = (long long)kAssumedCUs * fill / tiles;
        if (cand > rounds) cand = rounds;
        if (cand < 1) cand = 1;
        // (rows of a list: with a multiple of 8 blocks, block x of every tile runs on XCD x % 8, whose L2 the tiles share:
        // 200 queries, 1M of 4M items, m = 8, K = 10: 234 us with 19 blocks, 109 with 16)
        if (subset && (cand & 7) * (N >= 150000 ? 2 : 5) <= cand) cand = cand < 8 ? cand : cand & ~7LL;
        // (seventeen to twenty, whose floors are not shared, or sixteen, whose are: many results.  m = 4, two bytes, 110 queries, 1.1M items, K = 250 111 and 79; one byte,
        // 2M, K = 400 163 and 88; fewer results, m = 8, 212, 650,000, K = 30 58 and 65, m = 4, 205, 1.7M, K = 30 64 and 71, m = 16, 98, 260,000, K = 100 51 and 60)
        if (!subset && m <= 16 && K > (m <= 8 ? 128 : 256) && cand > 16 && cand <= 20 && !shares(cand) && shares(16)) cand = 16;
        const double per_cu = (double)((tiles * cand + kAssumedCUs - 1) / kAssumedCUs);
        // (workgroups that share their floors, or scan everything for their queries, score less.  In a list an item that is scored exactly costs its row from
        // another place in memory too, the more items the more results: with and without this term, 1M candidates, 300 queries, m = 8 (8 workgroups per query that share, 24
        // that do not), K = 10 151 and 178 us, K = 100 199 and 331, K = 200 292 and 526; 3M, 305, m = 4, K = 200 666 and 971; m = 16, 180, K = 100 220 and 342)
        const bool alike = cand == 1 || shares(cand);
        const double list_us = subset ? (alike ? 0.15 : 0.75) * K * queries / 16.0 : 0.0;
        const double us = per_cu * ((stream_us + gather_us) / (double)cand * (alike ? 1.0 : 1.2) + 8.0 + list_us);
        if (fill == 1 || us < best_us) { best_us = us; nb = cand; }
    }
    p.filter = true;
    p.tiled = p.short_scan = p.pair_scan = p.short_subset = p.subset_pair = p.long_scan = p.bytes = false;
    p.f_words = words;
    p.f_w16 = w16;
    p.f_queries = queries;
    p.f_cap = cap;
    p.f_entries = entries;
    p.f_batch = batch;
    const int sample_units = (row == 8 || row == 16 || row == 32) ? 2 : 1;
    p.f_prepare = batch >= 2 * kAssumedCUs && 4 * filter_prepare_lds_bytes(entries, m) <= kMaxLdsBytes ? kThreads : kFilterThreads;
    p.f_sample = p.f_prepare * ((subset && row < 16) ? sample_units * 16 / row : sample_units);
    // The sample: n items cost n * m lookups of 4 bytes, and (K / n) of the catalogue then passes the first floor and is
    // scored from device memory, an eighth as fast: least together at about 5 sqrt(K N), for few results of many queries 8 (300 queries,
    // 200,000 items, m = 4, K = 12 41 and 29 us; 478, 115,861, m = 8, K = 11 48 and 42; 300, 300,000, K = 26 52 and 56).  Where the workgroups
    // of a query share their floors those rise fast by themselves.  Over many items 7, since the sample reads runs of memory (calls with 5 and 7, us: 50M, m = 8, 32, K = 10 204.6 and
    // 200.6, 5M, 20 37.9 and 37.6, m = 16, 16 44.5 and 44.0, 13M, m = 4, 24, K = 39 51.8 and 50.6; 1.28M, m = 8, 64 31.3 and 31.9; m = 64, 6M, 8 157.7 and 159.3), but not for up to sixteen queries, whose sixteen parts have a
    // compute unit each, by more rounds of these (8.5M, m = 8, 3, K = 39 30.4 and 31.6, K = 217 41.7 and 43.4; m = 16, 13M, 2, K = 39 56.9 and 59.9, from nine queries on K = 10 8.5M, 16 61.2 and 60.2), nor for many results at m = 16 (2.6M, 40, K = 39 67.4 and 69.0,
    // 8.5M, 24 101.2 and 103.5).
    p.f_share = shares(nb);
    const long long items_per_round = (long long)p.f_sample * N / units;
    const bool few_of_many = K <= 16 && B > 128 && !subset && !p.f_share;
    auto rounds_of = [&](double times) -> long long { return (long long)(times * sqrt((double)K * (double)N)) / items_per_round; };
    long long want = rounds_of(few_of_many ? 8.0 : 5.0);
    if (!few_of_many && !subset && N >= 2500000 && (m < 16 || (m == 16 && K <= 16))) want = B > (m == 16 ? 8 : 16) ? rounds_of(7.0) : std::max(want, std::min<long long>(rounds_of(7.0), 16));
    // (... but at m = 32, where an exact score costs most, not within so short a time, if the catalogue is worth the sample: one round and four, 500,000 items, 480 queries,
    // K = 10 428 and 301, 800,000, 900, K = 20 1169 and 928, K = 30 (16-bit fields) 1139 and 1087; 200,000, 70, K = 100 66 and 80.  m = 16 with bytes alone, one and two: 900,
    // 500,000, K = 5 231 and 212)
    // Many results with shared floors, rounds of 1024 threads: m = 4, four and six, 2M, 300, K = 100 97.4 and 96.3; m = 8, two and three, 1.28M, 1024, K = 100 266.2 and 263.9, 700,000, 512, K = 64
    // 106.8 and 104.8 (four: 262.5 beside 261.3 with three); m = 16, one and three, 1M, 300, K = 100 190.6 and 181.9, 600,000, 600, K = 200 251.6 and 241.1.
    const long long few_rounds = K <= 32 ? (m == 16 && !fine && !w16 && !subset ? 2 : 1) : m == 4 ? 6 : m == 8 || m == 16 ? 3 : 1;
    const long long most_rounds = (nb > 16 ? 4 : m == 32 ? std::min<long long>(4, 1 + N / 170000) : few_rounds) * (kFilterThreads / p.f_prepare);
    if (p.f_share && want > most_rounds) want = most_rounds;
    if (want > N / 8 / items_per_round) want = N / 8 / items_per_round;
    if (want < 1) want = 1;
    long long parts = kAssumedCUs / batch;
    if (parts > 16) parts = 16;
    if (parts > want) parts = want;
    if (parts < 1 || 2 * K + 3 * parts > kFilterBest) parts = 1;
    long long sample_rounds = (want + parts / 2) / parts;
    if (sample_rounds > 8 * (kFilterThreads / p.f_prepare)) sample_rounds = 8 * (kFilterThreads / p.f_prepare);
    p.f_parts = (int)parts;
    p.f_rounds = (int)(sample_rounds < 1 ? 1 : sample_rounds);
    // The sample gives a query up of which more than three in ten items would pass its floor.  Floors that few workgroups share over long shares rise far above
    // the sample's, and the scan finds out by itself (given up at once, 1024 queries of heavy-tailed tables, m = 8, took 1.3 ms instead of 0.5); those of short
    // shares, or of more workgroups, rise less.  An entry that five items have, left to the scan and given up at once (us): m = 64, 60 queries, 3M items, K = 100
    // 4977 and 2272; m = 8, 200, 4M, K = 100 2559 and 988, 300, 500,000, K = 10 919 and 218; m = 4, 500, 300,000, K = 100 841 and 245.  But a sample of few items per
    // result has a floor that lets a part of that through, which bounds of bytes multiply (one round of 1024 at m = 16): 126 ordinary queries given up, 480,000 items,
    // m = 16, K = 500 1860 and 157 left to the scan, 300,000, K = 300 322 and 113, a list of 300,000, K = 500 622 and 146.
    const double sampled = (double)items_per_round * (double)(parts * p.f_rounds);
    p.f_patient = p.f_share && ((nb <= 16 && rounds / nb >= 32) || (double)K * (w16 ? 8.0 : m >= 16 ? 32.0 : 16.0) > sampled);
    // scores a part leaves: twice its share of the K best and two more, never more than K
    long long best = (2 * K + parts - 1) / parts + 2;
    p.f_best = (int)(best < K ? best : K);
    p.f_lanes = lanes;
    p.f_stride = stride;
    p.f_far = filter_far_splits(m, words, w16, lanes, subset, cw);
    p.f_near = p.f_far > 0 && lanes == 1 && (m == 8 ? filter_near_pays(rounds / nb, K, batch, p.f_share) : m == 16 && !p.f_share && filter_near_pays16(N, K, nb));
    if (p.f_near) p.f_far = 0;
    p.f_pitch = align16((size_t)(cw == 1 ? m : m - p.f_far) * stride * (w16 ? sizeof(uint16_t) : sizeof(uint8_t)));
    p.nblk = (int)nb;
    // Lists: what an item costs that passes is its row from another place in memory.  m = 8, floors shared, without 16-bit counts and with (us): 200,000 candidates, 500
    // queries, K = 10 85 and 80, K = 100 133 and 118, 1000, K = 100 222 and 199; 1M, 500, K = 10 210 and 184, K = 100 281 and 253; 200, K = 10 123 and 111.  Not shared:
    // 64, 200,000 28.6 and 35.0, 1M, K = 10 51 and 57.
    p.f_fine = fine || (fine_list && p.f_share);
    p.scan_lds = filter_lds_bytes(m, stride, words, w16, lanes, cap, p.f_fine);
    // (one-byte sub-ids: the tables are a static array)
    p.scan_dyn_lds = p.scan_lds - (cw == 2 ? 0 : filter_table_bytes(m, stride, words, w16, lanes));
}

size_t keys_bytes(const ScanPlan& p, int B, int K) {
    const size_t bytes = (size_t)B * p.nblk * K * sizeof(uint64_t);
    return (bytes + 255) & ~(size_t)255;
}

// workspace: [B][nblk][K] keys from the scan | filter scans, for the f_batch queries scanned together: tables of counts | FilterQuery
// records | histograms | 16-bit counts beside the bytes | the sample's best scores | the rows that stay in device memory
size_t counts_bytes(const ScanPlan& p) { return p.filter ? ((size_t)p.f_batch * p.f_pitch + 255) & ~(size_t)255 : 0; }
size_t far_bytes(const ScanPlan& p) {
    return p.filter ? ((size_t)((p.f_batch + p.f_queries - 1) / p.f_queries) * p.f_far * (size_t)p.f_stride * p.f_queries + 255) & ~(size_t)255 : 0;
}
size_t query_bytes(const ScanPlan& p) { return p.filter ? ((size_t)p.f_batch * sizeof(FilterQuery) + 255) & ~(size_t)255 : 0; }
size_t hist_bytes(const ScanPlan& p) { return p.filter ? (size_t)p.f_batch * kFilterBins * sizeof(uint32_t) : 0; }
size_t fine_bytes(const ScanPlan& p) { return p.filter && p.f_fine ? (size_t)p.f_batch * p.f_entries * sizeof(uint16_t) : 0; }
size_t best_bytes(const ScanPlan& p) { return p.filter && p.f_parts > 1 ? ((size_t)p.f_batch * p.f_parts * p.f_best * sizeof(float) + 255) & ~(size_t)255 : 0; }
size_t workspace_bytes(const ScanPlan& p, int B, int K) {
    return keys_bytes(p, B, K) + counts_bytes(p) + query_bytes(p) + hist_bytes(p) + fine_bytes(p) + best_bytes(p) + far_bytes(p);
}
bool fits_static_scratch(const ScanPlan& p, int B, int K) {
    return workspace_bytes(p, B, K) - far_bytes(p) <= kStaticScratchBytes && far_bytes(p) <= kStaticRowsBytes;   // (the rows come last)
}

// Lists that do not fit `bytes`: up to a quarter fewer item blocks per query, where the kernel takes any grid.  (The scan gets longer
// by that much at most; coarser grids are left to the caller, who can pass a workspace.)
void coarsen_to_fit(ScanPlan& p, int B, int K, size_t bytes) {
    if (p.filter || p.short_scan || p.pair_scan || p.long_scan || workspace_bytes(p, B, K) <= bytes) return;
    const long long most = (long long)(bytes / ((size_t)B * K * sizeof(uint64_t)));
    if (most >= 1 && 4 * most >= 3LL * p.nblk) {
        p.nblk = (int)most;
        p.direct = p.nblk == 1;
    }
}

// pq_score_topk_static()'s plan: what does not fit its scratch is left out, first pairs of queries or bounds, then item blocks.
ScanPlan make_static_plan(long long N, int B, int m, int K) {
    ScanPlan p = make_plan(N, B, m, K);
    for (int without = 0; (p.pair_scan || p.filter) && !fits_static_scratch(p, B, K);) {
        without |= p.pair_scan ? kNoPair : kNoFilter;
        p = make_plan(N, B, m, K, false, 1, kLutStride, without);
    }
    coarsen_to_fit(p, B, K, kStaticScratchBytes);
    return p;
}

int check_topk_shape(long long N, int B, int m, int b, int K, int cw) {
    if (N < 1 || B < 1 || m < 1 || b < 1 || K < 1 || b > (cw == 1 ? 256 : 65536) || K > N || N >= 2147483648LL)
        return PQ_ERR_SHAPE;
    if (K > PQ_MAX_K || m > PQ_MAX_M || B > PQ_MAX_B) return PQ_ERR_UNSUPPORTED;
    return PQ_OK;
}

int check_topk_args(const void* codes, const void* S, long long N, int B, int m, int b, int K, const void* out_ids,
                    const void* out_scores, const void* workspace, size_t workspace_bytes_given, int cw = 1) {
    if (!codes || !S || !out_ids || !out_scores || !workspace) return PQ_ERR_NULL;
    const int rc = check_topk_shape(N, B, m, b, K, cw);
    if (rc != PQ_OK) return rc;
    const ScanPlan p = make_plan(N, B, m, K, false, cw, b);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return PQ_ERR_UNSUPPORTED;
    if (((uintptr_t)codes & 15) || ((uintptr_t)workspace & 15) || ((uintptr_t)S & 3) || ((uintptr_t)out_ids & 3) ||
        ((uintptr_t)out_scores & 3))
        return PQ_ERR_ALIGN;
    if (workspace_bytes_given < workspace_bytes(p, B, K)) return PQ_ERR_WORKSPACE;
    return PQ_OK;
}

constexpr int kMaxDevices = 64;

// Kernels that take more than 64 KB of dynamic LDS need the limit raised, per kernel and device: done the first time a
// kernel asks for that much (and again only if it later asks for more), not on every call.
struct LdsGrant { const void* fn; int dev; size_t bytes; };
hipError_t allow_lds_once(const void* fn, size_t bytes) {
    static std::mutex mu;
    static LdsGrant grants[512];
    static int n_grants = 0;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lock(mu);
    LdsGrant* g = nullptr;
    for (int i = 0; i < n_grants && g == nullptr; ++i)
        if (grants[i].fn == fn && grants[i].dev == dev) g = &grants[i];
    if (g != nullptr && g->bytes >= bytes) return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
    if (g == nullptr && n_grants < 512) g = &grants[n_grants++];
    if (g != nullptr) *g = LdsGrant{fn, dev, bytes};           // (table full: the attribute is simply set again next time)
    return hipSuccess;
}
template <typename KernelT>
hipError_t allow_lds(KernelT kernel, size_t bytes) {
    if (bytes <= 64 * 1024) return hipSuccess;
    return allow_lds_once(reinterpret_cast<const void*>(kernel), bytes);
}

// Enqueue a kernel with its arguments.  (hipLaunchKernelGGL passes the configuration through two more runtime calls and the
// error through a third: 0.15 us of a launch's 3.)
template <typename... P, typename... A>
hipError_t launch(void (*kernel)(P...), dim3 grid, int threads, size_t dyn_lds, hipStream_t st, A... args) {
    std::tuple<P...> values(static_cast<P>(args)...);
    return std::apply([&](P&... v) {
        void* ptrs[] = {const_cast<void*>(static_cast<const void*>(&v))...};
        return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3((unsigned)threads), ptrs, dyn_lds, st);
    }, values);
}

template <int M, int CW = 1>
hipError_t launch_scan(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    if constexpr (CW == 1 && M >= 1 && M <= 8) {
        if (p.copies == kTableCopies) {
            hipError_t e = allow_lds(scan_topk_kernel<M, kTableCopies, kBigThreads>, p.scan_dyn_lds);
            if (e != hipSuccess) return e;
            return launch(scan_topk_kernel<M, kTableCopies, kBigThreads>, dim3(p.nblk, B), kBigThreads, p.scan_dyn_lds, st, a);
        }
    }
    if constexpr (CW == 2) {
        if (p.glut) {
            hipError_t e = allow_lds(scan_topk_kernel<M, 1, kThreads, 2, true>, p.scan_dyn_lds);
            if (e != hipSuccess) return e;
            return launch(scan_topk_kernel<M, 1, kThreads, 2, true>, dim3(p.nblk, B), kThreads, p.scan_dyn_lds, st, a);
        }
    }
    if constexpr (M == 0 || M == 64 || CW == 2) {
        if (p.big) {
            hipError_t e = allow_lds(scan_topk_kernel<M, 1, kBigThreads, CW>, p.scan_dyn_lds);
            if (e != hipSuccess) return e;
            return launch(scan_topk_kernel<M, 1, kBigThreads, CW>, dim3(p.nblk, B), kBigThreads, p.scan_dyn_lds, st, a);
        }
    }
    hipError_t e = allow_lds(scan_topk_kernel<M, 1, kThreads, CW>, p.scan_dyn_lds);
    if (e != hipSuccess) return e;
    return launch(scan_topk_kernel<M, 1, kThreads, CW>, dim3(p.nblk, B), kThreads, p.scan_dyn_lds, st, a);
}

// Where a lean kernel's K best go: the result's ids (and scores), or the workspace's lists (scores: nullptr).
void* out_of(const ScanArgs& a) { return a.out_ids != nullptr ? static_cast<void*>(a.out_ids) : static_cast<void*>(a.ws_keys); }
float* scores_of(const ScanArgs& a) { return a.out_ids != nullptr ? a.out_scores : nullptr; }

template <typename KernelT>
hipError_t launch_short_args(KernelT kernel, const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    return launch(kernel, dim3(p.nblk, B), kThreads, p.scan_dyn_lds, st, a.codes, a.S, out_of(a), scores_of(a), (uint32_t)a.N, a.b, a.K, a.stamps);
}

template <int M, int U>
hipError_t launch_short_units(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    if constexpr (short_has(U, short_held_units(M), short_max_units(M))) {
        if constexpr (M == 8) {
            if (a.stamps != nullptr) {
                return launch_short_args(scan_short_kernel<M, U, kThreads, true>, p, a, B, st);
            }
        }
        return launch_short_args(scan_short_kernel<M, U, kThreads, false>, p, a, B, st);
    } else {
        return hipErrorInvalidValue;                         // (the plan never asks for it)
    }
}
template <int M>
hipError_t launch_short_m(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    switch (short_instance(p.short_units, short_held_units(M))) {
        case 1: return launch_short_units<M, 1>(p, a, B, st);
        case 2: return launch_short_units<M, 2>(p, a, B, st);
        case 3: return launch_short_units<M, 3>(p, a, B, st);
        case 4: return launch_short_units<M, 4>(p, a, B, st);
        case 5: return launch_short_units<M, 5>(p, a, B, st);
        case 6: return launch_short_units<M, 6>(p, a, B, st);
        case 7: return launch_short_units<M, 7>(p, a, B, st);
        case 8: return launch_short_units<M, 8>(p, a, B, st);
        case 9: return launch_short_units<M, 9>(p, a, B, st);
        case 10: return launch_short_units<M, 10>(p, a, B, st);
        case 11: return launch_short_units<M, 11>(p, a, B, st);
        case 12: return launch_short_units<M, 12>(p, a, B, st);
        case 16: return launch_short_units<M, 16>(p, a, B, st);
        case 24: return launch_short_units<M, 24>(p, a, B, st);
        case 32: return launch_short_units<M, 32>(p, a, B, st);
        case 48: return launch_short_units<M, 48>(p, a, B, st);
        default: return hipErrorInvalidValue;
    }
}
hipError_t launch_short(const ScanPlan& p, const ScanArgs& a, int B, int m, hipStream_t st) {
    switch (m) {
        case 1: return launch_short_m<1>(p, a, B, st);
        case 2: return launch_short_m<2>(p, a, B, st);
        case 4: return launch_short_m<4>(p, a, B, st);
        case 8: return launch_short_m<8>(p, a, B, st);
        case 16: return launch_short_m<16>(p, a, B, st);
        case 32: return launch_short_m<32>(p, a, B, st);
        default: return launch_short_m<64>(p, a, B, st);
    }
}

template <int M, int CW, int C>
hipError_t launch_long_m(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    hipError_t e = allow_lds(scan_long_kernel<M, CW, C>, p.scan_dyn_lds);
    if (e != hipSuccess) return e;
    return launch(scan_long_kernel<M, CW, C>, dim3(p.nblk, B), kLongThreads, p.scan_dyn_lds, st, a.codes, a.S, out_of(a), scores_of(a), (uint32_t)a.N, a.b, a.K);
}
hipError_t launch_long(const ScanPlan& p, const ScanArgs& a, int B, int m, int cw, hipStream_t st) {
    if (cw == 2) return m == 4 ? launch_long_m<4, 2, 1>(p, a, B, st) : m == 8 ? launch_long_m<8, 2, 1>(p, a, B, st) : launch_long_m<16, 2, 1>(p, a, B, st);
    switch (m) {
        case 4: return launch_long_m<4, 1, kTableCopies>(p, a, B, st);
        case 8: return launch_long_m<8, 1, kTableCopies>(p, a, B, st);
        case 16: return launch_long_m<16, 1, 1>(p, a, B, st);
        case 32: return launch_long_m<32, 1, 1>(p, a, B, st);
        default: return launch_long_m<64, 1, 1>(p, a, B, st);
    }
}

template <int M, int U>
hipError_t launch_short16_units(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    if constexpr (short_has(U, short16_held_units(M), short16_max_units(M))) {
        hipError_t e = allow_lds(scan_short_kernel<M, U, kThreads, false, 2>, p.scan_dyn_lds);
        if (e != hipSuccess) return e;
        return launch_short_args(scan_short_kernel<M, U, kThreads, false, 2>, p, a, B, st);
    } else {
        return hipErrorInvalidValue;                         // (the plan never asks for it)
    }
}
template <int M>
hipError_t launch_short16_m(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    switch (short_instance(p.short_units, short16_held_units(M))) {
        case 1: return launch_short16_units<M, 1>(p, a, B, st);
        case 2: return launch_short16_units<M, 2>(p, a, B, st);
        case 3: return launch_short16_units<M, 3>(p, a, B, st);
        case 4: return launch_short16_units<M, 4>(p, a, B, st);
        case 5: return launch_short16_units<M, 5>(p, a, B, st);
        case 6: return launch_short16_units<M, 6>(p, a, B, st);
        case 7: return launch_short16_units<M, 7>(p, a, B, st);
        case 8: return launch_short16_units<M, 8>(p, a, B, st);
        case 9: return launch_short16_units<M, 9>(p, a, B, st);
        case 10: return launch_short16_units<M, 10>(p, a, B, st);
        case 11: return launch_short16_units<M, 11>(p, a, B, st);
        case 12: return launch_short16_units<M, 12>(p, a, B, st);
        case 16: return launch_short16_units<M, 16>(p, a, B, st);
        case 24: return launch_short16_units<M, 24>(p, a, B, st);
        case 32: return launch_short16_units<M, 32>(p, a, B, st);
        case 48: return launch_short16_units<M, 48>(p, a, B, st);
        default: return hipErrorInvalidValue;
    }
}

template <int M, int U, int CW>
hipError_t launch_pair_units(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    if constexpr (pair_has(U, M * CW)) {
        hipError_t e = allow_lds(scan_pair_kernel<M, U, kThreads, CW>, p.scan_dyn_lds);
        if (e != hipSuccess) return e;
        return launch(scan_pair_kernel<M, U, kThreads, CW>, dim3(p.nblk, (B + 1) / 2), kThreads, p.scan_dyn_lds, st, a.codes, a.S, out_of(a), scores_of(a), (uint32_t)a.N, a.b, B, a.K);
    } else {
        return hipErrorInvalidValue;                         // (the plan never asks for it)
    }
}
template <int M, int CW>
hipError_t launch_pair_m(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    switch (pair_instance(p.short_units, pair_held_units(M * CW))) {
        case 1: return launch_pair_units<M, 1, CW>(p, a, B, st);
        case 2: return launch_pair_units<M, 2, CW>(p, a, B, st);
        case 3: return launch_pair_units<M, 3, CW>(p, a, B, st);
        case 4: return launch_pair_units<M, 4, CW>(p, a, B, st);
        case 5: return launch_pair_units<M, 5, CW>(p, a, B, st);
        case 6: return launch_pair_units<M, 6, CW>(p, a, B, st);
        case 7: return launch_pair_units<M, 7, CW>(p, a, B, st);
        case 8: return launch_pair_units<M, 8, CW>(p, a, B, st);
        case 12: return launch_pair_units<M, 12, CW>(p, a, B, st);
        case 16: return launch_pair_units<M, 16, CW>(p, a, B, st);
        case 20: return launch_pair_units<M, 20, CW>(p, a, B, st);
        case 24: return launch_pair_units<M, 24, CW>(p, a, B, st);
        case 32: return launch_pair_units<M, 32, CW>(p, a, B, st);
        case 40: return launch_pair_units<M, 40, CW>(p, a, B, st);
        default: return hipErrorInvalidValue;
    }
}
hipError_t launch_pair(const ScanPlan& p, const ScanArgs& a, int B, int m, int cw, hipStream_t st) {
    if (cw == 2) return m == 4 ? launch_pair_m<4, 2>(p, a, B, st) : m == 8 ? launch_pair_m<8, 2>(p, a, B, st) : launch_pair_m<16, 2>(p, a, B, st);
    switch (m) {
        case 4: return launch_pair_m<4, 1>(p, a, B, st);
        case 8: return launch_pair_m<8, 1>(p, a, B, st);
        case 16: return launch_pair_m<16, 1>(p, a, B, st);
        case 32: return launch_pair_m<32, 1>(p, a, B, st);
        default: return launch_pair_m<64, 1>(p, a, B, st);
    }
}

template <int M>
hipError_t launch_subset_m(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    auto go = [&](auto kernel) {
        return launch(kernel, dim3(p.nblk, B), kThreads, p.scan_dyn_lds, st, a.codes, a.subset, a.S, out_of(a), scores_of(a), (uint32_t)a.N, a.n_items, a.b, a.K);
    };
    switch (p.subset_vecs) {
        case 1: return go(scan_subset_kernel<M, 1, kThreads>);
        case 2: return go(scan_subset_kernel<M, 2, kThreads>);
        case 3: return go(scan_subset_kernel<M, 3, kThreads>);
        case 4: return go(scan_subset_kernel<M, 4, kThreads>);
        case 5: return go(scan_subset_kernel<M, 5, kThreads>);
        case 6: return go(scan_subset_kernel<M, 6, kThreads>);
        case 7: return go(scan_subset_kernel<M, 7, kThreads>);
        case 8: return go(scan_subset_kernel<M, 8, kThreads>);
        default: return hipErrorInvalidValue;
    }
}

template <int M, int CW, bool SUB>
hipError_t launch_filter(const ScanPlan& p, const FilterArgs& a, hipStream_t st) {
    const size_t prep_lds = filter_prepare_lds_bytes(a.entries, M);
    hipError_t e = hipSuccess;
    auto prepare = [&](auto kernel) {
        e = allow_lds(kernel, prep_lds);
        if (e == hipSuccess) e = launch(kernel, dim3(p.f_parts, a.B), p.f_prepare, prep_lds, st, a);
    };
    if (p.f_prepare == kThreads) prepare(filter_prepare_kernel<M, CW, SUB, kThreads>);
    else prepare(filter_prepare_kernel<M, CW, SUB, kFilterThreads>);
    if (e != hipSuccess) return e;
    auto go = [&](auto kernel) {
        e = allow_lds(kernel, p.scan_dyn_lds);
        if (e != hipSuccess) return e;
        return launch(kernel, dim3(p.nblk, (a.B + p.f_queries - 1) / p.f_queries), kFilterThreads, p.scan_dyn_lds, st, a);
    };
    if (a.stamps != nullptr) {
        if constexpr ((M == 8 || M == 16) && CW == 1 && !SUB) {
            if (p.f_near) {
                if constexpr (M == 8)
                    if (p.f_share) return go(scan_filter_kernel<8, 1, 4, false, false, 1, true, true, false, true>);
                return go(scan_filter_kernel<M, 1, 4, false, false, 1, false, true, false, true>);
            }
            if (p.f_words == 4 && p.f_lanes == 1 && !p.f_w16)
                return p.f_share ? go(scan_filter_kernel<M, 1, 4, false, false, 1, true, true>) : go(scan_filter_kernel<M, 1, 4, false, false, 1, false, true>);
        }
        if constexpr (M == 8 && CW == 1 && !SUB) {
            if (p.f_words == 4 && p.f_lanes == 2)
                return p.f_share ? go(scan_filter_kernel<8, 1, 4, false, false, 2, true, true>) : go(scan_filter_kernel<8, 1, 4, false, false, 2, false, true>);
        }
        return hipErrorInvalidValue;                         // (pq_measure_step_stamps() has checked)
    }
    if constexpr ((M == 8 || M == 16) && CW == 1 && !SUB) {
        if (p.f_near) {
            if constexpr (M == 8)
                if (p.f_share) return go(scan_filter_kernel<8, 1, 4, false, false, 1, true, false, false, true>);
            return go(scan_filter_kernel<M, 1, 4, false, false, 1, false, false, false, true>);
        }
    }
    if constexpr (M == 16 && CW == 1 && !SUB) {
        if (p.f_fine) return p.f_share ? go(scan_filter_kernel<16, 1, 2, false, false, 1, true, false, true>) : go(scan_filter_kernel<16, 1, 2, false, false, 1, false, false, true>);
    }
    if constexpr (M == 8 && CW == 1 && SUB) {
        if (p.f_fine) return go(scan_filter_kernel<8, 1, 4, false, true, 1, true, false, true>);
    }
    if constexpr ((M == 16 || M == 32) && CW == 1) {
        if (p.f_w16 && p.f_words == 4) return p.f_share ? go(scan_filter_kernel<M, 1, 4, true, SUB, 1, true>) : go(scan_filter_kernel<M, 1, 4, true, SUB, 1, false>);
    }
    if constexpr (M == 16 && CW == 2) {
        if (p.f_w16) {
            switch (p.f_words) {
                case 1: return p.f_share ? go(scan_filter_kernel<16, 2, 1, true, false, 1, true>) : go(scan_filter_kernel<16, 2, 1, true, false, 1, false>);
                case 2: return p.f_share ? go(scan_filter_kernel<16, 2, 2, true, false, 1, true>) : go(scan_filter_kernel<16, 2, 2, true, false, 1, false>);
                default: return p.f_share ? go(scan_filter_kernel<16, 2, 4, true, false, 1, true>) : go(scan_filter_kernel<16, 2, 4, true, false, 1, false>);
            }
        }
    }
    if constexpr (M == 32) {
        if (p.f_w16) return p.f_share ? go(scan_filter_kernel<32, 1, 2, true, false, 1, true>) : go(scan_filter_kernel<32, 1, 2, true, false, 1, false>);
    }
    switch (p.f_words * p.f_lanes) {
        case 1:
            if constexpr (M == 64 || CW == 2)
                if (p.f_share) return go(scan_filter_kernel<M, CW, 1, M == 64, false, 1, true>);
            return go(scan_filter_kernel<M, CW, 1, M == 64, SUB, 1, false>);
        case 2:
            if constexpr (!(SUB && M == 16))
                if (p.f_share) return go(scan_filter_kernel<M, CW, 2, M == 64, SUB, 1, true>);
            return go(scan_filter_kernel<M, CW, 2, M == 64, SUB, 1, false>);
        case 4:
            if constexpr (M < 64) return p.f_share ? go(scan_filter_kernel<M, CW, 4, false, SUB, 1, true>) : go(scan_filter_kernel<M, CW, 4, false, SUB, 1, false>);
            break;
        default:
            if constexpr (M <= 16 && !(SUB && M != 4)) return p.f_share ? go(scan_filter_kernel<M, CW, 4, false, SUB, 2, true>) : go(scan_filter_kernel<M, CW, 4, false, SUB, 2, false>);
    }
    return hipErrorInvalidValue;                             // (the plan never asks for it)
}

hipError_t launch_filter(const ScanPlan& p, const FilterArgs& a, int m, int cw, hipStream_t st) {
    if (a.subset != nullptr) return m == 4 ? launch_filter<4, 1, true>(p, a, st) : m == 8 ? launch_filter<8, 1, true>(p, a, st) : launch_filter<16, 1, true>(p, a, st);
    if (cw == 2) return m == 4 ? launch_filter<4, 2, false>(p, a, st) : m == 8 ? launch_filter<8, 2, false>(p, a, st) : launch_filter<16, 2, false>(p, a, st);
    switch (m) {
        case 4: return launch_filter<4, 1, false>(p, a, st);
        case 8: return launch_filter<8, 1, false>(p, a, st);
        case 16: return launch_filter<16, 1, false>(p, a, st);
        case 32: return launch_filter<32, 1, false>(p, a, st);
        default: return launch_filter<64, 1, false>(p, a, st);
    }
}

template <int M, int U>
hipError_t launch_subset_pair_units(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    if constexpr (subset_pair_has(M, U)) {
        hipError_t e = allow_lds(scan_subset_pair_kernel<M, U, kThreads>, p.scan_dyn_lds);
        if (e != hipSuccess) return e;
        return launch(scan_subset_pair_kernel<M, U, kThreads>, dim3(p.nblk, (B + 1) / 2), kThreads, p.scan_dyn_lds, st, a.codes, a.subset, a.S, out_of(a), scores_of(a), (uint32_t)a.N, a.n_items, a.b, B, a.K);
    } else {
        return hipErrorInvalidValue;                         // (the plan never asks for it)
    }
}
template <int M>
hipError_t launch_subset_pair_m(const ScanPlan& p, const ScanArgs& a, int B, hipStream_t st) {
    switch (subset_pair_instance(p.subset_vecs)) {
        case 1: return launch_subset_pair_units<M, 1>(p, a, B, st);
        case 2: return launch_subset_pair_units<M, 2>(p, a, B, st);
        case 3: return launch_subset_pair_units<M, 3>(p, a, B, st);
        case 4: return launch_subset_pair_units<M, 4>(p, a, B, st);
        case 6: return launch_subset_pair_units<M, 6>(p, a, B, st);
        case 8: return launch_subset_pair_units<M, 8>(p, a, B, st);
        case 12: return launch_subset_pair_units<M, 12>(p, a, B, st);
        case 16: return launch_subset_pair_units<M, 16>(p, a, B, st);
        default: return launch_subset_pair_units<M, 24>(p, a, B, st);
    }
}

// Enqueue the catalogue scan: every workgroup's K best keys land in the workspace.
// `subset` / `n_items`: candidate list (then N is its length and the plan is a generic one) or nullptr / N
// `cw`: bytes per sub-id (2: `codes` holds uint16 values)
// A plan of one item block per query leaves nothing to fold: the scan writes the result.
int enqueue_scan(const ScanPlan& p, const uint8_t* codes, const float* S, long long N, int B, int m, int b, int K,
                 void* workspace, int* out_ids, float* out_scores, hipStream_t st, const int* subset = nullptr, long long n_items = 0, int cw = 1,
                 uint64_t* stamps = nullptr) {
    if (p.filter) {
        unsigned char* ws = static_cast<unsigned char*>(workspace) + keys_bytes(p, B, K);
        FilterArgs f;
        f.codes = codes; f.N = N; f.b = b; f.K = K; f.cap = p.f_cap;
        f.subset = subset; f.n_items = (uint32_t)(subset ? n_items : N);
        f.counts = ws;
        f.query = reinterpret_cast<FilterQuery*>(ws + counts_bytes(p));
        f.entries = p.f_entries;
        f.hist = reinterpret_cast<uint32_t*>(ws + counts_bytes(p) + query_bytes(p));
        f.pitch = (uint32_t)p.f_pitch;
        f.far = ws + counts_bytes(p) + query_bytes(p) + hist_bytes(p) + fine_bytes(p) + best_bytes(p);
        f.far_splits = p.f_far;
        f.tile = p.f_queries;
        f.wide = p.f_w16;
        f.fine = p.f_fine ? reinterpret_cast<uint16_t*>(ws + counts_bytes(p) + query_bytes(p) + hist_bytes(p)) : nullptr;
        f.best = reinterpret_cast<float*>(ws + counts_bytes(p) + query_bytes(p) + hist_bytes(p) + fine_bytes(p));
        f.sample = p.f_sample;
        f.rounds = p.f_rounds;
        f.parts = p.f_parts;
        f.best_per_part = p.f_best;
        f.patient = p.f_patient;
        f.stamps = stamps;
        for (int q0 = 0; q0 < B; q0 += p.f_batch) {          // (once, unless the batch is one of thousands)
            f.B = B - q0 < p.f_batch ? B - q0 : p.f_batch;
            f.S = S + (size_t)q0 * m * b;
            f.ws_keys = static_cast<uint64_t*>(workspace) + (size_t)q0 * p.nblk * K;
            f.out_ids = p.direct ? out_ids + (size_t)q0 * K : nullptr;
            f.out_scores = out_scores + (size_t)q0 * K;
            const hipError_t e = launch_filter(p, f, m, cw, st);
            if (e != hipSuccess) return record_hip(e);
        }
        return PQ_OK;
    }
    ScanArgs a;
    a.codes = codes; a.S = S; a.N = N; a.m = m; a.b = b; a.K = K;
    a.subset = subset; a.n_items = (uint32_t)(subset ? n_items : N);
    a.stamps = stamps;
    a.cap = p.cap; a.candmax = p.candmax;
    // Batched kernel, small K: lists are cut back to their K best once they pass 2K + 8 keys, short enough to rank in
    // one pass; from K = 13 on its shared floors and final filter do better without (K = 16: 53 -> 48 us, K = 28:
    // 63 -> 52 us at batch 24).  The single-query kernel never cuts early: lists are sorted when full, and the shared
    // floor of long scans keeps them from filling (K = 10: 50M items 79.7 -> 77.5 us, m = 4 at batch 64 57 -> 49 us).
    a.prune_at = (p.tiled && K <= 12) ? 2 * K + 8 : 0;
    a.ws_keys = static_cast<uint64_t*>(workspace);
    a.out_ids = p.direct ? out_ids : nullptr; a.out_scores = out_scores;
    hipError_t e;
    if (p.bytes) {
        if (stamps != nullptr && m != 8) return PQ_ERR_UNSUPPORTED;
        auto go = [&](auto kernel) {
            hipError_t err = allow_lds(kernel, p.scan_dyn_lds);
            return err != hipSuccess ? err : launch(kernel, dim3(p.nblk, B), kBytesThreads, p.scan_dyn_lds, st, a);
        };
        if (stamps != nullptr) return record_hip(go(scan_bytes_kernel<8, 1, true>));
        if (cw == 2) return record_hip(m == 4 ? go(scan_bytes_kernel<4, 2>) : m == 8 ? go(scan_bytes_kernel<8, 2>) : go(scan_bytes_kernel<16, 2>));
        switch (m) {
            case 4: return record_hip(go(scan_bytes_kernel<4>));
            case 8: return record_hip(go(scan_bytes_kernel<8>));
            case 16: return record_hip(go(scan_bytes_kernel<16>));
            case 32: return record_hip(go(scan_bytes_kernel<32>));
            default: return record_hip(go(scan_bytes_kernel<64>));
        }
    }
    if (p.short_scan && cw == 2) {
        if (stamps != nullptr) return PQ_ERR_UNSUPPORTED;
        return record_hip(m == 4 ? launch_short16_m<4>(p, a, B, st) : m == 8 ? launch_short16_m<8>(p, a, B, st) : launch_short16_m<16>(p, a, B, st));
    }
    if (p.short_scan) {
        if (stamps != nullptr && m != 8) return PQ_ERR_UNSUPPORTED;
        return record_hip(launch_short(p, a, B, m, st));
    }
    if (p.pair_scan) {
        if (stamps != nullptr) return PQ_ERR_UNSUPPORTED;
        return record_hip(launch_pair(p, a, B, m, cw, st));
    }
    if (p.long_scan) {
        if (stamps != nullptr) return PQ_ERR_UNSUPPORTED;
        return record_hip(launch_long(p, a, B, m, cw, st));
    }
    if (p.subset_pair) {
        if (subset == nullptr || stamps != nullptr) return PQ_ERR_UNSUPPORTED;   // (the plan is only made for candidate lists)
        return record_hip(m == 4 ? launch_subset_pair_m<4>(p, a, B, st) : m == 8 ? launch_subset_pair_m<8>(p, a, B, st) : launch_subset_pair_m<16>(p, a, B, st));
    }
    if (p.short_subset) {
        if (subset == nullptr || stamps != nullptr) return PQ_ERR_UNSUPPORTED;   // (the plan is only made for candidate lists)
        return record_hip(m == 4 ? launch_subset_m<4>(p, a, B, st) : m == 8 ? launch_subset_m<8>(p, a, B, st) : launch_subset_m<16>(p, a, B, st));
    }
    if (p.tiled) {
        const dim3 grid(p.nblk, (B + kQ - 1) / kQ);
        auto launch_tiled = [&](auto kernel) {
            hipError_t err = allow_lds(kernel, p.scan_dyn_lds);
            if (err == hipSuccess) {
                hipLaunchKernelGGL(kernel, grid, dim3(kThreads), p.scan_dyn_lds, st, a, B);
                err = hipGetLastError();
            }
            return err;
        };
        if (stamps != nullptr) e = m == 8 ? launch_tiled(scan_topk_tiled_kernel<8, true>) : launch_tiled(scan_topk_tiled_kernel<16, true>);
        else e = m == 8 ? launch_tiled(scan_topk_tiled_kernel<8, false>) : launch_tiled(scan_topk_tiled_kernel<16, false>);
        return record_hip(e);
    }
    if (stamps != nullptr) {
        // single-query scans: measurement instances exist for m = 8 only
        if (cw != 1 || !p.vec || m != 8 || p.big != (p.copies == kTableCopies)) return PQ_ERR_UNSUPPORTED;
        if (p.copies == kTableCopies) {
            e = allow_lds(scan_topk_kernel<8, kTableCopies, kBigThreads, 1, false, true>, p.scan_dyn_lds);
            if (e == hipSuccess)
                hipLaunchKernelGGL((scan_topk_kernel<8, kTableCopies, kBigThreads, 1, false, true>), dim3(p.nblk, B),
                                   dim3(kBigThreads), p.scan_dyn_lds, st, a);
        } else {
            e = allow_lds(scan_topk_kernel<8, 1, kThreads, 1, false, true>, p.scan_dyn_lds);
            if (e == hipSuccess)
                hipLaunchKernelGGL((scan_topk_kernel<8, 1, kThreads, 1, false, true>), dim3(p.nblk, B), dim3(kThreads),
                                   p.scan_dyn_lds, st, a);
        }
        return record_hip(e == hipSuccess ? hipGetLastError() : e);
    }
    if (cw == 2) {
        switch (p.vec ? m : 0) {
            case 4: e = launch_scan<4, 2>(p, a, B, st); break;
            case 8: e = launch_scan<8, 2>(p, a, B, st); break;
            case 16: e = launch_scan<16, 2>(p, a, B, st); break;
            default: e = launch_scan<0, 2>(p, a, B, st); break;
        }
        return record_hip(e);
    }
    switch (p.vec ? m : 0) {
        case 1: e = launch_scan<1>(p, a, B, st); break;
        case 2: e = launch_scan<2>(p, a, B, st); break;
        case 4: e = launch_scan<4>(p, a, B, st); break;
        case 8: e = launch_scan<8>(p, a, B, st); break;
        case 16: e = launch_scan<16>(p, a, B, st); break;
        case 32: e = launch_scan<32>(p, a, B, st); break;
        case 64: e = launch_scan<64>(p, a, B, st); break;
        default: e = launch_scan<0>(p, a, B, st); break;
    }
    return record_hip(e);
}

// Which fold takes `nlists` lists of K keys.  fold_small_kernel's waves let K keys or more pass each, which it ranks by counting:
// right for few of them; fold_lists_kernel lets 1.3 K pass.  Steps without Eq. 4 (us; fold_small and fold_lists), one user,
// 256 lists: K = 5 8.5 and 8.8, 10 8.9 and 9.3, 11 9.5 and 9.2, 12 10.1 and 9.5, 13 10.1 and 9.1, 16 18.2 and 9.3, 24 16.0 and 9.8;
// 128 lists, two users: K = 12 12.4 and 12.3, 16 15.6 and 11.6; 20 lists: K = 13 6.5 and 6.6, 16 6.6 and 6.6, 20 7.1 and 6.7, 31 9.4
// and 7.3; 34 lists: K = 13 6.6 and 6.9, 16 7.2 and 6.9; 13 lists of 31, 300 users: 107.8 and 108.2; 4 lists of 30, 64 users: 12.8 and 13.4.
bool fold_small_pays(int nlists, int K) {
    const long long keys = (long long)nlists * K;
    return keys <= (K <= 10 ? kThreads * kFoldSmallRegsMax : K <= 12 ? 2048 : K < kRegisterSelectMinK ? 448 : 0);
}

// Enqueue the fold of the workspace's lists into the outputs.
int enqueue_fold(const ScanPlan& p, int B, int K, void* workspace, int* out_ids, float* out_scores, hipStream_t st,
                 uint64_t* stamps = nullptr) {
    const int nlists = p.nblk;
    if (p.direct) return PQ_OK;               // (the scan has written the result)
    FoldArgs f;
    f.ws_keys = static_cast<const uint64_t*>(workspace);
    f.nlists = nlists; f.K = K;
    f.chunk = f.depth = f.need = f.groups = f.group_mask = 0;
    f.out_ids = out_ids; f.out_scores = out_scores;
    f.stamps = stamps;
    if (fold_small_pays(nlists, K) && !(g_force_general.load(std::memory_order_relaxed) & 2)) {
        const bool few = (long long)nlists * K <= (long long)kThreads * kFoldSmallRegs;
        auto go = [&](auto kernel) {
            return record_hip(launch(kernel, dim3(1, B), kThreads, 0, st, f.ws_keys, out_ids, out_scores, nlists, K, stamps));
        };
        if (stamps != nullptr) return few ? go(fold_small_kernel<kThreads, kFoldSmallRegs, true>) : go(fold_small_kernel<kThreads, kFoldSmallRegsMax, true>);
        return few ? go(fold_small_kernel<kThreads, kFoldSmallRegs, false>) : go(fold_small_kernel<kThreads, kFoldSmallRegsMax, false>);
    }
    // (see fold_lists_kernel: a chunk holds what a list has of the K best in all but one case of thousands, when they are
    // spread at random: reading on is another round trip; and the depth at which at most 60 % of the lists have to reach the floor)
    const double share = (double)K / nlists, most = share + 3.5 * sqrt(share) + 2.0;
    f.chunk = 4;
    while (f.chunk < K && f.chunk < most && 2LL * f.chunk * nlists <= kFoldSlots) f.chunk *= 2;
    f.depth = 1;
    while (f.depth < f.chunk && f.depth < K && 10LL * ((K + f.depth - 1) / f.depth) > 6LL * nlists) ++f.depth;
    f.need = (K + f.depth - 1) / f.depth;
    // (groups: at least four times as many as have to reach the floor, so that 15 % more keys at most pass it)
    f.groups = 64;
    while (f.groups < 4 * f.need) f.groups *= 2;
    f.group_mask = f.groups - 1;
    if (f.groups >= nlists) {
        f.groups = (nlists + 15) & ~15;
        f.group_mask = kFoldLists - 1;
    }
    if (nlists > kFoldLists || (long long)nlists * f.chunk > kFoldSlots) return PQ_ERR_UNSUPPORTED;   // (no plan makes that many)
    if (stamps != nullptr && B > kAssumedCUs)
        return record_hip(launch(fold_lists_kernel<kFoldThreadsMany, true>, dim3(1, B), kFoldThreadsMany, p.fold_lds, st, f));
    if (stamps != nullptr) return record_hip(launch(fold_lists_kernel<kFoldThreads, true>, dim3(1, B), kFoldThreads, p.fold_lds, st, f));
    if (B <= kAssumedCUs) return record_hip(launch(fold_lists_kernel<kFoldThreads>, dim3(1, B), kFoldThreads, p.fold_lds, st, f));
    return record_hip(launch(fold_lists_kernel<kFoldThreadsMany>, dim3(1, B), kFoldThreadsMany, p.fold_lds, st, f));
}

// Batch from which Eq. 4 runs on the matrix cores.  The scalar kernels are faster below: a wave's chain of d/m matrix
// instructions takes as long for one tile of 32 queries as for a GPU full of them.  Scalar kernels and matrix cores (us): d = 512, m = 8, b = 256 256
// queries 3.97 and 5.10, 400 5.21 and 5.20, 448 5.32 and 5.25, 640 6.25 and 5.47, 1024 8.69 and 5.98, 4096 27.7 and 19.9; m = 16 320 4.29 and 4.32, 448 5.20
// and 4.62.  The line is one for all: with more sub-ids it could lie lower (b = 1024 200 7.59 and 5.71), with shorter chunks higher (d = 256 448 3.74 and 4.10, 640
// 4.32 and 4.32; d = 128 448 2.88 and 3.63, 1024 4.30 and 4.26).
constexpr int kSubMfmaMinBatch = 448;
constexpr int kDefaultMfmaMinBatch = 3;    // default scoring: batch from which one matrix-core pass over W beats B mat-vec passes

// Eq. 4 on the matrix cores when the shape allows: rows 16-byte aligned, d/m a multiple of 16.  `ldS`: floats from one
// query's row of S to the next.
bool launch_subitem_mfma(const float* queries, const float* centroids, float* S, int B, int d, int m, long long b, long long ldS,
                         hipStream_t st) {
    const int s = d / m;
    if (s % 16 != 0 || d % 4 != 0 || ((((uintptr_t)queries | (uintptr_t)centroids)) & 15) != 0) return false;
    const long long jtiles = (b + 63) / 64;
    if (m * jtiles > 2147483647LL) return false;
    const dim3 grid((unsigned)(m * jtiles), (B + kSubMfmaQueries - 1) / kSubMfmaQueries);
    if (s % 64 == 0) hipLaunchKernelGGL(subitem_scores_mfma_kernel<64>, grid, dim3(kSubMfmaThreads), 0, st, queries, centroids, S, B, d, m, (int)b, ldS);
    else if (s % 32 == 0) hipLaunchKernelGGL(subitem_scores_mfma_kernel<32>, grid, dim3(kSubMfmaThreads), 0, st, queries, centroids, S, B, d, m, (int)b, ldS);
    else hipLaunchKernelGGL(subitem_scores_mfma_kernel<16>, grid, dim3(kSubMfmaThreads), 0, st, queries, centroids, S, B, d, m, (int)b, ldS);
    return true;
}

constexpr int kSubBatchMin = 3;            // batch from which the interleaved kernel beats one query after the other

template <int S_ELEMS>
hipError_t launch_subitem(const float* queries, const float* centroids, float* S, int B, int d, int m, int b, hipStream_t st) {
    const bool rows_aligned = (((uintptr_t)queries | (uintptr_t)centroids) & 15) == 0 && d % 4 == 0 && (d / m) % 4 == 0;
    if constexpr (S_ELEMS % 4 == 0 && S_ELEMS > 0) {
        if (B >= kSubBatchMin && rows_aligned) {
            // One or two chains to a wave while that leaves a workgroup at most to a compute unit: four make each wave's time in LDS longer, and one
            // workgroup's chunks are fewer to read.  Calls with four chains and with what this takes (d = 512, b = 256, us): m = 8, 16 queries 3.16 and
            // 2.43, 32 3.17 and 2.49, 64 (two) 3.26 and 2.81; m = 16, 16 2.41 and 2.30; m = 4, 60 4.88 and 3.33.
            const long long blocks = (long long)m * ((b + kSubThreads - 1) / kSubThreads);
            auto fits = [&](int each) { return blocks * ((B + kSubBatchWaves * each - 1) / (kSubBatchWaves * each)) <= kAssumedCUs; };
            auto go = [&](auto each) {
                constexpr int I = decltype(each)::value;
                const dim3 grid((unsigned)blocks, (B + kSubBatchWaves * I - 1) / (kSubBatchWaves * I));
                return launch(subitem_scores_batched_kernel<S_ELEMS, I>, grid, kSubBatchThreads, 0, st, queries, centroids, S, B, d, m, b);
            };
            if (B <= kSubBatchWaves || fits(1)) return go(std::integral_constant<int, 1>());
            if (B <= 2 * kSubBatchWaves || fits(2)) return go(std::integral_constant<int, 2>());
            return go(std::integral_constant<int, kSubInterleave>());
        }
    }
    if constexpr (S_ELEMS == 0) {
        if (rows_aligned) {
            dim3 grid(m * ((b + kSubThreads - 1) / kSubThreads), (B + kSubAnyTile - 1) / kSubAnyTile);
            return launch(subitem_scores_any_kernel<kSubAnyTile>, grid, kSubThreads, 0, st, queries, centroids, S, B, d, m, b);
        }
    }
    dim3 grid((m * b + kSubThreads - 1) / kSubThreads, (B + kSubQueryTile - 1) / kSubQueryTile);
    if constexpr (S_ELEMS != 0 && S_ELEMS % 4 == 0 && S_ELEMS <= 128) {
        // whole waves of 16-byte aligned rows: the wave reads its block of sub-item embeddings piece after piece
        if (((long long)m * b) % kSubThreads == 0 && ((uintptr_t)centroids & 15) == 0) {
            return launch(subitem_scores_kernel<S_ELEMS, false, true>, grid, kSubThreads, 0, st, queries, centroids, S, B, d, m, b, nullptr);
        }
    }
    return launch(subitem_scores_kernel<S_ELEMS>, grid, kSubThreads, 0, st, queries, centroids, S, B, d, m, b, nullptr);
}

// ---- the built-in scratch of pq_score_topk_static(): one array per GPU, held until the process ends
// Device address of `scratch` on the current device.  In host code the array's name is only a handle for
// hipGetSymbolAddress(): every GPU holds its own copy at its own address, looked up once per device and kept.
int static_scratch(void** out) {
    static void* ptr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return record_hip(e);
    if (dev < 0 || dev >= kMaxDevices) return PQ_ERR_UNSUPPORTED;
    void* p = __atomic_load_n(&ptr[dev], __ATOMIC_ACQUIRE);
    if (p == nullptr) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));      // (the same answer from every thread that races here)
        if (e != hipSuccess) return record_hip(e);
        if (p == nullptr) return PQ_ERR_HIP;
        __atomic_store_n(&ptr[dev], p, __ATOMIC_RELEASE);
    }
    *out = p;
    return PQ_OK;
}

}  // namespace

extern "C" {

int pq_subitem_scores(const float* queries, const float* centroids, float* S, int B, int d, int m, int b,
                      void* stream) {
    if (!queries || !centroids || !S) return PQ_ERR_NULL;
    if (B < 1 || d < 1 || m < 1 || b < 1 || b > 65536 || d % m != 0) return PQ_ERR_SHAPE;
    if (B > PQ_MAX_B || m > PQ_MAX_M) return PQ_ERR_UNSUPPORTED;
    if (((uintptr_t)queries & 3) || ((uintptr_t)centroids & 3) || ((uintptr_t)S & 3)) return PQ_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (B >= kSubMfmaMinBatch && !(g_force_general.load(std::memory_order_relaxed) & 4) &&
        launch_subitem_mfma(queries, centroids, S, B, d, m, b, (long long)m * b, st))
        return record_hip(hipGetLastError());
    switch (d / m) {
        case 4: return record_hip(launch_subitem<4>(queries, centroids, S, B, d, m, b, st));
        case 8: return record_hip(launch_subitem<8>(queries, centroids, S, B, d, m, b, st));
        case 16: return record_hip(launch_subitem<16>(queries, centroids, S, B, d, m, b, st));
        case 32: return record_hip(launch_subitem<32>(queries, centroids, S, B, d, m, b, st));
        case 64: return record_hip(launch_subitem<64>(queries, centroids, S, B, d, m, b, st));
        case 128: return record_hip(launch_subitem<128>(queries, centroids, S, B, d, m, b, st));
        default: return record_hip(launch_subitem<0>(queries, centroids, S, B, d, m, b, st));
    }
}

size_t pq_score_topk_workspace_bytes(long long N, int B, int m, int b, int K) {
    if (check_topk_shape(N, B, m, b, K, 1) != PQ_OK) return 0;
    const ScanPlan p = make_plan(N, B, m, K);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return 0;
    return workspace_bytes(p, B, K);
}

int pq_score_topk(const uint8_t* codes, const float* S, long long N, int B, int m, int b, int K, int* out_ids,
                  float* out_scores, void* workspace, size_t workspace_bytes_given, void* stream) {
    int rc = check_topk_args(codes, S, N, B, m, b, K, out_ids, out_scores, workspace, workspace_bytes_given);
    if (rc != PQ_OK) return rc;
    const ScanPlan p = make_plan(N, B, m, K);
    hipStream_t st = static_cast<hipStream_t>(stream);
    rc = enqueue_scan(p, codes, S, N, B, m, b, K, workspace, out_ids, out_scores, st);
    if (rc != PQ_OK) return rc;
    return enqueue_fold(p, B, K, workspace, out_ids, out_scores, st);
}

int pq_score_topk_static(const uint8_t* codes, const float* S, long long N, int B, int m, int b, int K, int* out_ids,
                         float* out_scores, void* stream) {
    if (!codes || !S || !out_ids || !out_scores) return PQ_ERR_NULL;
    int rc = check_topk_shape(N, B, m, b, K, 1);
    if (rc != PQ_OK) return rc;
    const ScanPlan p = make_static_plan(N, B, m, K);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return PQ_ERR_UNSUPPORTED;
    if (((uintptr_t)codes & 15) || ((uintptr_t)S & 3) || ((uintptr_t)out_ids & 3) || ((uintptr_t)out_scores & 3))
        return PQ_ERR_ALIGN;
    if (!fits_static_scratch(p, B, K)) return PQ_ERR_TOO_LARGE;
    void* ws = nullptr;
    rc = static_scratch(&ws);
    if (rc != PQ_OK) return rc;
    hipStream_t st = static_cast<hipStream_t>(stream);
    rc = enqueue_scan(p, codes, S, N, B, m, b, K, ws, out_ids, out_scores, st);
    if (rc != PQ_OK) return rc;
    return enqueue_fold(p, B, K, ws, out_ids, out_scores, st);
}

}  // extern "C"

namespace {
// scan launches of a pq_score_topk / pq_score_topk_u16 call timed between two events (one untimed launch first)
int profile_scan(const uint8_t* codes, const float* S, long long N, int B, int m, int b, int K, int* out_ids,
                 float* out_scores, void* workspace, size_t workspace_bytes_given, void* stream, int iters,
                 float* scan_ms, int cw) {
    if (!scan_ms) return PQ_ERR_NULL;
    int rc = check_topk_args(codes, S, N, B, m, b, K, out_ids, out_scores, workspace, workspace_bytes_given, cw);
    if (rc != PQ_OK) return rc;
    if (iters < 1) return PQ_ERR_SHAPE;
    const ScanPlan p = make_plan(N, B, m, K, false, cw, b);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    hipError_t e = hipEventCreate(&ev0);
    if (e != hipSuccess) return record_hip(e);
    e = hipEventCreate(&ev1);
    if (e != hipSuccess) { (void)hipEventDestroy(ev0); return record_hip(e); }
    auto scan = [&]() { return enqueue_scan(p, codes, S, N, B, m, b, K, workspace, out_ids, out_scores, st, nullptr, 0, cw); };
    rc = scan();                                                            // untimed warm-up launch
    if (rc == PQ_OK) rc = record_hip(hipEventRecord(ev0, st));
    for (int it = 0; it < iters && rc == PQ_OK; ++it) rc = scan();
    if (rc == PQ_OK) rc = record_hip(hipEventRecord(ev1, st));
    if (rc == PQ_OK) rc = enqueue_fold(p, B, K, workspace, out_ids, out_scores, st);
    if (rc == PQ_OK) rc = record_hip(hipStreamSynchronize(st));
    float ms = 0.0f;
    if (rc == PQ_OK) rc = record_hip(hipEventElapsedTime(&ms, ev0, ev1));
    (void)hipEventDestroy(ev0);
    (void)hipEventDestroy(ev1);
    if (rc == PQ_OK) *scan_ms = ms / (float)iters;
    return rc;
}
}  // namespace

extern "C" {

int pq_score_topk_profile(const uint8_t* codes, const float* S, long long N, int B, int m, int b, int K,
                          int* out_ids, float* out_scores, void* workspace, size_t workspace_bytes_given,
                          void* stream, int iters, float* scan_ms) {
    return profile_scan(codes, S, N, B, m, b, K, out_ids, out_scores, workspace, workspace_bytes_given, stream, iters,
                        scan_ms, 1);
}

int pq_measure_force_general(int mask) {
    return g_force_general.exchange(mask & 2047, std::memory_order_relaxed);
}

int pq_measure_plan(long long N, int B, int m, int b, int K, int kind, int* plan) {
    if (!plan) return PQ_ERR_NULL;
    if (kind < PQ_PLAN_BYTES || kind > PQ_PLAN_STATIC) return PQ_ERR_SHAPE;
    const int cw = kind == PQ_PLAN_WIDE ? 2 : 1;
    const int rc = check_topk_shape(N, B, m, b, K, cw);
    if (rc != PQ_OK) return rc;
    const ScanPlan p = kind == PQ_PLAN_LIST ? make_plan(N, B, m, K, true) : kind == PQ_PLAN_WIDE ? make_plan(N, B, m, K, false, 2, b)
                       : kind == PQ_PLAN_STATIC ? make_static_plan(N, B, m, K) : make_plan(N, B, m, K);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return PQ_ERR_UNSUPPORTED;
    if (kind == PQ_PLAN_STATIC && !fits_static_scratch(p, B, K)) return PQ_ERR_TOO_LARGE;
    for (int i = 0; i < PQ_PLAN_FIELDS; ++i) plan[i] = 0;
    plan[PQ_PLAN_KERNEL] = p.filter ? PQ_KERNEL_BOUNDS : p.pair_scan ? PQ_KERNEL_PAIRS : p.tiled ? PQ_KERNEL_BATCHED : p.short_scan ? PQ_KERNEL_SHORT : p.long_scan ? PQ_KERNEL_LONG
                           : p.short_subset ? PQ_KERNEL_SHORT_LIST : p.subset_pair ? PQ_KERNEL_LIST_PAIRS : PQ_KERNEL_GENERAL;
    plan[PQ_PLAN_GROUPS] = p.nblk;
    plan[PQ_PLAN_QUERIES] = p.filter ? p.f_queries : p.tiled ? kQ : p.pair_scan || p.subset_pair ? 2 : 1;
    if (p.bytes) plan[PQ_PLAN_FIELD_BITS] = 8;
    if (p.filter) {
        plan[PQ_PLAN_FIELD_BITS] = p.f_w16 ? 16 : 8;
        plan[PQ_PLAN_FINE] = p.f_fine;
        plan[PQ_PLAN_SHARED] = p.f_share;
        plan[PQ_PLAN_PARTS] = p.f_parts;
        plan[PQ_PLAN_ROUNDS] = p.f_rounds;
        plan[PQ_PLAN_FAR] = p.f_far;
    }
    return PQ_OK;
}

int pq_measure_step_stamps(const float* queries, const float* centroids, const uint8_t* codes, long long N, int B,
                           int d, int m, int b, int K, float* S, int* out_ids, float* out_scores, void* workspace,
                           size_t workspace_bytes_given, uint64_t* stamps, size_t stamps_bytes, int* scan_grid,
                           void* stream) {
    if (!queries || !centroids || !S || !stamps) return PQ_ERR_NULL;
    int rc = check_topk_args(codes, S, N, B, m, b, K, out_ids, out_scores, workspace, workspace_bytes_given);
    if (rc != PQ_OK) return rc;
    if (d < 1 || d % m != 0) return PQ_ERR_SHAPE;
    if (((uintptr_t)queries & 3) || ((uintptr_t)centroids & 3) || ((uintptr_t)stamps & 7)) return PQ_ERR_ALIGN;
    if (stamps_bytes < PQ_STAMP_BYTES) return PQ_ERR_WORKSPACE;
    static_assert(PQ_STAMP_SLOTS == kStampSlots, "header and kernels agree on the record size");
    // (the scan in segments has no measurement instance, that by upper bounds those of the named workloads: otherwise the kernels
    // that would run without them)
    ScanPlan p = make_plan(N, B, m, K, false, 1, kLutStride, kNoLong | kNoPair | (m == 8 ? 0 : kNoBytes));
    if (p.filter && (p.f_w16 || p.f_fine || p.f_words != 4 || !(m == 8 || (m == 16 && p.f_lanes == 1))))
        p = make_plan(N, B, m, K, false, 1, kLutStride, kNoLong | kNoPair | kNoFilter | kNoBytes);
    if (workspace_bytes_given < workspace_bytes(p, B, K)) return PQ_ERR_WORKSPACE;
    if (!(p.filter || p.tiled || m == 8))
        return PQ_ERR_UNSUPPORTED;                             // (scan kernels with a measurement instance)
    const int waves = p.filter ? kFilterWaves : (!p.tiled && p.big) ? kMaxWaves : kWaves;
    const long long scan_groups = p.filter ? (long long)p.nblk * ((B + p.f_queries - 1) / p.f_queries) : p.tiled ? (long long)p.nblk * ((B + kQ - 1) / kQ) : (long long)p.nblk * B;
    if (scan_groups * waves > PQ_STAMP_RECORDS || (long long)B * ((B <= kAssumedCUs ? kFoldThreads : kThreads) / kWave) > PQ_STAMP_RECORDS) return PQ_ERR_UNSUPPORTED;
    if (scan_grid != nullptr) { scan_grid[0] = (int)scan_groups; scan_grid[1] = waves; }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t section = (size_t)PQ_STAMP_RECORDS * PQ_STAMP_SLOTS;
    if (B == 1 && d / m == 64 && (m * b + kSubThreads - 1) / kSubThreads <= PQ_STAMP_RECORDS) {
        if (((long long)m * b) % kSubThreads == 0 && ((uintptr_t)centroids & 15) == 0)
            hipLaunchKernelGGL((subitem_scores_kernel<64, true, true>), dim3(m * b / kSubThreads, 1), dim3(kSubThreads), 0,
                               st, queries, centroids, S, B, d, m, b, stamps);
        else
            hipLaunchKernelGGL((subitem_scores_kernel<64, true>), dim3((m * b + kSubThreads - 1) / kSubThreads, 1), dim3(kSubThreads), 0,
                               st, queries, centroids, S, B, d, m, b, stamps);
        rc = record_hip(hipGetLastError());
    } else {
        rc = pq_subitem_scores(queries, centroids, S, B, d, m, b, stream);   // (no measurement instance: section 0 stays empty)
    }
    if (rc != PQ_OK) return rc;
    rc = enqueue_scan(p, codes, S, N, B, m, b, K, workspace, out_ids, out_scores, st, nullptr, 0, 1, stamps + section);
    if (rc != PQ_OK) return rc;
    return enqueue_fold(p, B, K, workspace, out_ids, out_scores, st, stamps + 2 * section);
}

size_t pq_score_topk_u16_workspace_bytes(long long N, int B, int m, int b, int K) {
    if (check_topk_shape(N, B, m, b, K, 2) != PQ_OK) return 0;
    const ScanPlan p = make_plan(N, B, m, K, false, 2, b);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return 0;
    return workspace_bytes(p, B, K);
}

int pq_score_topk_u16(const uint16_t* codes, const float* S, long long N, int B, int m, int b, int K, int* out_ids,
                      float* out_scores, void* workspace, size_t workspace_bytes_given, void* stream) {
    int rc = check_topk_args(codes, S, N, B, m, b, K, out_ids, out_scores, workspace, workspace_bytes_given, 2);
    if (rc != PQ_OK) return rc;
    const ScanPlan p = make_plan(N, B, m, K, false, 2, b);
    hipStream_t st = static_cast<hipStream_t>(stream);
    rc = enqueue_scan(p, reinterpret_cast<const uint8_t*>(codes), S, N, B, m, b, K, workspace, out_ids, out_scores, st, nullptr, 0, 2);
    if (rc != PQ_OK) return rc;
    return enqueue_fold(p, B, K, workspace, out_ids, out_scores, st);
}

int pq_score_topk_u16_profile(const uint16_t* codes, const float* S, long long N, int B, int m, int b, int K,
                              int* out_ids, float* out_scores, void* workspace, size_t workspace_bytes_given,
                              void* stream, int iters, float* scan_ms) {
    return profile_scan(reinterpret_cast<const uint8_t*>(codes), S, N, B, m, b, K, out_ids, out_scores, workspace,
                        workspace_bytes_given, stream, iters, scan_ms, 2);
}

size_t pq_score_topk_subset_workspace_bytes(long long n_subset, int B, int m, int b, int K) {
    if (n_subset < 1 || B < 1 || m < 1 || b < 1 || K < 1 || b > 256 || K > n_subset || n_subset >= 2147483648LL) return 0;
    if (K > PQ_MAX_K || m > PQ_MAX_M || B > PQ_MAX_B) return 0;
    const ScanPlan p = make_plan(n_subset, B, m, K, true);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return 0;
    return workspace_bytes(p, B, K);
}

int pq_score_topk_subset(const uint8_t* codes, const float* S, const int* subset, long long n_subset, long long N,
                         int B, int m, int b, int K, int* out_ids, float* out_scores, void* workspace,
                         size_t workspace_bytes_given, void* stream) {
    if (!codes || !S || !subset || !out_ids || !out_scores || !workspace) return PQ_ERR_NULL;
    if (n_subset < 1 || N < 1 || B < 1 || m < 1 || b < 1 || K < 1 || b > 256 || K > n_subset || n_subset > N ||
        N >= 2147483648LL)
        return PQ_ERR_SHAPE;
    if (K > PQ_MAX_K || m > PQ_MAX_M || B > PQ_MAX_B) return PQ_ERR_UNSUPPORTED;
    const ScanPlan p = make_plan(n_subset, B, m, K, true);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return PQ_ERR_UNSUPPORTED;
    if (((uintptr_t)codes & 15) || ((uintptr_t)workspace & 15) || ((uintptr_t)S & 3) || ((uintptr_t)subset & 3) ||
        ((uintptr_t)out_ids & 3) || ((uintptr_t)out_scores & 3))
        return PQ_ERR_ALIGN;
    if (workspace_bytes_given < workspace_bytes(p, B, K)) return PQ_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    int rc = enqueue_scan(p, codes, S, n_subset, B, m, b, K, workspace, out_ids, out_scores, st, subset, N);
    if (rc != PQ_OK) return rc;
    return enqueue_fold(p, B, K, workspace, out_ids, out_scores, st);
}

int pq_read_bandwidth_profile(const void* data, size_t bytes, void* stream, int iters, float* read_ms) {
    if (!data || !read_ms) return PQ_ERR_NULL;
    if (bytes < 16 || iters < 1) return PQ_ERR_SHAPE;
    if ((uintptr_t)data & 15) return PQ_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const long long nvec = (long long)(bytes / 16);
    long long blocks = (nvec + kReadThreads - 1) / kReadThreads;
    if (blocks > 2LL * kAssumedCUs) blocks = 2LL * kAssumedCUs;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    hipError_t e = hipEventCreate(&ev0);
    if (e != hipSuccess) return record_hip(e);
    e = hipEventCreate(&ev1);
    if (e != hipSuccess) { (void)hipEventDestroy(ev0); return record_hip(e); }
    auto launch = [&]() {
        hipLaunchKernelGGL(stream_read_kernel, dim3((unsigned)blocks), dim3(kReadThreads), 0, st,
                           static_cast<const uint4*>(data), nvec);
        return record_hip(hipGetLastError());
    };
    int rc = launch();                                       // untimed warm-up launch
    if (rc == PQ_OK) rc = record_hip(hipEventRecord(ev0, st));
    for (int it = 0; it < iters && rc == PQ_OK; ++it) rc = launch();
    if (rc == PQ_OK) rc = record_hip(hipEventRecord(ev1, st));
    if (rc == PQ_OK) rc = record_hip(hipStreamSynchronize(st));
    float ms = 0.0f;
    if (rc == PQ_OK) rc = record_hip(hipEventElapsedTime(&ms, ev0, ev1));
    (void)hipEventDestroy(ev0);
    (void)hipEventDestroy(ev1);
    if (rc == PQ_OK) *read_ms = ms / (float)iters;
    return rc;
}

// ---- the comparison scorers (Section 2's default scoring, Algorithm 2) and TopK over score rows

namespace {
// plan of pq_topk_scores: blocks per query, list and candidate sizes (as for the scan), LDS of the two launches
ScanPlan make_topk_scores_plan(long long N, int B, int K) {
    ScanPlan p = {};
    const long long vecs = N / 4;
    const long long per_round = (long long)kThreads * kScoreVecs;
    long long rounds = (vecs + per_round - 1) / per_round;
    if (rounds < 1) rounds = 1;
    long long most = (kBlocksPerCU * (long long)kAssumedCUs) / B;
    if (most < 8) most = 8;
    p.nblk = (int)(rounds < most ? rounds : most);
    p.cap = list_capacity(K);
    p.candmax = next_pow2(2 * K);
    if (p.candmax < 512) p.candmax = 512;
    p.copies = 1;
    p.scan_dyn_lds = p.scan_lds = scan_lds_bytes(0, p.cap, p.candmax, K, kWaves);
    p.fold_lds = fold_lds_bytes(K);
    return p;
}

int check_topk_scores_shape(long long ld, long long N, int B, int K) {
    if (N < 1 || B < 1 || K < 1 || K > N || ld < N || N >= 2147483648LL) return PQ_ERR_SHAPE;
    if (K > PQ_MAX_K || B > PQ_MAX_B) return PQ_ERR_UNSUPPORTED;
    return PQ_OK;
}
}  // namespace

size_t pq_topk_scores_workspace_bytes(long long N, int B, int K) {
    if (check_topk_scores_shape(N, N, B, K) != PQ_OK) return 0;
    const ScanPlan p = make_topk_scores_plan(N, B, K);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return 0;
    return workspace_bytes(p, B, K);
}

int pq_topk_scores(const float* scores, long long ld, long long N, int B, int K, int* out_ids, float* out_scores,
                   void* workspace, size_t workspace_bytes_given, void* stream) {
    if (!scores || !out_ids || !out_scores || !workspace) return PQ_ERR_NULL;
    int rc = check_topk_scores_shape(ld, N, B, K);
    if (rc != PQ_OK) return rc;
    const ScanPlan p = make_topk_scores_plan(N, B, K);
    if (p.scan_lds > kMaxLdsBytes || p.fold_lds > kMaxLdsBytes) return PQ_ERR_UNSUPPORTED;
    if (((uintptr_t)scores & 15) || (B > 1 && (ld & 3)) || ((uintptr_t)workspace & 15) || ((uintptr_t)out_ids & 3) ||
        ((uintptr_t)out_scores & 3))
        return PQ_ERR_ALIGN;
    if (workspace_bytes_given < workspace_bytes(p, B, K)) return PQ_ERR_WORKSPACE;
    hipStream_t st = static_cast<hipStream_t>(stream);
    TopkScoresArgs a;
    a.scores = scores; a.ld = ld; a.N = N; a.K = K; a.cap = p.cap; a.candmax = p.candmax;
    a.prune_at = (K <= 28) ? 2 * K + 8 : 0;
    a.ws_keys = static_cast<uint64_t*>(workspace);
    hipError_t e = allow_lds(topk_scores_kernel, p.scan_dyn_lds);
    if (e != hipSuccess) return record_hip(e);
    hipLaunchKernelGGL(topk_scores_kernel, dim3(p.nblk, B), dim3(kThreads), p.scan_dyn_lds, st, a);
    e = hipGetLastError();
    if (e != hipSuccess) return record_hip(e);
    return enqueue_fold(p, B, K, workspace, out_ids, out_scores, st);
}

int pq_recjpq_scores(const uint8_t* codes, const float* S, long long N, int B, int m, int b, float* scores,
                     long long ld, void* stream) {
    if (!codes || !S || !scores) return PQ_ERR_NULL;
    if (N < 1 || B < 1 || m < 1 || b < 1 || b > 256 || ld < N || N >= 2147483648LL) return PQ_ERR_SHAPE;
    if (m > PQ_MAX_M || B > PQ_MAX_B) return PQ_ERR_UNSUPPORTED;
    if (((uintptr_t)S & 3) || ((uintptr_t)scores & 3)) return PQ_ERR_ALIGN;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid((unsigned)((N + 4LL * kRecjpqThreads - 1) / (4LL * kRecjpqThreads)), B);
    for (int k = 0; k < m; ++k) {                            // Algorithm 2's outer loop: one pass over the items per split
        hipLaunchKernelGGL(recjpq_pass_kernel, grid, dim3(kRecjpqThreads), 0, st, codes, S, scores, ld, N, m, b, k);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return record_hip(e);
    }
    return PQ_OK;
}

int pq_reconstruct_items(const uint8_t* codes, const float* centroids, long long N, int d, int m, int b, float* W,
                         void* stream) {
    if (!codes || !centroids || !W) return PQ_ERR_NULL;
    if (N < 1 || d < 1 || m < 1 || b < 1 || b > 256 || d % m != 0 || N >= 2147483648LL) return PQ_ERR_SHAPE;
    if (m > PQ_MAX_M) return PQ_ERR_UNSUPPORTED;
    if (((uintptr_t)centroids & 3) || ((uintptr_t)W & 3)) return PQ_ERR_ALIGN;
    const long long total = N * d;
    long long blocks = (total + 255) / 256;
    if (blocks > 64 * kAssumedCUs) blocks = 64 * kAssumedCUs;
    hipLaunchKernelGGL(reconstruct_kernel, dim3((unsigned)blocks), dim3(256), 0, static_cast<hipStream_t>(stream), codes,
                       centroids, W, N, d, m, b);
    return record_hip(hipGetLastError());
}

int pq_default_scores(const float* W, const float* queries, long long N, int B, int d, float* scores, long long ld,
                      void* stream) {
    if (!W || !queries || !scores) return PQ_ERR_NULL;
    if (N < 1 || B < 1 || d < 1 || ld < N || N >= 2147483648LL) return PQ_ERR_SHAPE;
    if (B > PQ_MAX_B || d % 4 != 0 || (size_t)d * sizeof(float) > 64 * 1024) return PQ_ERR_UNSUPPORTED;
    if (((uintptr_t)W & 15) || ((uintptr_t)queries & 15) || ((uintptr_t)scores & 3)) return PQ_ERR_ALIGN;
    // batches: one pass over W for all queries, on the matrix cores (the same kernel as Eq. 4: one split, the items in
    // the place of the sub-ids); a single query, or a shape that kernel does not take: one mat-vec pass per query
    if (B >= kDefaultMfmaMinBatch && !(g_force_general.load(std::memory_order_relaxed) & 4) &&
        launch_subitem_mfma(queries, W, scores, B, d, 1, N, ld, static_cast<hipStream_t>(stream)))
        return record_hip(hipGetLastError());
    long long blocks = (N + kDefaultThreads / 16 - 1) / (kDefaultThreads / 16);
    if (blocks > 16 * kAssumedCUs) blocks = 16 * kAssumedCUs;
    hipLaunchKernelGGL(default_scores_kernel, dim3((unsigned)blocks, B), dim3(kDefaultThreads), (size_t)d * sizeof(float),
                       static_cast<hipStream_t>(stream), W, queries, scores, ld, N, d);
    return record_hip(hipGetLastError());
}

const char* pq_strerror(int code) {
    switch (code) {
        case PQ_OK: return "ok";
        case PQ_ERR_NULL: return "a required pointer is NULL";
        case PQ_ERR_SHAPE:
            return "bad shape: need B,d,m,b,K,N >= 1, d % m == 0, b <= 256 (65536 with 16-bit sub-ids), K <= N (K <= |V| <= N with a "
                   "candidate list), N < 2^31";
        case PQ_ERR_UNSUPPORTED:
            return "unsupported: K > 512, m > 128, B > 65535, or score tables plus candidate lists exceed LDS";
        case PQ_ERR_WORKSPACE: return "workspace smaller than pq_score_topk_workspace_bytes()";
        case PQ_ERR_ALIGN: return "pointer alignment: codes and workspace 16 bytes, float/int arrays 4 bytes";
        case PQ_ERR_HIP: return g_hip_error;
        case PQ_ERR_TOO_LARGE: return "problem needs more scratch than the library's built-in array holds (PQ_STATIC_SCRATCH_BYTES)";
        default: return "unknown pqtopk error code";
    }
}

}  // extern "C"
