// Device code of the PQTopK library: every kernel template, in namespace pqk, and the list of scan-kernel instances.
//
// The catalogue-scan kernels are large (40-120 KB of code each), so they are compiled in translation units of their
// own (inst_*.hip, each instantiating one group of the list below); every other translation unit sees them as
// `extern template` and only launches them.  The small kernels (Eq. 4, fold, comparison scorers) are instantiated
// where they are launched.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace pqk {

#include "common.hpp"
#include "subitem_scores.hpp"
#include "topk_parts.hpp"
#include "select_small.hpp"
#include "scan_single.hpp"
#include "scan_bytes.hpp"
#include "scan_short.hpp"
#include "scan_pair.hpp"
#include "scan_long.hpp"
#include "scan_subset.hpp"
#include "scan_batched.hpp"
#include "scan_filter.hpp"
#include "fold.hpp"
#ifndef PQ_INSTANCE_TU
#include "comparison.hpp"   // (kernels that are no templates: defined once, in the translation unit that launches them)
#endif

// scan_topk_kernel<M, C, NT, CW, GL> instances, by translation unit.  X(M, C, NT, CW, GL).
// one-byte sub-ids, rows of 1, 2 and 4 bytes (each with and without replicated tables)
#define PQ_SCAN_INSTANCES_U8_NARROW(X) \
    X(1, kTableCopies, kBigThreads, 1, false) X(1, 1, kThreads, 1, false) \
    X(2, kTableCopies, kBigThreads, 1, false) X(2, 1, kThreads, 1, false) \
    X(4, kTableCopies, kBigThreads, 1, false) X(4, 1, kThreads, 1, false)
// one-byte sub-ids, m = 8 and 16 (the named workloads)
#define PQ_SCAN_INSTANCES_U8_MAIN(X) \
    X(8, kTableCopies, kBigThreads, 1, false) X(8, 1, kThreads, 1, false) X(16, 1, kThreads, 1, false)
// one-byte sub-ids, m = 32 and 64
#define PQ_SCAN_INSTANCES_U8_WIDE(X) \
    X(32, 1, kThreads, 1, false) X(64, 1, kBigThreads, 1, false) X(64, 1, kThreads, 1, false)
// any m, row by row (also the candidate-list scan)
#define PQ_SCAN_INSTANCES_GENERIC(X) \
    X(0, 1, kBigThreads, 1, false) X(0, 1, kThreads, 1, false) \
    X(0, 1, kThreads, 2, true) X(0, 1, kBigThreads, 2, false) X(0, 1, kThreads, 2, false)
// two-byte sub-ids, rows of 8, 16 and 32 bytes
#define PQ_SCAN_INSTANCES_U16(X) \
    X(4, 1, kThreads, 2, true) X(4, 1, kBigThreads, 2, false) X(4, 1, kThreads, 2, false) \
    X(8, 1, kThreads, 2, true) X(8, 1, kBigThreads, 2, false) X(8, 1, kThreads, 2, false) \
    X(16, 1, kThreads, 2, true) X(16, 1, kBigThreads, 2, false) X(16, 1, kThreads, 2, false)
// measurement instances (wall-clock stamps per wave) of the two kernels the named single-query workloads run
#define PQ_SCAN_INSTANCES_STAMPED(X) X(8, 1, kThreads, 1, false, true) X(8, kTableCopies, kBigThreads, 1, false, true)
// scan_short_kernel<M, U, NT, STAMP> instances: every number of units per thread up to short_held_units(M) and the
// larger instances; measurement instances for m = 8
#define PQ_SHORT_U(X, M, U) X(M, U, kThreads, false)
#define PQ_SHORT_U4(X, M, U) PQ_SHORT_U(X, M, U) PQ_SHORT_U(X, M, U + 1) PQ_SHORT_U(X, M, U + 2) PQ_SHORT_U(X, M, U + 3)
#define PQ_SHORT_INSTANCES_A(X) \
    PQ_SHORT_U4(X, 8, 1) PQ_SHORT_U4(X, 8, 5) PQ_SHORT_U4(X, 8, 9) \
    X(8, 1, kThreads, true) X(8, 2, kThreads, true) X(8, 3, kThreads, true) X(8, 4, kThreads, true) X(8, 5, kThreads, true) \
    X(8, 6, kThreads, true) X(8, 7, kThreads, true) X(8, 8, kThreads, true) \
    PQ_SHORT_U(X, 1, 1) PQ_SHORT_U(X, 1, 2) PQ_SHORT_U(X, 2, 1) PQ_SHORT_U(X, 2, 2) \
    PQ_SHORT_U4(X, 4, 1) PQ_SHORT_U(X, 4, 5) PQ_SHORT_U(X, 4, 6)
#define PQ_SHORT_INSTANCES_D(X) \
    X(8, 9, kThreads, true) X(8, 10, kThreads, true) X(8, 11, kThreads, true) X(8, 12, kThreads, true) \
    X(8, 16, kThreads, true) X(8, 24, kThreads, true) X(8, 32, kThreads, true) \
    PQ_SHORT_U(X, 4, 8) PQ_SHORT_U(X, 4, 12) PQ_SHORT_U(X, 4, 16) PQ_SHORT_U(X, 8, 16) PQ_SHORT_U(X, 8, 24) PQ_SHORT_U(X, 8, 32) \
    PQ_SHORT_U(X, 16, 16) PQ_SHORT_U(X, 16, 24) PQ_SHORT_U(X, 16, 32) PQ_SHORT_U(X, 16, 48)
#define PQ_SHORT_INSTANCES_E(X) \
    PQ_SHORT_U(X, 32, 12) PQ_SHORT_U(X, 32, 16) PQ_SHORT_U(X, 32, 24) PQ_SHORT_U(X, 32, 32) \
    PQ_SHORT_U(X, 64, 8) PQ_SHORT_U(X, 64, 12) PQ_SHORT_U(X, 64, 16) PQ_SHORT_U(X, 64, 24) PQ_SHORT_U(X, 64, 32)
#define PQ_SHORT_INSTANCES_B(X) \
    PQ_SHORT_U4(X, 16, 1) PQ_SHORT_U4(X, 16, 5) PQ_SHORT_U4(X, 16, 9)
#define PQ_SHORT_INSTANCES_C(X) \
    PQ_SHORT_U4(X, 32, 1) PQ_SHORT_U4(X, 32, 5) PQ_SHORT_U4(X, 64, 1)
// scan_short_kernel<M, U, NT, false, 2>: two-byte sub-ids, m = 4, 8 (up to 12 code vectors per thread), 16 (up to 6 items)
#define PQ_SHORT16_U(X, M, U) X(M, U, kThreads, false, 2)
// scan_pair_kernel<M, U, NT, CW>: every number of units up to pair_held_units() and the larger instances, up to pair_max_units()
#define PQ_PAIR_U(X, M, U, CW) X(M, U, kThreads, CW)
#define PQ_PAIR_U4(X, M, U, CW) PQ_PAIR_U(X, M, U, CW) PQ_PAIR_U(X, M, U + 1, CW) PQ_PAIR_U(X, M, U + 2, CW) PQ_PAIR_U(X, M, U + 3, CW)
#define PQ_PAIR_20(X, M, CW) PQ_PAIR_U(X, M, 12, CW) PQ_PAIR_U(X, M, 16, CW) PQ_PAIR_U(X, M, 20, CW)
#define PQ_PAIR_40(X, M, CW) PQ_PAIR_20(X, M, CW) PQ_PAIR_U(X, M, 24, CW) PQ_PAIR_U(X, M, 32, CW) PQ_PAIR_U(X, M, 40, CW)
#define PQ_PAIR_INSTANCES_A(X) \
    PQ_PAIR_U4(X, 4, 1, 1) PQ_PAIR_U4(X, 4, 5, 1) \
    PQ_PAIR_U4(X, 8, 1, 1) PQ_PAIR_U4(X, 8, 5, 1) PQ_PAIR_20(X, 8, 1) \
    PQ_PAIR_U4(X, 16, 1, 1) PQ_PAIR_U4(X, 16, 5, 1) PQ_PAIR_40(X, 16, 1)
#define PQ_PAIR_INSTANCES_B(X) \
    PQ_PAIR_U4(X, 32, 1, 1) PQ_PAIR_U(X, 32, 8, 1) PQ_PAIR_40(X, 32, 1) \
    PQ_PAIR_U(X, 64, 1, 1) PQ_PAIR_U(X, 64, 2, 1) PQ_PAIR_U(X, 64, 4, 1) PQ_PAIR_U(X, 64, 8, 1) PQ_PAIR_20(X, 64, 1) PQ_PAIR_U(X, 64, 24, 1)
#define PQ_PAIR_INSTANCES_C(X) \
    PQ_PAIR_U4(X, 4, 1, 2) PQ_PAIR_U4(X, 4, 5, 2) PQ_PAIR_20(X, 4, 2) \
    PQ_PAIR_U4(X, 8, 1, 2) PQ_PAIR_U4(X, 8, 5, 2) PQ_PAIR_40(X, 8, 2) \
    PQ_PAIR_U4(X, 16, 1, 2) PQ_PAIR_U(X, 16, 8, 2) PQ_PAIR_40(X, 16, 2)
#define PQ_SHORT16_INSTANCES(X) \
    PQ_SHORT16_U(X, 4, 1) PQ_SHORT16_U(X, 4, 2) PQ_SHORT16_U(X, 4, 3) PQ_SHORT16_U(X, 4, 4) PQ_SHORT16_U(X, 4, 5) PQ_SHORT16_U(X, 4, 6) \
    PQ_SHORT16_U(X, 4, 7) PQ_SHORT16_U(X, 4, 8) PQ_SHORT16_U(X, 4, 9) PQ_SHORT16_U(X, 4, 10) PQ_SHORT16_U(X, 4, 11) PQ_SHORT16_U(X, 4, 12) \
    PQ_SHORT16_U(X, 8, 1) PQ_SHORT16_U(X, 8, 2) PQ_SHORT16_U(X, 8, 3) PQ_SHORT16_U(X, 8, 4) PQ_SHORT16_U(X, 8, 5) PQ_SHORT16_U(X, 8, 6) \
    PQ_SHORT16_U(X, 8, 7) PQ_SHORT16_U(X, 8, 8) PQ_SHORT16_U(X, 8, 9) PQ_SHORT16_U(X, 8, 10) PQ_SHORT16_U(X, 8, 11) PQ_SHORT16_U(X, 8, 12) \
    PQ_SHORT16_U(X, 4, 16) PQ_SHORT16_U(X, 4, 24) PQ_SHORT16_U(X, 4, 32) \
    PQ_SHORT16_U(X, 8, 16) PQ_SHORT16_U(X, 8, 24) PQ_SHORT16_U(X, 8, 32) PQ_SHORT16_U(X, 8, 48) \
    PQ_SHORT16_U(X, 16, 8) PQ_SHORT16_U(X, 16, 12) PQ_SHORT16_U(X, 16, 16) PQ_SHORT16_U(X, 16, 24) PQ_SHORT16_U(X, 16, 32) \
    PQ_SHORT16_U(X, 16, 1) PQ_SHORT16_U(X, 16, 2) PQ_SHORT16_U(X, 16, 3) PQ_SHORT16_U(X, 16, 4) PQ_SHORT16_U(X, 16, 5) PQ_SHORT16_U(X, 16, 6)
// scan_bytes_kernel<M, CW, STAMP> instances (measurement: m = 8)
#define PQ_BYTES_INSTANCES(X) \
    X(4, 1, false) X(8, 1, false) X(16, 1, false) X(32, 1, false) X(64, 1, false) X(4, 2, false) X(8, 2, false) X(16, 2, false) X(8, 1, true)
// scan_long_kernel<M, CW, C>
#define PQ_LONG_INSTANCES(X) \
    X(4, 1, kTableCopies) X(8, 1, kTableCopies) X(16, 1, 1) X(32, 1, 1) X(64, 1, 1) X(4, 2, 1) X(8, 2, 1) X(16, 2, 1)
// scan_subset_kernel<M, U, NT>: rows of 4, 8, 16 bytes, every number of vectors per thread
#define PQ_SUBSET_M(X, M) X(M, 1, kThreads) X(M, 2, kThreads) X(M, 3, kThreads) X(M, 4, kThreads) X(M, 5, kThreads) \
    X(M, 6, kThreads) X(M, 7, kThreads) X(M, 8, kThreads)
#define PQ_SUBSETP_M(X, M) X(M, 1, kThreads) X(M, 2, kThreads) X(M, 3, kThreads) X(M, 4, kThreads) X(M, 6, kThreads) X(M, 8, kThreads)
#define PQ_SUBSETP_INSTANCES(X) PQ_SUBSETP_M(X, 4) PQ_SUBSETP_M(X, 8) PQ_SUBSETP_M(X, 16) X(8, 12, kThreads) X(8, 16, kThreads) \
    X(16, 12, kThreads) X(16, 16, kThreads) X(16, 24, kThreads)
#define PQ_SUBSET_INSTANCES(X) PQ_SUBSET_M(X, 4) PQ_SUBSET_M(X, 8) PQ_SUBSET_M(X, 16)
// scan_filter_kernel<M, CW, W, W16, SUB, G, SHARE> and filter_prepare_kernel<M, CW, SUB, NT>, by translation unit.  X for scans, Y
// for the kernels that prepare them
#define PQ_FILTER_BOTH(X, M, CW, W, W16, SUB, G) X(M, CW, W, W16, SUB, G, false) X(M, CW, W, W16, SUB, G, true)
#define PQ_FILTER_W(X, M, CW, SUB) X(M, CW, 1, false, SUB, 1, false) PQ_FILTER_BOTH(X, M, CW, 2, false, SUB, 1) PQ_FILTER_BOTH(X, M, CW, 4, false, SUB, 1)
#define PQ_FILTER_G(X, M, CW, SUB) PQ_FILTER_W(X, M, CW, SUB) PQ_FILTER_BOTH(X, M, CW, 4, false, SUB, 2)
#define PQ_FILTER_INSTANCES_A(X, Y) PQ_FILTER_G(X, 4, 1, false) Y(4, 1, false)
#define PQ_FILTER_INSTANCES_A8(X, Y) PQ_FILTER_G(X, 8, 1, false) Y(8, 1, false)
#define PQ_FILTER_INSTANCES_B(X, Y) PQ_FILTER_G(X, 16, 1, false) PQ_FILTER_BOTH(X, 16, 1, 4, true, false, 1) Y(16, 1, false)
// (64 splits: 16-bit fields always, and room for four queries)
#define PQ_FILTER_INSTANCES_C(X, Y) \
    X(32, 1, 1, false, false, 1, false) PQ_FILTER_BOTH(X, 32, 1, 2, false, false, 1) PQ_FILTER_BOTH(X, 32, 1, 4, false, false, 1) \
    PQ_FILTER_BOTH(X, 32, 1, 2, true, false, 1) PQ_FILTER_BOTH(X, 32, 1, 4, true, false, 1) \
    PQ_FILTER_BOTH(X, 64, 1, 1, true, false, 1) PQ_FILTER_BOTH(X, 64, 1, 2, true, false, 1) Y(32, 1, false) Y(64, 1, false)
// (lists: pairs of lanes at m = 4 alone; m = 16: eight queries of bytes are a workgroup's where there are no more, over too short shares to share floors)
#define PQ_FILTER_INSTANCES_SUBSET(X, Y) PQ_FILTER_G(X, 4, 1, true) PQ_FILTER_W(X, 8, 1, true) Y(4, 1, true) Y(8, 1, true)
#define PQ_FILTER_INSTANCES_SUBSET16(X, Y) X(16, 1, 1, false, true, 1, false) X(16, 1, 2, false, true, 1, false) PQ_FILTER_BOTH(X, 16, 1, 4, false, true, 1) PQ_FILTER_BOTH(X, 16, 1, 4, true, true, 1) Y(16, 1, true)
#define PQ_FILTER_INSTANCES_U16(X, Y) PQ_FILTER_G(X, 4, 2, false) PQ_FILTER_G(X, 8, 2, false) X(4, 2, 1, false, false, 1, true) X(8, 2, 1, false, false, 1, true) Y(4, 2, false) Y(8, 2, false)
#define PQ_FILTER_INSTANCES_U16_16(X, Y) PQ_FILTER_G(X, 16, 2, false) X(16, 2, 1, false, false, 1, true) \
    PQ_FILTER_BOTH(X, 16, 2, 1, true, false, 1) PQ_FILTER_BOTH(X, 16, 2, 2, true, false, 1) PQ_FILTER_BOTH(X, 16, 2, 4, true, false, 1) Y(16, 2, false)
// measurement instances (wall-clock stamps per wave) of those the named batch workloads run
#define PQ_FILTER_STAMPED(X, M, G) X(M, 1, 4, false, false, G, false, true) X(M, 1, 4, false, false, G, true, true)
#define PQ_FILTER_INSTANCES_STAMPED(X) PQ_FILTER_STAMPED(X, 8, 1) PQ_FILTER_STAMPED(X, 8, 2) PQ_FILTER_STAMPED(X, 16, 1)
// all splits in LDS: short shares (m = 8), many results (m = 16)
#define PQ_FILTER_INSTANCES_NEAR(X) X(8, 1, 4, false, false, 1, false, false, false, true) X(8, 1, 4, false, false, 1, true, false, false, true) X(16, 1, 4, false, false, 1, false, false, false, true)
#define PQ_FILTER_INSTANCES_NEAR_STAMPED(X) X(8, 1, 4, false, false, 1, false, true, false, true) X(8, 1, 4, false, false, 1, true, true, false, true) X(16, 1, 4, false, false, 1, false, true, false, true)
// ... and those with 16-bit counts beside the bytes
#define PQ_FILTER_INSTANCES_FINE(X) X(16, 1, 2, false, false, 1, false, false, true) X(16, 1, 2, false, false, 1, true, false, true) X(8, 1, 4, false, true, 1, true, false, true)
// the batched kernel
#define PQ_TILED_INSTANCES(X) X(8, false) X(16, false) X(8, true) X(16, true)

#define PQ_SCAN_DEFINE(M, C, NT, CW, GL) template __global__ void scan_topk_kernel<M, C, NT, CW, GL>(ScanArgs);
#define PQ_SCAN_EXTERN(M, C, NT, CW, GL) extern PQ_SCAN_DEFINE(M, C, NT, CW, GL)
#define PQ_SCAN_DEFINE6(M, C, NT, CW, GL, ST) template __global__ void scan_topk_kernel<M, C, NT, CW, GL, ST>(ScanArgs);
#define PQ_SCAN_EXTERN6(M, C, NT, CW, GL, ST) extern PQ_SCAN_DEFINE6(M, C, NT, CW, GL, ST)
#define PQ_SHORT_DEFINE(M, U, NT, ST) template __global__ void scan_short_kernel<M, U, NT, ST>(const uint8_t*, const float*, void*, float*, uint32_t, int, int, uint64_t*);
#define PQ_SHORT_EXTERN(M, U, NT, ST) extern PQ_SHORT_DEFINE(M, U, NT, ST)
#define PQ_SHORT16_DEFINE(M, U, NT, ST, CW) template __global__ void scan_short_kernel<M, U, NT, ST, CW>(const uint8_t*, const float*, void*, float*, uint32_t, int, int, uint64_t*);
#define PQ_PAIR_DEFINE(M, U, NT, CW) template __global__ void scan_pair_kernel<M, U, NT, CW>(const uint8_t*, const float*, void*, float*, uint32_t, int, int, int);
#define PQ_PAIR_EXTERN(M, U, NT, CW) extern PQ_PAIR_DEFINE(M, U, NT, CW)
#define PQ_SHORT16_EXTERN(M, U, NT, ST, CW) extern PQ_SHORT16_DEFINE(M, U, NT, ST, CW)
#define PQ_BYTES_DEFINE(M, CW, ST) template __global__ void scan_bytes_kernel<M, CW, ST>(ScanArgs);
#define PQ_BYTES_EXTERN(M, CW, ST) extern PQ_BYTES_DEFINE(M, CW, ST)
#define PQ_LONG_DEFINE(M, CW, C) template __global__ void scan_long_kernel<M, CW, C>(const uint8_t*, const float*, void*, float*, uint32_t, int, int);
#define PQ_LONG_EXTERN(M, CW, C) extern PQ_LONG_DEFINE(M, CW, C)
#define PQ_SUBSET_DEFINE(M, U, NT) template __global__ void scan_subset_kernel<M, U, NT>(const uint8_t*, const int*, const float*, void*, float*, uint32_t, uint32_t, int, int);
#define PQ_SUBSET_EXTERN(M, U, NT) extern PQ_SUBSET_DEFINE(M, U, NT)
#define PQ_SUBSETP_DEFINE(M, U, NT) template __global__ void scan_subset_pair_kernel<M, U, NT>(const uint8_t*, const int*, const float*, void*, float*, uint32_t, uint32_t, int, int, int);
#define PQ_SUBSETP_EXTERN(M, U, NT) extern PQ_SUBSETP_DEFINE(M, U, NT)
#define PQ_FILTER_DEFINE(M, CW, W, W16, SUB, G, SH) template __global__ void scan_filter_kernel<M, CW, W, W16, SUB, G, SH>(FilterArgs);
#define PQ_FILTER_EXTERN(M, CW, W, W16, SUB, G, SH) extern PQ_FILTER_DEFINE(M, CW, W, W16, SUB, G, SH)
#define PQ_FILTER_DEFINE8(M, CW, W, W16, SUB, G, SH, ST) template __global__ void scan_filter_kernel<M, CW, W, W16, SUB, G, SH, ST>(FilterArgs);
#define PQ_FILTER_EXTERN8(M, CW, W, W16, SUB, G, SH, ST) extern PQ_FILTER_DEFINE8(M, CW, W, W16, SUB, G, SH, ST)
#define PQ_FILTER_DEFINE9(M, CW, W, W16, SUB, G, SH, ST, FI) template __global__ void scan_filter_kernel<M, CW, W, W16, SUB, G, SH, ST, FI>(FilterArgs);
#define PQ_FILTER_EXTERN9(M, CW, W, W16, SUB, G, SH, ST, FI) extern PQ_FILTER_DEFINE9(M, CW, W, W16, SUB, G, SH, ST, FI)
#define PQ_FILTER_DEFINE10(M, CW, W, W16, SUB, G, SH, ST, FI, NE) template __global__ void scan_filter_kernel<M, CW, W, W16, SUB, G, SH, ST, FI, NE>(FilterArgs);
#define PQ_FILTER_EXTERN10(M, CW, W, W16, SUB, G, SH, ST, FI, NE) extern PQ_FILTER_DEFINE10(M, CW, W, W16, SUB, G, SH, ST, FI, NE)
#define PQ_FILTERP_DEFINE(M, CW, SUB) template __global__ void filter_prepare_kernel<M, CW, SUB, kFilterThreads>(FilterArgs); \
    template __global__ void filter_prepare_kernel<M, CW, SUB, kThreads>(FilterArgs);
#define PQ_FILTERP_EXTERN(M, CW, SUB) extern template __global__ void filter_prepare_kernel<M, CW, SUB, kFilterThreads>(FilterArgs); \
    extern template __global__ void filter_prepare_kernel<M, CW, SUB, kThreads>(FilterArgs);
#define PQ_TILED_DEFINE(M, ST) template __global__ void scan_topk_tiled_kernel<M, ST>(ScanArgs, int);
#define PQ_TILED_EXTERN(M, ST) extern PQ_TILED_DEFINE(M, ST)

#ifndef PQ_INSTANCE_TU
PQ_SCAN_INSTANCES_U8_NARROW(PQ_SCAN_EXTERN)
PQ_SCAN_INSTANCES_U8_MAIN(PQ_SCAN_EXTERN)
PQ_SCAN_INSTANCES_U8_WIDE(PQ_SCAN_EXTERN)
PQ_SCAN_INSTANCES_GENERIC(PQ_SCAN_EXTERN)
PQ_SCAN_INSTANCES_U16(PQ_SCAN_EXTERN)
PQ_SCAN_INSTANCES_STAMPED(PQ_SCAN_EXTERN6)
PQ_SHORT_INSTANCES_A(PQ_SHORT_EXTERN)
PQ_SHORT_INSTANCES_B(PQ_SHORT_EXTERN)
PQ_SHORT_INSTANCES_C(PQ_SHORT_EXTERN)
PQ_SHORT_INSTANCES_D(PQ_SHORT_EXTERN)
PQ_SHORT_INSTANCES_E(PQ_SHORT_EXTERN)
PQ_LONG_INSTANCES(PQ_LONG_EXTERN)
PQ_BYTES_INSTANCES(PQ_BYTES_EXTERN)
PQ_SUBSET_INSTANCES(PQ_SUBSET_EXTERN)
PQ_SUBSETP_INSTANCES(PQ_SUBSETP_EXTERN)
PQ_SHORT16_INSTANCES(PQ_SHORT16_EXTERN)
PQ_PAIR_INSTANCES_A(PQ_PAIR_EXTERN)
PQ_PAIR_INSTANCES_B(PQ_PAIR_EXTERN)
PQ_PAIR_INSTANCES_C(PQ_PAIR_EXTERN)
PQ_TILED_INSTANCES(PQ_TILED_EXTERN)
PQ_FILTER_INSTANCES_STAMPED(PQ_FILTER_EXTERN8)
PQ_FILTER_INSTANCES_FINE(PQ_FILTER_EXTERN9)
PQ_FILTER_INSTANCES_NEAR(PQ_FILTER_EXTERN10)
PQ_FILTER_INSTANCES_NEAR_STAMPED(PQ_FILTER_EXTERN10)
PQ_FILTER_INSTANCES_A(PQ_FILTER_EXTERN, PQ_FILTERP_EXTERN)
PQ_FILTER_INSTANCES_A8(PQ_FILTER_EXTERN, PQ_FILTERP_EXTERN)
PQ_FILTER_INSTANCES_B(PQ_FILTER_EXTERN, PQ_FILTERP_EXTERN)
PQ_FILTER_INSTANCES_C(PQ_FILTER_EXTERN, PQ_FILTERP_EXTERN)
PQ_FILTER_INSTANCES_SUBSET(PQ_FILTER_EXTERN, PQ_FILTERP_EXTERN)
PQ_FILTER_INSTANCES_U16(PQ_FILTER_EXTERN, PQ_FILTERP_EXTERN)
PQ_FILTER_INSTANCES_U16_16(PQ_FILTER_EXTERN, PQ_FILTERP_EXTERN)
PQ_FILTER_INSTANCES_SUBSET16(PQ_FILTER_EXTERN, PQ_FILTERP_EXTERN)
#endif

}  // namespace pqk
