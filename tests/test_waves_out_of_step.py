"""The scan by one-byte bounds on the CPU, one workgroup, waves far out of step (no GPU): what no barrier orders gives other results or waves that
wait at different barriers."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2408_09992_amd", "csrc")
PARTS = ("common.hpp", "topk_parts.hpp", "scan_single.hpp", "scan_bytes.hpp")

MAIN = r"""
#include "workgroup_on_cpu.hpp"
namespace pqk {
#include "common.hpp"
#include "topk_parts.hpp"
#include "scan_single.hpp"
#include "scan_bytes.hpp"
}
template <int M, int CW>
bool go(const pqk::ScanArgs& a, const std::vector<int>& order) { return emu::run(pqk::kBytesThreads, order, [&]() { pqk::scan_bytes_kernel<M, CW>(a); }); }
int main(int argc, char** argv) {   // file of codes, of scores, of keys; m, bytes of a sub-id, b, N, K, capacity of a list, of the candidates; waves in order
    auto read = [](const char* name) {
        FILE* f = fopen(name, "rb");
        fseek(f, 0, SEEK_END);
        std::vector<uint4> v(ftell(f) / 16 + 1);
        rewind(f);
        if (fread(v.data(), 1, v.size() * 16, f) == 0) abort();
        fclose(f);
        return v;
    };
    const std::vector<uint4> codes = read(argv[1]), scores = read(argv[2]);
    pqk::ScanArgs a{};
    a.codes = reinterpret_cast<const uint8_t*>(codes.data());
    a.S = reinterpret_cast<const float*>(scores.data());
    const int cw = atoi(argv[5]);
    a.m = atoi(argv[4]); a.b = atoi(argv[6]); a.N = atoll(argv[7]); a.K = atoi(argv[8]); a.cap = atoi(argv[9]); a.candmax = atoi(argv[10]);
    std::vector<uint64_t> keys(a.K);
    a.ws_keys = keys.data();
    a.n_items = (uint32_t)a.N;
    std::vector<int> order;
    for (int i = 11; i < argc; ++i) order.push_back(atoi(argv[i]));
    const bool ok = cw == 2 ? go<8, 2>(a, order) : a.m == 8 ? go<8, 1>(a, order) : go<64, 1>(a, order);
    FILE* f = fopen(argv[3], "wb");
    fwrite(keys.data(), 8, keys.size(), f);
    fclose(f);
    printf("%lld %lld %lld\n", emu::counted, emu::scored, emu::barriers);
    return ok ? 0 : 1;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("needs g++")
    at = tmp_path_factory.mktemp("waves")
    for name in PARTS:
        with open(os.path.join(CSRC, name)) as f:
            text = f.read()
        text = text.replace("extern __shared__ __align__(16) unsigned char smem[];", "unsigned char* const smem = emu::lds;")
        (at / name).write_text(text)
    (at / "main.cpp").write_text(MAIN)
    build = subprocess.run([gxx, "-std=c++17", "-O1", "-fno-strict-aliasing", "-ffp-contract=off", "-w", "-I", str(at), "-I", os.path.join(ROOT, "tests"), str(at / "main.cpp"), "-o", str(at / "main")],
                           capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-4000:]
    return at


def scan(at, codes, S, K, order):
    """the workgroup's K best: (ids, scores), [additions to counters, pieces scored exactly, barriers]"""
    codes.tofile(at / "codes")
    S.astype(np.float32).tofile(at / "scores")
    cap = 1
    while cap < K + 64:
        cap *= 2
    run = subprocess.run([str(at / "main"), str(at / "codes"), str(at / "scores"), str(at / "keys"), str(codes.shape[1]), str(codes.dtype.itemsize), str(S.shape[1]), str(codes.shape[0]), str(K),
                          str(max(cap, 128)), "512"] + [str(w) for w in order], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, (run.stdout + run.stderr)[-2000:]
    keys = np.fromfile(at / "keys", dtype=np.uint64)
    high, low = (keys >> np.uint64(32)).astype(np.uint32), (keys & np.uint64(0xFFFFFFFF)).astype(np.uint32)
    return (~low).astype(np.int32), np.where(high >> 31, high ^ np.uint32(0x80000000), ~high).astype(np.uint32).view(np.float32), [int(x) for x in run.stdout.split()]


def expected(codes, S, K):
    score = S[0, codes[:, 0]].astype(np.float32)
    for k in range(1, codes.shape[1]):
        score = score + S[k, codes[:, k]]
    ids = np.argsort(-score, kind="stable")[:K]
    return ids.astype(np.int32), score[ids]


# a wave that is late everywhere, the first or the last, and waves front to back
ORDERS = [list(range(16)), list(range(1, 16)) + [0], list(range(15, -1, -1)), [w for w in range(16) if w != 7] + [7]]


def same(at, codes, S, K):
    ids, sc = expected(codes, S, K)
    for order in ORDERS:
        got, got_sc, _ = scan(at, codes, S, K, order)
        assert np.array_equal(got, ids) and np.array_equal(got_sc, sc), order


def near_limit(best, n, seed):
    """m = 8: the first `best` of the sample's 2048 items and every item behind it share the largest score"""
    rng = np.random.default_rng(seed)
    codes = rng.integers(0, 255, (n, 8), dtype=np.uint8)
    codes[rng.choice(2048, best, replace=False), 0] = 255
    codes[2048:, 0] = 255
    S = np.zeros((8, 256), np.float32)
    S[0] = rng.uniform(0.0, 0.9, 256)
    S[0, 255] = 1.0
    return codes, S


# the sample's bucket of the K-th best holds as many as are let be, one less and one more: waves that are ahead count into it while others still look at it
@pytest.mark.parametrize("K,best", [(1, 65), (1, 66), (1, 67), (10, 84)])
def test_whether_the_sample_is_taken_apart_is_one_decision(program, K, best):
    same(program, *near_limit(best, 5001, K + best), K)


# all scores alike: more keys than are ranked at once and no floor, so the lists' own range is taken; the words that gave the floor are written for it
@pytest.mark.parametrize("m,K", [(8, 32), (8, 100)])
def test_floor_of_the_waves_lists_is_read_before_it_is_written_over(program, m, K):
    rng = np.random.default_rng(K)
    codes = rng.integers(0, 256, (2500, m), dtype=np.uint8)
    same(program, codes, np.ones((m, 256), np.float32), K)


# bounds of every kind, in the stream (six units to a wave), lists that overflow among them
@pytest.mark.parametrize("m,dtype,b,n,K", [(8, np.uint8, 256, 12_345, 10), (8, np.uint8, 250, 12_345, 512), (64, np.uint8, 256, 6_000, 17), (8, np.uint16, 300, 6_000, 100)])
def test_bounds_that_are_exact_loose_or_useless(program, m, dtype, b, n, K):
    rng = np.random.default_rng(m + b + K)
    codes = rng.integers(0, b, (n, m)).astype(dtype)
    S = rng.standard_normal((m, b)).astype(np.float32)
    masked, far, deep = S.copy(), S.copy(), S.copy()
    masked[1, :b // 3] = -1e9
    far[2, 1] = 1e4
    deep[0, :-1] = -1e9
    for name, T in (("normal", S), ("uneven", S * np.where(np.arange(m) == 1, 50.0, 0.02)[:, None]), ("masked", masked), ("far entry", far), ("one entry of a split counts", deep), ("ties", np.round(S)),
                    ("zeros", 0 * S), ("negative", S - 20), ("offset", S + np.float32(1e7)), ("heavy tails", np.tan(np.pi * (rng.random(S.shape) - 0.5)))):
        ids, sc = expected(codes, T.astype(np.float32), K)
        got, got_sc, _ = scan(program, codes, T, K, rng.permutation(16))
        assert np.array_equal(got, ids) and np.array_equal(got_sc, sc), name
    rising = S.copy()
    rising[0] = np.arange(b) * 0.5
    codes[:, 0] = np.arange(n) * b // n
    same(program, codes, rising, K)


# most items far below the others, and of the sample fewer than twice K and 64 not among them: floors rise by what lies between the others all the same
def test_far_scores_do_not_keep_floors_from_rising(program):
    rng = np.random.default_rng(3)
    codes = rng.integers(0, 256, (120_000, 8), dtype=np.uint8)
    S = rng.standard_normal((8, 256)).astype(np.float32)
    S[4:6, np.arange(256) % 4 != 0] = -1e9
    ids, sc = expected(codes, S, 40)
    got, got_sc, (counted, _, _) = scan(program, codes, S, 40, [])
    assert np.array_equal(got, ids) and np.array_equal(got_sc, sc)
    assert counted <= 2048 + 1000, counted                     # (the sample; 7500 items are not masked)


# of two scores the larger one is an eighth of the items': taking it apart leaves nothing to tell, and that score is the floor
def test_taking_ties_apart_keeps_the_floor(program):
    rng = np.random.default_rng(4)
    codes = rng.integers(0, 256, (20_000, 64), dtype=np.uint8)
    S = np.zeros((64, 256), np.float32)
    S[0, :32] = 100.0
    ids, sc = expected(codes, S, 20)
    got, got_sc, (_, scored, _) = scan(program, codes, S, 20, [])
    assert np.array_equal(got, ids) and np.array_equal(got_sc, sc)
    assert scored <= 4 * (1024 + 20_000 // 4), scored          # (a row's four vectors; the sample, and who passes)


# all scores alike: a list that is full of them takes no more, whichever waves are ahead
@pytest.mark.parametrize("K", [10, 100])
def test_ties_beyond_a_full_list_are_not_taken(program, K):
    rng = np.random.default_rng(5)
    codes = rng.integers(0, 256, (100_000, 8), dtype=np.uint8)
    S = np.ones((8, 256), np.float32)
    ids, sc = expected(codes, S, K)
    for order in ORDERS + [[]]:
        got, got_sc, (counted, _, _) = scan(program, codes, S, K, order)
        assert np.array_equal(got, ids) and np.array_equal(got_sc, sc), order
        assert counted <= 60_000, counted                      # (the sample, a list of every wave, and the selection from these)


# more keys in the waves' lists than are ranked at once, and a range that tells them apart no further (a far score, ties): narrowed down by their bits, not sorted
@pytest.mark.parametrize("K", [512])
@pytest.mark.parametrize("name", ["one entry +1e4", "few values", "negative"])
def test_many_keys_in_few_buckets_are_narrowed_down(program, name, K):
    rng = np.random.default_rng(6)
    codes = rng.integers(0, 256, (20_000, 8), dtype=np.uint8)
    S = rng.standard_normal((8, 256)).astype(np.float32)
    if name == "few values":
        S = np.round(0.3 * S)
    if name == "negative":
        S -= 30.0
        S[1:] *= np.float32(1e-7)
    codes[7, 4] = 17
    S[4, 17] += 1e4
    ids, sc = expected(codes, S, K)
    got, got_sc, (_, _, barriers) = scan(program, codes, S, K, [])
    assert np.array_equal(got, ids) and np.array_equal(got_sc, sc)
    assert barriers <= 90, barriers


# scores that rise along the first quarter of the catalogue, where bounds dismiss nothing, and are low in the rest: waves that went on without bounds come back
def test_waves_come_back_to_their_bounds(program):
    rng = np.random.default_rng(7)
    codes = rng.integers(0, 256, (400_000, 8), dtype=np.uint8)
    S = rng.standard_normal((8, 256)).astype(np.float32)
    S[0] = np.arange(256)
    codes[:100_000, 0] = 1 + np.arange(100_000) * 255 // 100_000
    codes[100_000:, 0] = 0
    ids, sc = expected(codes, S, 10)
    got, got_sc, (_, scored, _) = scan(program, codes, S, 10, [])
    assert np.array_equal(got, ids) and np.array_equal(got_sc, sc)
    assert scored <= 120_000, scored                           # (of 200,000 code vectors)
