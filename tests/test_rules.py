"""Which kernel a call gets (no GPU): the rules are compiled for the host alone and asked."""

import os
import random

import pytest

import test_gpu_rows
from fa_testlib import APPEND_CALLS, GENERAL_CALLS, HIPCC, HOST_ONLY, ROWS_CALLS, host_program

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")

# a line: dtype B Hkv G D Dkc Dvc M T N W per_sequence -> waves of the general middle-row kernel (0: another form), full-width rows
# apart, chunks as planned, chunks as run, C_k by single floats
DECODE = HOST_ONLY + r"""
#include "fa_decode.hip"
int main() {
  int dt, B, Hkv, G, D, Dkc, Dvc, M, T, N, W, seq;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d", &dt, &B, &Hkv, &G, &D, &Dkc, &Dvc, &M, &T, &N, &W, &seq) == 12) {
    fa::DecodePlan pl{};
    const bool ok = fa::make_plan(pl, dt, B, Hkv * G, Hkv, D, Dkc, Dvc, M, N, W, 0);
    if (ok) fa::make_local(pl, dt, B, Hkv * G, Hkv, D, Dkc, Dvc, N, W, 0, fa::local_form(M, T));
    const int planned = pl.Sm;
    if (ok) fa::join_chunks(pl, dt, B, Hkv, N, seq != 0);
    std::printf("%d %d %d %d %d\n", !ok || pl.local.use || pl.fused || pl.fast ? 0 : pl.nw, pl.rides, planned, pl.Sm,
                fa::prepare_by_floats(B * Hkv, G, Dkc, M));
  }
}
"""


@pytest.fixture(scope="module")
def decode(tmp_path_factory):
    return host_program(tmp_path_factory.mktemp("decode"), DECODE, ["fa_local.hip"])


def _call(c, per_sequence=0):
    dt, B, Hkv, G, D, Dkc, Dvc, M, N, W = c
    return (0 if dt == "f32" else 1, B, Hkv, G, D, Dkc, Dvc, M, N, N, W, per_sequence)


def test_general_calls_are_what_they_say(decode):
    """The shapes of test_gpu_general.py reach the kernel with eight waves, two of them with joined chunks."""
    rows = decode([_call(c) for c in GENERAL_CALLS])
    assert all(r[0] == 8 for r in rows), rows
    assert all(r[3] < r[2] for r in rows[:2]) and all(r[3] == r[2] for r in rows[2:]), rows
    assert rows[1][1] == 1, rows


def test_chunks_are_joined_neither_in_fp32_nor_per_sequence(decode):
    """Joined chunks add more rows up in fp32, and wait for the longest sequence."""
    rng = random.Random(5)
    calls = []
    for _ in range(4000):
        M = rng.randint(130, 1024)
        N = max(M, int(2 ** rng.uniform(9, 14.2)))
        calls.append((rng.choice([0, 1]), rng.choice([4, 8, 16, 20]), rng.choice([4, 8, 16]), rng.choice([1, 4, 6, 16]), rng.choice([64, 128]), 40, 30,
                      M, N, N, 0, rng.choice([0, 1])))
    joined = [0, 0]
    for c, r in zip(calls, decode(calls)):
        if r[0] == 8:
            free = c[0] == 1 and not c[-1]
            joined[free] += r[3] < r[2]
    assert joined[0] == 0 and joined[1] > 20, joined


def test_full_width_rows_go_apart_where_that_is_faster(decode):
    """Beside the coefficients: many heads, or more workgroups than units.  In the launch of the middle rows: few heads in one round, fewer
    than four compressed K dims, and at head dim 256 few heads or many pairs."""
    calls = {(1, 1, 8, 1, 128, 96, 64, 343, 2359, 2359, 2442, 0): 0, (1, 1, 8, 6, 128, 96, 64, 343, 2359, 2359, 2442, 0): 1,
             (1, 16, 16, 1, 128, 96, 64, 343, 900, 900, 132, 0): 1, (1, 1, 8, 6, 128, 3, 64, 343, 2359, 2359, 2442, 0): 0,
             (1, 8, 16, 6, 256, 192, 192, 622, 700, 700, 205, 0): 0, (1, 2, 4, 16, 256, 192, 192, 622, 700, 700, 205, 0): 1,
             (1, 2, 4, 1, 256, 192, 192, 622, 700, 700, 205, 0): 0}
    got = decode(list(calls))
    assert all(r[0] == 8 for r in got) and [r[1] for r in got] == list(calls.values()), got


def test_coefficients_by_floats(decode):
    """Fewer than four dims; few states of many heads with a vector or two a row, or a few of them and few pairs.  Never rows of whole vectors."""
    of = lambda pairs, G, Dkc, M: decode([(1, 1, pairs, G, 128, Dkc, 64, M, 200, 200, 0, 0)])[0][4]
    assert [of(4, 1, 3, 128), of(4, 8, 5, 40), of(20, 12, 7, 63), of(6, 12, 30, 20)] == [1] * 4
    assert [of(4, 8, 4, 40), of(4, 4, 5, 40), of(4, 8, 5, 64), of(200, 16, 5, 40), of(40, 16, 30, 20), of(6, 8, 30, 20), of(6, 16, 33, 20), of(6, 16, 28, 20)] == [0] * 8


# a line: pairs D -> head dims of a workgroup of fa_append
APPEND = HOST_ONLY + r"""
#include "fa_append.hip"
int main() {
  int pairs, D;
  while (std::scanf("%d %d", &pairs, &D) == 2) std::printf("%d\n", fa::append_dims(pairs, D));
}
"""


def test_append_slices(tmp_path):
    """The calls of test_gpu_append.py are in slices of the width they say; few pairs and heads that would not fill wide slices are not."""
    ask = host_program(tmp_path, APPEND, [])
    assert [r[0] for r in ask([(c[0] * c[1], c[2]) for c in APPEND_CALLS])] == [c[-1] for c in APPEND_CALLS]
    rng = random.Random(3)
    calls = [(int(2 ** rng.uniform(0, 12)), 8 * rng.randint(1, 32)) for _ in range(500)]
    for (pairs, D), (dims,) in zip(calls, ask(calls)):
        assert dims == 16 or dims < 2 * D
        assert dims == 16 or 2 * pairs * -(-D // 16) >= 1400


# The library's own entry points with the launches noted down instead of made.  A line: entry (0 fa_compress, 1 fa_compress_kv, 2 fa_select_dims)
# dtype B H N D Dkc Dvc M T t0 accumulate layout keep_offset with_keep sx_n workspace (0: what the query says) -> status, then for each launch
# the kernel, grid x y z, threads, and hw and chunks of project_rows, -1 and the blocks of fa_expand (-1 else)
ROUTES = r"""
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <cxxabi.h>
#include "fa_rows.hpp"
static std::map<const void*, std::string>& names() { static std::map<const void*, std::string> m; return m; }
static dim3 g_, b_;
extern "C" {
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  char* d = abi::__cxa_demangle(name, nullptr, nullptr, nullptr);
  std::string s = d ? d : name;
  s = s.substr(s.find("fa::") + 4);
  names()[f] = s.substr(0, s.find_first_of("<("));
}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) { g_ = g; b_ = b; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* n, hipStream_t* st) { *g = g_; *b = b_; *n = 0; *st = nullptr; return hipSuccess; }
hipError_t hipPeekAtLastError() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
  const std::string& n = names()[f];
  const bool rows = n == "project_rows";
  const fa::RowsParams* p = static_cast<const fa::RowsParams*>(args[0]);
  std::printf("%s %u %u %u %u %d %d ", n.c_str(), g.x, g.y, g.z, b.x, rows ? p->hw : -1, rows ? (p->part ? int(g.z) : 1) : n == "fa_expand" ? static_cast<const fa::MomentParams*>(args[0])->blocks : -1);
  return hipSuccess;
}
}
int main() {
  int e, dt, B, H, N, D, Dk, Dv, M, T, t0, acc, lay, off, keep;
  long sx; size_t bytes;
  while (std::scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %ld %zu", &e, &dt, &B, &H, &N, &D, &Dk, &Dv, &M, &T, &t0, &acc, &lay, &off, &keep, &sx, &bytes) == 17) {
    char* at = reinterpret_cast<char*>(1 << 20);   // (nothing is read through it)
    if (!bytes) bytes = e == 0 ? fa_compress_workspace_bytes_for(dt, B, H, N, D, Dk, M) : e == 1 ? fa_compress_kv_workspace_bytes_for(dt, B, H, N, D, Dk, Dv, M)
                                                                                  : fa_select_workspace_bytes(dt, B, H, N, D, M);
    const auto mask = reinterpret_cast<uint8_t*>(at);
    const auto c = reinterpret_cast<float*>(at);
    void* k = keep ? at : nullptr;
    int st;
    if (e == 0) st = fa_compress(at, dt, sx * N * H, sx * N, sx, B, H, N, D, mask, Dk, M, T, t0, acc, c, k, lay, 0, off, at, bytes, nullptr);
    else if (e == 1) st = fa_compress_kv(at, at, dt, sx * N * H, sx * N, sx, B, H, N, D, mask, Dk, mask, Dv, M, T, t0, acc, c, c, k, 0, k, 0, off, at, bytes, nullptr);
    else st = fa_select_dims(at, dt, sx * N * H, sx * N, sx, B, H, N, D, M, Dk, mask, c, at, bytes, nullptr);
    std::printf("%d\n", st);
  }
}
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    ask = host_program(tmp_path_factory.mktemp("routes"), ROUTES, ["fa_compress.hip", "fa_moments.hip", "fa_rows.hip", "fa_select.hip"])

    def launches(calls):
        """Each call's launches: (kernel, grid, threads, hw, chunks or blocks)."""
        out = []
        for row in ask(calls):
            assert row[-1] == 0, row
            out.append([(r[0], r[1:4], r[4], r[5], r[6]) for r in (row[i:i + 7] for i in range(0, len(row) - 1, 7))])
        return out
    return launches


def _compress(dt, B, H, N, D, Dc, M, T=0, t0=0, acc=0, layout=0, off=0, keep=1, Dv=None):
    return (0 if Dv is None else 1, 0 if dt == "f32" else 1, B, H, N, D, Dc, Dv or 0, M, T or max(N, M), t0, acc, layout, off, keep, D, 0)


def test_rows_calls_are_what_they_say(routes):
    """The calls of test_gpu_rows.py reach project_rows with the tiles and chunks they name (the mean alone: but for a pair)."""
    calls = [_compress(dt, 1, H, N, D, Dk, M, T, T - N, 1, 0, off, 1, Dv) for dt, H, N, D, Dk, Dv, M, T, off, _, _ in ROWS_CALLS]
    for c, got in zip(ROWS_CALLS, routes(calls)):
        assert (got[0][0], *got[0][3:]) == ("project_rows", *c[-2:]), (c, got)
        assert len(got) == (2 if c[-1] > 1 else 1), (c, got)
    for D, N, M, T, t0, off, Dc in test_gpu_rows.CASES:
        for dt in ("bf16", "f32"):
            got = routes([_compress(dt, 1, 3, N, D, Dc, M, T, t0, 1, layout, off) for layout in (0, 1)])
            assert [g[0][0] for g in got] == ["compress_project" if M == 1 else "project_rows"] * 2, (D, N, M, got)


def test_rows_are_taken_where_they_are_faster(routes):
    """The mean alone, fp32 with at most half of the dims compressed, one column group at head dim 256: by the estimates.  fp32 with more, and short bf16 segments of more
    states: always, closer and faster but for a few."""
    direct = [_compress("f32", 4, 8, 3410, 64, 7, 1, 3417, 4, 1, 0, 8, 1, 60), _compress("f32", 2, 4, 11135, 128, 25, 1, layout=1, off=8),
              _compress("bf16", 3, 8, 1, 256, 232, 1, 3, 2, 1), _compress("bf16", 6, 3, 42, 128, 121, 1, 126, 9, 0, 1, 3),
              _compress("f32", 1, 16, 34532, 128, 18, 1006, 37016, 952, 1, 1, 8), _compress("f32", 25, 2, 10658, 128, 13, 510, acc=1, Dv=13),
              _compress("bf16", 2, 32, 1378, 256, 29, 992, 1386, 2, 0, 0, 8), _compress("bf16", 28, 16, 920, 256, 72, 751, layout=1)]
    for c, got in zip(direct, routes(direct)):
        assert got[0][0] == "compress_project", (c, got)
    rng = random.Random(7)
    calls = []
    for _ in range(3000):
        dt, D = rng.choice(["f32", "bf16"]), rng.choice([64, 128, 256])
        N = int(2 ** rng.uniform(1, 15 if dt == "f32" else 9))
        M = max(2, min(N, int(2 ** rng.uniform(1, 10))))
        Dc = rng.randint(D // 2 + 1 if dt == "f32" else 1, D)
        calls.append(_compress(dt, 1, int(2 ** rng.uniform(0, 8)), N, D, Dc, M, layout=rng.choice([0, 1]), off=rng.choice([0, 3]),
                               Dv=rng.choice([None, rng.randint(1, D)])))
    for c, got in zip(calls, routes(calls)):
        assert got[0][0] == "project_rows", (c, got)


def test_selection_shares_the_blocks(routes):
    """fa_expand: eight shares of 64 blocks or more for fewer workgroups than compute units, else four, and twelve waves at most."""
    rng = random.Random(9)
    calls = []
    for _ in range(1500):
        D, N = rng.choice([64, 128, 256]), int(2 ** rng.uniform(9, 16))
        calls.append((2, 1, 1, int(2 ** rng.uniform(0, 8)), N, D, D // 2, 0, max(1, min(N // 8, int(2 ** rng.uniform(0, 9)))), N, 0, 0, 0, 0, 0, D, 0))
    most = {}
    for got in routes(calls):
        for name, grid, threads, _, blocks in got:
            if name == "fa_expand":
                key = "many" if grid[0] * grid[1] * grid[2] >= 256 else "long" if blocks >= 64 else "short"
                most[key] = max(most.get(key, 0), threads // 64)
    assert most == {"many": 12, "long": 8, "short": 4}
