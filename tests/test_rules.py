"""Which kernel a call gets (no GPU): the rules are compiled for the host alone and asked."""

import os
import random

import pytest

from fa_testlib import APPEND_CALLS, GENERAL_CALLS, HIPCC, HOST_ONLY, host_program

pytestmark = pytest.mark.skipif(not os.path.exists(HIPCC), reason="no hipcc")

# a line: dtype B Hkv G D Dkc Dvc M T N W per_sequence -> waves of the general middle-row kernel (0: another form), full-width rows
# apart, chunks as planned, chunks as run
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
    std::printf("%d %d %d %d\n", !ok || pl.local.use || pl.fused || pl.fast ? 0 : pl.nw, pl.rides, planned, pl.Sm);
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
