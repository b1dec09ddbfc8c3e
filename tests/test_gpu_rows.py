"""The projection whose basis is formed per token (fp32, short bf16 segments, fast harmonics): edges of steps, harmonic tiles, column
halves and groups of eight, tiles per workgroup and chunks of tokens.  Which calls of CASES and ROWS_CALLS it serves is asked in
test_rules.py; the mean alone (M = 1) of one tensor and slow harmonics of long bf16 segments take other forms, held to the same here."""

import numpy as np
import pytest
import torch

import oracle.fourier_kv as fk
from fa_testlib import ROWS_CALLS, rows_to_tok8, to_dev
from workloads.synth import rel_err, round_to_bf16

pytestmark = pytest.mark.gpu


def _segment(D, N, Dc, H, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((1, H, N, D)) + 0.5
    mask = np.zeros((1, H, D), np.uint8)
    for h in range(H):
        mask[0, h, rng.choice(D, Dc, replace=False)] = 1
    return round_to_bf16(x.astype(np.float32)), mask


# D, N, M, T, t0, token offset of the kept dims, compressed dims
CASES = [
    (128, 1, 1, 7, 5, 0, 128),            # one row, the mean alone, nothing kept
    (128, 1, 3, 9000, 8191, 5, 100),      # one row inside a group of eight
    (128, 31, 32, 40, 0, 0, 96),          # less than a step, one tile less its last sine
    (128, 33, 33, 33, 0, 3, 1),           # one row past a step, a tile and no more, one column
    (64, 257, 35, 300, 11, 6, 41),        # one row past eight steps, one harmonic past a tile
    (64, 512, 512, 512, 0, 0, 64),        # as many states as rows, twice the last order is the period
    (256, 129, 66, 4000, 100, 8, 179),    # both column halves
    (256, 700, 300, 701, 1, 2, 7),        # two terms
    (128, 513, 171, 600, 87, 0, 91),      # the first length with two terms
]


@pytest.mark.parametrize("D,N,M,T,t0,off,Dc", CASES + [(128, 9000, 40, 9000, 0, 4, 90), (256, 3001, 70, 3500, 11, 1, 200)])
@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
def test_rows_projection_matches_oracle(D, N, M, T, t0, off, Dc, layout, dt):
    import paper_2506_11886_amd as fa
    print(f"[case] rows {dt} D{D} N{N} M{M} T{T} t0 {t0} off {off} Dc{Dc} layout {layout}", flush=True)
    x, mask = _segment(D, N, Dc, 3, N + M)
    if dt == torch.float32:      # (all 24 bits of a value)
        x = x * np.float32(1.2345678)
    want, keep = fk.compress_batched(x, mask, M, T, t0)
    Du = D - Dc
    prev = torch.randn((1, 3, M, Dc), device="cuda")
    shape = (1, 3, off + N, fa.keep_rows_pitch(Du)) if layout == fa.FA_KEEP_ROWS else (1, 3, fa.tok8_numel(off + N, Du))
    slab = torch.full(shape, 7.0, dtype=dt, device="cuda")
    c, _ = fa.fa_compress(to_dev(x, dtype=dt), to_dev(mask), Dc, M, T, t0, True, prev.clone(), slab, layout, off)
    torch.cuda.synchronize()
    # 2^-17 of a basis value's size at two terms, fp32 at three; a state sums N values of size 1
    tol = 2e-5 if N > 512 and dt == torch.bfloat16 else 2e-6
    assert rel_err(c.cpu().numpy(), want + prev.cpu().numpy().astype(np.float64), np.sqrt(N)) <= tol
    if Du:
        if layout == fa.FA_KEEP_ROWS:
            got = slab.float().cpu().numpy()
            assert np.array_equal(got[:, :, off:, :Du], keep.astype(np.float32)) and not got[:, :, off:, Du:].any()
            assert (got[:, :, :off] == 7.0).all()
        else:
            got = fa.keep_rows_from_tok8(slab, off + N, Du).float().cpu().numpy()
            assert np.array_equal(got[:, :, off:], keep.astype(np.float32)) and (got[:, :, :off] == 7.0).all()


@pytest.mark.parametrize("D,B,N,M,Dkc,Dvc", [(128, 70, 290, 90, 96, 101), (64, 40, 300, 150, 40, 64), (256, 20, 300, 64, 200, 150),
                                             (128, 2, 6001, 40, 96, 101)])
@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float32])
def test_rows_projection_of_a_pair(D, B, N, M, Dkc, Dvc, dt):
    """Enough pairs that a workgroup takes several harmonic tiles, or few of them and fp32 tokens in chunks; rows of a wider tensor."""
    import paper_2506_11886_amd as fa
    print(f"[case] rows pair D{D} B{B} N{N} M{M} {Dkc}/{Dvc}", flush=True)
    k, kmask = _segment(D, N, Dkc, B, 1)
    v, vmask = _segment(D, N, Dvc, B, 2)
    wide = lambda a: torch.nn.functional.pad(to_dev(a, dtype=dt), (0, 8))[..., :D]
    ck, kk, cv, vk = fa.fa_compress_kv(wide(k), wide(v), to_dev(kmask), to_dev(vmask), Dkc, Dvc, M, N + 100, t0=50)
    torch.cuda.synchronize()
    for x, mask, c in ((k, kmask, ck), (v, vmask, cv)):
        want, keep = fk.compress_batched(x, mask, M, N + 100, 50)
        assert rel_err(c.cpu().numpy(), want, np.sqrt(N)) <= (2e-5 if N > 512 and dt == torch.bfloat16 else 2e-6)
        if x is k:
            assert np.array_equal(kk[..., :D - Dkc].float().cpu().numpy(), keep.astype(np.float32))
        else:
            assert np.array_equal(vk.float().cpu().numpy(), rows_to_tok8(keep.astype(np.float32)))


@pytest.mark.parametrize("D,N,M", [(128, 300, 100), (64, 64, 64), (256, 1025, 130), (128, 33, 1), (128, 2000, 500)])
def test_rows_selection_matches_oracle(D, N, M):
    import paper_2506_11886_amd as fa
    print(f"[case] rows select D{D} N{N} M{M}", flush=True)
    x, _ = _segment(D, N, D // 2, 2, 3)
    mask, mse = fa.fa_select_dims(to_dev(x, dtype=torch.bfloat16), M, D // 2)
    torch.cuda.synchronize()
    for h in range(2):
        want = fk.reconstruction_mse(x[0, h], M)
        scale = np.mean(x[0, h].astype(np.float64) ** 2, axis=0)
        # a difference of sums of the energy's size, each of fp32 precision
        assert np.all(np.abs(mse[0, h].cpu().numpy() - want) <= 5e-6 * scale)
        assert int(mask[0, h].sum()) == D // 2


@pytest.mark.parametrize("call", ROWS_CALLS, ids=lambda c: "-".join(map(str, c)))
def test_rows_forms_match_oracle(call):
    """Tiles per workgroup and chunks of tokens (what each call gets is asked in test_rules.py), onto states that are there already."""
    import paper_2506_11886_amd as fa
    dt, H, N, D, Dkc, Dvc, M, T, off, hw, chunks = call
    print(f"[case] rows form {call}", flush=True)
    tt = torch.float32 if dt == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(N + M)
    sides = []
    for dc in (Dkc,) if Dvc is None else (Dkc, Dvc):
        x, mask = _segment(D, N, dc, H, N + dc)
        if dt == "f32":
            x = x * np.float32(1.2345678)
        sides.append((x, mask, torch.randn((1, H, M, dc), generator=g, device="cuda"), dc))
    kk = torch.full((1, H, off + N, fa.keep_rows_pitch(D - Dkc)), 7.0, dtype=tt, device="cuda")
    states = [s[2].clone() for s in sides]
    if Dvc is None:
        fa.fa_compress(to_dev(sides[0][0], dtype=tt), to_dev(sides[0][1]), Dkc, M, T, T - N, True, states[0], kk, fa.FA_KEEP_ROWS, off)
    else:
        vk = torch.full((1, H, fa.tok8_numel(off + N, D - Dvc)), 7.0, dtype=tt, device="cuda")
        fa.fa_compress_kv(*(to_dev(s[0], dtype=tt) for s in sides), *(to_dev(s[1]) for s in sides), Dkc, Dvc, M, T, t0=T - N, accumulate=True,
                          ck=states[0], cv=states[1], k_keep=kk, v_keep=vk, keep_offset=off)
    torch.cuda.synchronize()
    # a state sums N values of size 1; a basis value of two terms is off by 2^-18 of its size at most, of three by fp32 rounding
    tol = 4e-6 if N > 512 and dt == "bf16" else 2e-6
    for i, (x, mask, prev, dc) in enumerate(sides):
        for h in {0, H // 2, H - 1}:
            want, keep = fk.compress_batched(x[:, h:h + 1], mask[:, h:h + 1], M, T, T - N)
            err = rel_err(states[i][:, h].cpu().numpy(), want[:, 0] + prev[:, h].cpu().numpy().astype(np.float64), np.sqrt(N))
            assert err <= tol, (i, h, err)
            got = kk[:, h:h + 1, :, :D - dc] if i == 0 else fa.keep_rows_from_tok8(vk[:, h:h + 1], off + N, D - dc)
            assert np.array_equal(got[:, :, off:].float().cpu().numpy(), keep.astype(np.float32)) and (got[:, :, :off] == 7.0).all()


def test_rows_infinity_stays_in_its_column():
    import paper_2506_11886_amd as fa
    x, mask = _segment(128, 200, 90, 2, 5)
    d = int(np.flatnonzero(mask[0, 1])[4])
    x[0, 1, 77, d] = np.inf
    c, _ = fa.fa_compress(to_dev(x, dtype=torch.bfloat16), to_dev(mask), 90, 60, 200, 0)
    c = c.cpu().numpy()
    assert not np.isfinite(c[0, 1, :, 4]).any() and np.isfinite(c).sum() == c.size - 60
