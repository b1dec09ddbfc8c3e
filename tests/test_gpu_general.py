"""The general middle-row kernel with eight waves (more than 256 states, or 128 in fp32, outside the specialised shapes): chunks
joined after the plan, full-width rows apart or in its launch, and positions of their own."""

import numpy as np
import pytest
import torch

import oracle.fourier_kv as fk
from fa_testlib import GENERAL_CALLS, rows_pad8, rows_to_tok8, to_dev
from workloads.synth import rel_err, round_to_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", GENERAL_CALLS, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("per_sequence", [False, True])
def test_general_kernel_matches_oracle(call, per_sequence):
    import paper_2506_11886_amd as fa
    dt, B, H, G, D, Dkc, Dvc, M, N, W = call
    print(f"[case] general {call} per_sequence {per_sequence}", flush=True)
    rng = np.random.default_rng(M + N)
    tt = torch.float32 if dt == "f32" else torch.bfloat16
    draw = lambda *s: (lambda a: a if dt == "f32" else round_to_bf16(a))(rng.standard_normal(s).astype(np.float32))
    q, kk, vk, kf, vf = draw(B, H * G, D), draw(B, H, N, D - Dkc), draw(B, H, N, D - Dvc), draw(B, H, W, D), draw(B, H, W, D)
    ck = (np.sqrt(N / M) * rng.standard_normal((B, H, M, Dkc))).astype(np.float32)
    cv = (np.sqrt(N / M) * rng.standard_normal((B, H, M, Dvc))).astype(np.float32)
    masks = []
    for dc in (Dkc, Dvc):
        m = np.zeros((B, H, D), np.uint8)
        np.put_along_axis(m, rng.random((B, H, D)).argsort(-1)[..., :dc], 1, -1)
        masks.append(m)
    seq_n, seq_w = np.full(B, N), np.full(B, W)
    if per_sequence:
        seq_n, seq_w = rng.integers(0, N + 1, B), rng.integers(0, W + 1, B)
        seq_n[:3], seq_w[:3] = (N, 0, 1), (W, W, 0)
    args = (to_dev(q, dtype=tt), to_dev(ck), to_dev(masks[0]), to_dev(cv), to_dev(masks[1]), M, N, 0, N)
    tail = (to_dev(rows_pad8(kk), dtype=tt), to_dev(rows_to_tok8(vk), dtype=tt))
    full = (to_dev(kf, dtype=tt), to_dev(vf, dtype=tt)) if W else (None, None)
    lists = [to_dev(x.astype(np.int32)) for x in (seq_n, seq_w)]
    if per_sequence:
        out = fa.fa_decode_varlen(*args, lists[0], *tail, *full, lists[1] if W else None)
    else:
        out = fa.fa_decode(*args, *tail, *full)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert np.isfinite(out).all()
    for b, h in {(0, 0), (1, H - 1), (2, 0), (B - 1, H // 2)}:
        n, w = int(seq_n[b]), int(seq_w[b])
        got = out[b, h * G:(h + 1) * G]
        if n + w == 0:
            assert not got.any()
            continue
        want = fk.decode_head_group(q[b, h * G:(h + 1) * G], ck[b, h].astype(np.float64), masks[0][b, h], cv[b, h].astype(np.float64), masks[1][b, h],
                                    N, 0, n, kk[b, h, :n], vk[b, h, :n], kf[b, h, :w], vf[b, h, :w])
        assert rel_err(got, want) <= (1e-5 if dt == "f32" else 2e-3), (b, h, n, w, rel_err(got, want))
