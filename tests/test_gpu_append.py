"""fa_append and fa_append_varlen in slices of 32 and 64 head dims, which many (sequence, head) pairs take."""

import pytest
import torch

from fa_testlib import APPEND_CALLS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", APPEND_CALLS, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("per_sequence", [False, True])
def test_append_wide_slices(call, per_sequence):
    """One fold: states against fp64, kept dims, ring rows and everything that is not written bit for bit.  With lists one sequence is left
    alone, one only stores its token."""
    import paper_2506_11886_amd as fa
    B, H, D, Dkc, Dvc, M, dtype, _ = call
    print(f"[case] append {call} per_sequence {per_sequence}", flush=True)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    W, cap, T = 7, 50, 5003
    g = torch.Generator(device="cuda").manual_seed(D + M)
    draw = lambda *s: torch.randn(s, generator=g, device="cuda").clamp(-5.0, 5.0)
    slot, n = torch.full((B,), 4, dtype=torch.int32), torch.full((B,), 41, dtype=torch.int32)
    if per_sequence:
        slot = (torch.arange(B) % W).to(torch.int32)
        n = (torch.arange(B) * 11 % cap).to(torch.int32)
        slot[1], n[2] = -1, -1
    new, rows, masks, C0 = [], [], [], []
    for dc in (Dkc, Dvc):
        new.append(draw(B, H, D).to(dt))
        rows.append(draw(B, H, W, D).to(dt))
        masks.append((torch.rand((B, H, D), generator=g, device="cuda").argsort(-1) < dc).to(torch.uint8))
        C0.append(draw(B, H, M, dc))
    kk = torch.full((B, H, cap, fa.keep_rows_pitch(D - Dkc)), 3.0, dtype=dt, device="cuda")
    vk = torch.full((B, H, fa.tok8_numel(cap, D - Dvc)), 3.0, dtype=dt, device="cuda")
    full, C = [r.clone() for r in rows], [c.clone() for c in C0]
    keep = (kk if D > Dkc else None, vk if D > Dvc else None)
    if per_sequence:
        fa.fa_append_varlen(*new, *full, slot.cuda(), *masks, M, T, n.cuda(), cap, *C, *keep)
    else:
        fa.fa_append(*new, *full, 4, True, *masks, M, T, 41, *C, *keep, kk_stride_bh=kk.stride(1), vk_stride_bh=vk.stride(1))
    torch.cuda.synchronize()

    order = torch.arange(M, dtype=torch.int64)
    ang = 2.0 * torch.pi * (((order + 1) // 2).view(1, -1) * n.view(-1, 1).long() % T).double() / T
    phi = torch.where((order % 2 == 1) | (order == 0), ang.cos(), ang.sin()).cuda()
    folds = (slot >= 0) & (n >= 0)
    for i in range(2):
        want_rows, want, want_keep = rows[i].clone(), C0[i].double(), torch.full((B, H, cap, D - (Dkc, Dvc)[i]), 3.0, dtype=dt, device="cuda")
        for b in range(B):
            if slot[b] < 0:
                continue
            old, m = rows[i][b, :, slot[b]], masks[i][b].bool()
            want_rows[b, :, slot[b]] = new[i][b]
            if folds[b]:
                want[b] += phi[b].view(1, -1, 1) * old[m].double().view(H, 1, -1)
                want_keep[b, :, n[b]] = old[~m].view(H, -1)
        assert torch.equal(full[i], want_rows)
        assert torch.equal(C[i][~folds], C0[i][~folds])
        # |C|, |x| <= 5.  Basis value: the turn is rounded to 2^-24, times pi, and sincospi adds 1.5 ulp: 2.8e-7, times |x|;
        # the sum (below 16) is rounded by half of 2^-20
        if C[i].numel():
            assert (C[i].double() - want).abs().max().item() <= 1.4e-6 + 4.8e-7 + 1e-7
        got = kk[..., :D - Dkc] if i == 0 else fa.keep_rows_from_tok8(vk, cap, D - Dvc)
        assert torch.equal(got, want_keep)
