"""The calls a serving program makes on this library, at the sizes it makes them at.

A case is one pass through the public entry points of `paper_2506_11886_amd`, with the buffers a
program keeps between passes (caches, states, outputs, workspaces) already in hand:

  decode      fa_decode                            one new token, cache untouched
  step        fa_append + fa_decode                one whole decode step of one batch
  serve       fa_append_varlen + fa_decode_varlen  the same, every sequence at its own position
  verify      fa_decode_mq                         several drafted tokens at once
  prefill     fa_compress_kv                       the middle of a prompt, K and V, in one go
  chunk       fa_compress(accumulate) of K, of V   one more piece of a chunked prefill
  calibrate   fa_select_dims                       which head dims to compress, per head

Fields: B sequences, Hkv KV heads with G query heads each, D head dim, N middle tokens (full-width
rows besides: 4 sink tokens and a window of W - 4), Dkc / Dvc compressed K / V dims, M states per
dim, T basis period, dtype.  Signals follow the repository's synthetic caches: a compressed dim is
three in-band tones and a little noise, everything else is white.
"""

import math

import torch

import paper_2506_11886_amd as fa

SINK = 4        # sink rows in front of the window ring
RING = 32       # decode steps after which a pass starts again at the first position


def _case(kind, **kw):
    c = {"kind": kind, "B": 1, "Hkv": 8, "G": 4, "D": 128, "W": 0, "Dkc": 96, "Dvc": 96, "dtype": "bf16"}
    c.update(kw)
    return c


def listed():
    return [
        # the smallest cache of the configurations, fp32: a call that is all latency
        _case("decode", name="decode_tiny_f32", Hkv=1, D=64, N=380, W=132, Dkc=48, Dvc=48, M=32, T=380, dtype="f32"),
        # the ordinary decode step: one sequence, 32 K tokens, grouped heads; the token that leaves the window
        # is folded, the new one stored, then attention
        _case("step", name="step_32k", N=31740, W=1028, M=256, T=31740 + RING),
        # the largest single-sequence context
        _case("decode", name="decode_128k", N=129020, W=2052, Dkc=112, Dvc=112, M=512, T=129020),
        # one query head per KV head, a small batch
        _case("decode", name="decode_mha_8x4k", B=8, Hkv=32, G=1, N=4096, W=516, M=256, T=4096),
        # batched serving: sixteen sequences that stand anywhere between a quarter of and all of 8 K tokens
        _case("serve", name="serve_16x8k", B=16, N=7676, W=516, M=128, T=7676 + RING),
        # the state count of the paper's own setting at its 32 K context
        _case("decode", name="decode_m1023_32k", N=31740, W=1028, M=1023, T=31740),
        # eight query heads per KV head, counts that divide nothing, a period longer than the segment
        _case("decode", name="decode_gqa8_ragged", B=3, G=8, N=5003, W=304, Dkc=91, Dvc=101, M=130, T=9001),
        # four drafted tokens checked at once
        _case("verify", name="verify_4x32k", Tq=4, N=31740, W=1028, M=256, T=31740),
        # prompts: ordinary and largest
        _case("prefill", name="prefill_32k", N=31740, M=256, T=31740),
        _case("prefill", name="prefill_128k", N=129020, Dkc=112, Dvc=112, M=512, T=129020),
        # an eighth 2 K piece of a chunked prefill; the sink tokens shift every later piece by four rows
        _case("chunk", name="chunk_2k_of_32k", N=2048, t0=7 * 2048 - SINK, M=256, T=31740),
        # calibration of one layer's K cache
        _case("calibrate", name="calibrate_32k", N=31740, M=256, T=31740),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _dims(rng, D):
    """Compressed dims of one side: three fifths to nine tenths of the head, mostly in eights."""
    n = rng.uniform(0.62, 0.9) * D
    return int(n // 8) * 8 if rng.random() < 0.6 else int(n)


def draw(rng):
    kind = rng.choice(["decode", "decode", "step", "serve", "verify", "prefill", "prefill", "chunk", "calibrate"])
    D = rng.choice([64, 64, 128, 128, 128, 128, 128, 128, 256])
    dtype = "f32" if rng.random() < 0.12 else "bf16"
    Hkv = rng.choice([1, 2, 4, 8, 8, 8, 16, 32])
    G = rng.choice([1, 2, 3, 4, 4, 4, 8])
    B = _log(rng, 1, 16)
    N = _log(rng, 300, 129020)
    M = min(_log(rng, 32, 1023 if dtype == "bf16" else 256), N // 2)
    c = _case(kind, B=B, Hkv=Hkv, G=G, D=D, Dkc=_dims(rng, D), Dvc=_dims(rng, D), M=M, dtype=dtype)
    rows = B * Hkv                      # (sequence, KV head) pairs
    if kind in ("decode", "step", "serve", "verify"):
        if kind == "verify":
            c["Tq"] = rng.randint(2, max(2, min(8, 16 // G)))
        # rows * states of the largest listed decode calls; fp32 caches are short
        most = (1_050_000 if dtype == "bf16" else 131_072) // max(1, -(-M // 256)) // (2 if D > 128 else 1)
        N = max(300, min(N, most // max(1, G * c.get("Tq", 1) // 4) // rows))
        c["W"] = SINK + _log(rng, 60, 2048)
        if rows * (N + c["W"]) > 1_200_000:
            c["W"] = SINK + 60
    elif kind == "chunk":
        c["B"], N = rng.randint(1, 4), _log(rng, 256, 4096)
        c["M"] = min(M, N)
    else:
        Dc = D if kind == "calibrate" else max(c["Dkc"], c["Dvc"])
        if kind == "calibrate":
            c["M"] = M = min(M, 512, max(32, N // 8))
            flops = 16.6e9
        else:
            flops = 8e9 if dtype == "f32" else 2.3e11 if D == 128 else 6e10
        per = (1 if kind == "calibrate" else 2) * 2 * M * Dc * rows                        # per token
        by = (1 if kind == "calibrate" else 2) * D * rows * (2 if dtype == "bf16" else 4)
        most = 4e7 if kind == "calibrate" else 5.3e8 if dtype == "bf16" and D == 128 else 2e8
        N = max(300, min(N, int(flops / per), int(most / by)))
    c["N"] = N
    c["M"] = min(c["M"], N // 2)
    c["T"] = N + RING if kind in ("step", "serve") else N
    if kind == "chunk":
        c["t0"] = rng.randint(1, 12) * N - SINK
        c["T"] = c["t0"] + N + rng.randint(0, 4 * N)
    elif kind != "calibrate" and rng.random() < 0.3:
        c["T"] += rng.randint(1, 3 * N)             # the period is the longest context, the segment part of it
    return c


def _dt(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _mask(g, B, H, D, Dc):
    """[B,H,D] bytes, Dc random ones per row."""
    order = torch.rand((B, H, D), generator=g, device="cuda").argsort(-1)
    return (order < Dc).to(torch.uint8)


def _tones(g, c):
    """Order, amplitude and phase of three tones for every dim: [3,B,H,D] each."""
    shape = (3, c["B"], c["Hkv"], c["D"])
    top = max(1, (c["M"] - 1) // 2)
    n = torch.randint(1, top + 1, shape, generator=g, device="cuda").float()
    a = 0.5 + torch.rand(shape, generator=g, device="cuda")
    psi = 2.0 * math.pi * torch.rand(shape, generator=g, device="cuda")
    return n, a, psi


def _rows(g, c, tones, mask, t0, count):
    """`count` rows [B,H,count,D] from position t0 on: tones where the mask is set, white noise elsewhere."""
    n, a, psi = tones
    shape = (c["B"], c["Hkv"], count, c["D"])
    pos = torch.arange(t0, t0 + count, device="cuda").float().view(1, 1, count, 1)
    noise = torch.randn(shape, generator=g, device="cuda")
    sig = 0.1 * noise
    for r in range(3):
        sig += a[r].unsqueeze(2) * torch.cos(pos * (n[r] * (2.0 * math.pi / c["T"])).unsqueeze(2) + psi[r].unsqueeze(2))
    return torch.where(mask.bool().unsqueeze(2), sig, noise).to(_dt(c))


def _coeffs(g, c, tones, N, Dc):
    """[B,H,M,Dc] coefficients of such rows: N/2 a (cos psi, -sin psi) at a tone's order, noise of the
    projected white part everywhere."""
    n, a, psi = (t[..., :Dc] for t in tones)
    C = 0.1 * math.sqrt(N / 2.0) * torch.randn((c["B"], c["Hkv"], c["M"], Dc), generator=g, device="cuda")
    for r in range(3):
        i = (2 * n[r].long() - 1).unsqueeze(2)
        C.scatter_add_(2, i.clamp(max=c["M"] - 1), (0.5 * N * a[r] * torch.cos(psi[r])).unsqueeze(2))
        C.scatter_add_(2, (i + 1).clamp(max=c["M"] - 1), (-0.5 * N * a[r] * torch.sin(psi[r])).unsqueeze(2))
    return C


def prepare(case, seed):
    c = dict(case)
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    dt, B, H, G, D, N, M, T = _dt(c), c["B"], c["Hkv"], c["G"], c["D"], c["N"], c["M"], c["T"]
    Dkc, Dvc, W = c["Dkc"], c["Dvc"], c["W"]
    s = {"c": c, "kind": c["kind"], "i": 0}
    s["kmask"], s["vmask"] = _mask(g, B, H, D, Dkc), _mask(g, B, H, D, Dvc)

    if c["kind"] == "calibrate":
        s["x"] = _rows(g, c, _tones(g, c), s["kmask"], 0, N)
        code = fa.FA_F32 if dt == torch.float32 else fa.FA_BF16
        s["ws"] = torch.empty(fa.select_workspace_bytes(code, B, H, N, D, M), dtype=torch.uint8, device="cuda")
        return s

    if c["kind"] in ("prefill", "chunk"):
        t0 = c.get("t0", 0)
        kt, vt = _tones(g, c), _tones(g, c)
        s["k"], s["v"] = _rows(g, c, kt, s["kmask"], t0, N), _rows(g, c, vt, s["vmask"], t0, N)
        cap = t0 + N                                    # tokens the kept slabs hold
        s["kk_pitch"], s["vk_slab"] = fa.keep_rows_pitch(D - Dkc), fa.tok8_numel(cap, D - Dvc)
        s["kk"] = torch.zeros((B, H, cap, s["kk_pitch"]), dtype=dt, device="cuda")
        s["vk"] = torch.zeros((B, H, s["vk_slab"]), dtype=dt, device="cuda")
        if t0:
            s["ck"], s["cv"] = _coeffs(g, c, kt, t0, Dkc), _coeffs(g, c, vt, t0, Dvc)
            ws = max(fa.compress_workspace_bytes(B, H, N, D, d, M, dt) for d in (Dkc, Dvc))
        else:
            s["ck"] = torch.empty((B, H, M, Dkc), dtype=torch.float32, device="cuda")
            s["cv"] = torch.empty((B, H, M, Dvc), dtype=torch.float32, device="cuda")
            ws = fa.compress_kv_workspace_bytes(B, H, N, D, Dkc, Dvc, M, dt)
        s["ws"] = torch.empty(max(ws, 256), dtype=torch.uint8, device="cuda")
        return s

    # decode: coefficients, kept dims (room for a ring of further tokens), full-width rows, queries
    cap = N + RING if c["kind"] in ("step", "serve") else N
    kt, vt = _tones(g, c), _tones(g, c)
    s["ck"], s["cv"] = _coeffs(g, c, kt, N, Dkc), _coeffs(g, c, vt, N, Dvc)
    kp = fa.keep_rows_pitch(D - Dkc)
    s["kk"] = torch.randn((B, H, cap, kp), generator=g, device="cuda").to(dt)
    s["kk"][..., D - Dkc:] = 0
    s["vk"] = torch.randn((B, H, fa.tok8_numel(cap, D - Dvc)), generator=g, device="cuda").to(dt)
    s["kf"], s["vf"] = _rows(g, c, kt, s["kmask"], N, W), _rows(g, c, vt, s["vmask"], N, W)
    tq = c.get("Tq", 0)
    shape = (B, H, tq, G, D) if tq else (B, H * G, D)
    s["q"] = torch.randn(shape, generator=g, device="cuda").to(dt)
    s["out"] = torch.empty(shape, dtype=torch.float32, device="cuda")
    ws = fa.decode_workspace_bytes(B, H * G * max(tq, 1), H, D, Dkc, Dvc, M, cap, W)
    s["ws"] = torch.empty(max(ws, 256), dtype=torch.uint8, device="cuda")
    if cap > N:
        # the tokens that arrive, and for sequences at positions of their own the lists of each step
        s["kk_stride"], s["vk_stride"] = cap * kp, fa.tok8_numel(cap, D - Dvc)
        s["k_new"] = torch.randn((RING, B, H, D), generator=g, device="cuda").to(dt)
        s["v_new"] = torch.randn((RING, B, H, D), generator=g, device="cuda").to(dt)
        if c["kind"] == "serve":
            at = torch.randint(N // 4, N + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
            if B > 1:
                at[0] = N
            step = torch.arange(RING, device="cuda", dtype=torch.int32).unsqueeze(1)
            s["nmid"] = (at + step).contiguous()
            s["slot"] = (SINK + (at + step) % (W - SINK)).to(torch.int32).contiguous()
            s["seq_n"] = (s["nmid"] + 1).contiguous()
    return s


def run(s):
    c = s["c"]
    kind, N, M, T = s["kind"], c["N"], c["M"], c["T"]
    if kind == "decode":
        return fa.fa_decode(s["q"], s["ck"], s["kmask"], s["cv"], s["vmask"], M, T, 0, N, s["kk"], s["vk"],
                            s["kf"], s["vf"], out=s["out"], workspace=s["ws"])
    if kind == "verify":
        return fa.fa_decode_mq(s["q"], s["ck"], s["kmask"], s["cv"], s["vmask"], M, T, 0, N, s["kk"], s["vk"],
                               s["kf"], s["vf"], out=s["out"], workspace=s["ws"])
    if kind == "prefill":
        return fa.fa_compress_kv(s["k"], s["v"], s["kmask"], s["vmask"], c["Dkc"], c["Dvc"], M, T, ck=s["ck"],
                                 cv=s["cv"], k_keep=s["kk"], v_keep=s["vk"], workspace=s["ws"])
    if kind == "chunk":
        t0 = c["t0"]
        fa.fa_compress(s["k"], s["kmask"], c["Dkc"], M, T, t0, True, s["ck"], s["kk"], fa.FA_KEEP_ROWS, t0,
                       (t0 + N) * s["kk_pitch"], workspace=s["ws"])
        fa.fa_compress(s["v"], s["vmask"], c["Dvc"], M, T, t0, True, s["cv"], s["vk"], fa.FA_KEEP_TOK8, t0,
                       s["vk_slab"], workspace=s["ws"])
        return s["ck"], s["kk"], s["cv"], s["vk"]
    if kind == "calibrate":
        return fa.fa_select_dims(s["x"], M, c["Dkc"], workspace=s["ws"])
    i = s["i"]
    s["i"] = (i + 1) % RING
    if kind == "step":
        fa.fa_append(s["k_new"][i], s["v_new"][i], s["kf"], s["vf"], SINK + i % (c["W"] - SINK), True, s["kmask"],
                     s["vmask"], M, T, N + i, s["ck"], s["cv"], s["kk"], s["vk"], None, s["kk_stride"],
                     s["vk_stride"])
        fa.fa_decode(s["q"], s["ck"], s["kmask"], s["cv"], s["vmask"], M, T, 0, N + i + 1, s["kk"], s["vk"],
                     s["kf"], s["vf"], out=s["out"], workspace=s["ws"], kk_stride_bh=s["kk_stride"],
                     vk_stride_bh=s["vk_stride"])
    else:
        fa.fa_append_varlen(s["k_new"][i], s["v_new"][i], s["kf"], s["vf"], s["slot"][i], s["kmask"], s["vmask"], M,
                            T, s["nmid"][i], N + RING, s["ck"], s["cv"], s["kk"], s["vk"], None, s["kk_stride"],
                            s["vk_stride"])
        fa.fa_decode_varlen(s["q"], s["ck"], s["kmask"], s["cv"], s["vmask"], M, T, 0, N + RING, s["seq_n"][i],
                            s["kk"], s["vk"], s["kf"], s["vf"], None, out=s["out"], workspace=s["ws"],
                            kk_stride_bh=s["kk_stride"], vk_stride_bh=s["vk_stride"])
    return s["out"], s["ck"], s["cv"], s["kk"], s["vk"], s["kf"], s["vf"]


def work(case):
    c = case
    e = 4 if c["dtype"] == "f32" else 2
    B, H, G, D, N, M, W = c["B"], c["Hkv"], c["G"], c["D"], c["N"], c["M"], c["W"]
    Dkc, Dvc = c["Dkc"], c["Dvc"]
    P = B * H
    if c["kind"] == "calibrate":
        return {"bytes": P * (N * D * e + D * 5), "flops": 2 * P * N * M * D}
    if c["kind"] in ("prefill", "chunk"):
        states = P * M * (Dkc + Dvc) * 4
        return {"bytes": P * N * (2 * D + 2 * D - Dkc - Dvc) * e + states * (2 if c["kind"] == "chunk" else 1)
                + P * 2 * D, "flops": 2 * P * N * M * (Dkc + Dvc)}
    # serve: sequences stand at 5/8 of N on average
    n = N * 5 // 8 if c["kind"] == "serve" else N
    keep = 2 * D - Dkc - Dvc
    Q = G * c.get("Tq", 1)
    states = P * M * (Dkc + Dvc) * 4
    by = P * Q * D * (e + 4) + states + P * n * keep * e + P * W * 2 * D * e + P * 2 * D
    # scores and outputs through the states (q . C once, then M per row and side), kept dims, full rows
    fl = 2 * P * Q * (M * (Dkc + Dvc) + n * (2 * M + keep) + W * 2 * D)
    if c["kind"] in ("step", "serve"):
        by += states + P * 4 * D * e + P * keep * e         # the state comes back too; two rows in and out
        fl += 2 * P * M * (Dkc + Dvc)
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "calibrate":
        return {"rel": 1e-5}        # fp32 sums (bf16 rows are widened first)
    if case["dtype"] == "f32":      # fp32 sums; behind a softmax they count twice
        return {"rel": 1e-5 if case["kind"] in ("prefill", "chunk") else 2e-5}
    return {"rel": 4e-3}            # bf16 basis and probabilities: 2^-9 each
