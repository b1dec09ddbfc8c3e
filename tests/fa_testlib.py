"""Helpers shared by the GPU parity tests (no method arithmetic here)."""

from __future__ import annotations

import os
import subprocess

import numpy as np
import torch

import oracle.fourier_kv as fk
from workloads import make_context


def torch_dtype(cfg):
    return torch.float32 if cfg.dtype == "f32" else torch.bfloat16


def to_dev(a: np.ndarray, cfg=None, dtype=None):
    t = torch.from_numpy(np.ascontiguousarray(a))
    if t.dtype == torch.float32 and (cfg is not None or dtype is not None):
        t = t.to(dtype if dtype is not None else torch_dtype(cfg))
    return t.cuda()


def rows_to_tok8(x: np.ndarray) -> np.ndarray:
    """[..., n, Du] rows -> [..., ceil(n/8)*Du*8] token-interleaved-by-8 slab."""
    *lead, n, du = x.shape
    g = (n + 7) // 8
    pad = np.zeros((*lead, g * 8, du), dtype=x.dtype)
    pad[..., :n, :] = x
    return np.ascontiguousarray(pad.reshape(*lead, g, 8, du).swapaxes(-1, -2)).reshape(*lead, g * du * 8)


def rows_pad8(x: np.ndarray) -> np.ndarray:
    """[..., n, Du] rows -> [..., n, Du rounded up to 8] with zero pad columns."""
    *lead, n, du = x.shape
    pitch = (du + 7) // 8 * 8
    out = np.zeros((*lead, n, pitch), dtype=x.dtype)
    out[..., :du] = x
    return out


def oracle_state(cfg, ctx, heads=None):
    """Oracle compression of the middle segment.  `heads`: list of (b, hkv) to
    evaluate (others left as zeros), None = all.  Coefficients are rounded to
    fp32, which is what the decode step is handed."""
    B, H, N, D, M, T = cfg.B, cfg.Hkv, cfg.N, cfg.D, cfg.M, cfg.T
    ck = np.zeros((B, H, M, cfg.Dkc)); cv = np.zeros((B, H, M, cfg.Dvc))
    kk = np.zeros((B, H, N, D - cfg.Dkc), np.float32); vk = np.zeros((B, H, N, D - cfg.Dvc), np.float32)
    todo = heads if heads is not None else [(b, h) for b in range(B) for h in range(H)]
    for b, h in todo:
        c, k = fk.compress_segment(ctx["k_mid"][b, h], ctx["kmask"][b, h], M, T, cfg.t0)
        ck[b, h], kk[b, h] = c, k
        c, k = fk.compress_segment(ctx["v_mid"][b, h], ctx["vmask"][b, h], M, T, cfg.t0)
        cv[b, h], vk[b, h] = c, k
    return {"ck": ck, "cv": cv, "kk": kk, "vk": vk,
            "ck32": ck.astype(np.float32), "cv32": cv.astype(np.float32)}


def oracle_decode_heads(cfg, ctx, st, heads, from_f32_coeffs=True):
    """Oracle outputs for the listed (b, hkv): dict (b,h) -> [G, D]."""
    out = {}
    G = cfg.G
    for b, h in heads:
        ck = st["ck32"][b, h].astype(np.float64) if from_f32_coeffs else st["ck"][b, h]
        cv = st["cv32"][b, h].astype(np.float64) if from_f32_coeffs else st["cv"][b, h]
        out[(b, h)] = fk.decode_head_group(
            ctx["q"][b, h * G:(h + 1) * G], ck, ctx["kmask"][b, h], cv, ctx["vmask"][b, h],
            cfg.T, cfg.t0, cfg.N, st["kk"][b, h], st["vk"][b, h], ctx["k_full"][b, h], ctx["v_full"][b, h])
    return out


def sample_heads(cfg, k, seed=0):
    allh = [(b, h) for b in range(cfg.B) for h in range(cfg.Hkv)]
    if k is None or k >= len(allh):
        return allh
    rng = np.random.default_rng(seed)
    idx = sorted(rng.choice(len(allh), size=k, replace=False))
    return [allh[i] for i in idx]


def cached_context(cfg, _cache={}):
    key = (cfg.name, cfg.index)
    if key not in _cache:
        _cache.clear()  # keep at most one big context alive
        _cache[key] = make_context(cfg)
    return _cache[key]


HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2506_11886_amd", "csrc")
HOST_ONLY = r"""
#include <cstdio>
extern "C" {   // nothing is launched: the registration of kernels has nothing to do
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
}
"""


def host_program(directory, main, sources):
    """`main` (it includes the .hip file whose rules it asks for) and the library's `sources`, compiled for the host alone without
    the HIP runtime: a function from a list of tuples to the program's lines as tuples."""
    (directory / "main.hip").write_text(main)
    flags = ["-O1", "-std=c++17", "--offload-arch=gfx950", "--offload-host-only", "-I", os.path.join(os.path.dirname(os.path.dirname(CSRC)), "include"),
             "-I", CSRC]
    objects = [(directory / "main.hip", directory / "main.o")] + [(os.path.join(CSRC, s), directory / (s + ".o")) for s in sources]
    jobs = [subprocess.Popen([HIPCC, *flags, "-c", str(src), "-o", str(obj)]) for src, obj in objects]
    assert all([j.wait() == 0 for j in jobs])
    exe = str(directory / "rules")
    # (what the rules do not call stays unresolved)
    subprocess.run(["g++", "-no-pie", *[str(obj) for _, obj in objects], "-o", exe, "-Wl,--unresolved-symbols=ignore-all"], check=True)

    def ask(calls):
        text = "\n".join(" ".join(map(str, c)) for c in calls)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(int(w) if w.lstrip("-").isdigit() else w for w in line.split()) for line in out.splitlines()]
    return ask


# Calls of the general middle-row kernel with eight waves: dtype, B, Hkv, heads a KV head, D, Dkc, Dvc, M, N (= period), W
GENERAL_CALLS = [
    ("bf16", 16, 10, 1, 64, 41, 48, 795, 1640, 0),      # chunks joined, one query head
    ("bf16", 20, 7, 6, 128, 97, 60, 300, 1299, 270),    # chunks joined, six heads, kept V past two tiles, full-width rows apart
    ("bf16", 3, 2, 16, 64, 40, 30, 1023, 1100, 130),     # the longest series, sixteen heads
    ("bf16", 5, 4, 6, 64, 40, 30, 300, 900, 130),       # eight chunks, full-width rows apart
    ("bf16", 5, 3, 3, 128, 70, 77, 301, 1500, 9),       # few heads: full-width rows in the launch of the middle rows
    ("f32", 3, 5, 6, 64, 45, 40, 255, 900, 70),
]

# Folds in slices of 32 and 64 head dims: B, Hkv, D, Dkc, Dvc, M, dtype, dims of a slice
APPEND_CALLS = [
    (18, 5, 128, 96, 5, 257, "bf16", 32),      # (five compressed dims: slices without one)
    (15, 10, 72, 31, 72, 130, "f32", 32),      # a last slice of eight dims, nothing kept of V
    (64, 8, 24, 20, 9, 129, "bf16", 32),       # one slice that the head does not fill
    (3, 22, 192, 130, 0, 1, "bf16", 32),
    (24, 7, 128, 91, 128, 255, "f32", 64),
    (26, 10, 72, 3, 50, 65, "bf16", 64),       # a last slice of eight dims
    (110, 4, 40, 40, 17, 1023, "f32", 64),     # one slice that the head does not fill
    (9, 9, 256, 200, 131, 300, "bf16", 64),
]

# Calls of project_rows: dtype, H, N, D, Dkc, Dvc (None: fa_compress of K alone), M, T, token offset of the kept dims; harmonic tiles of a workgroup,
# chunks of the tokens
ROWS_CALLS = [
    ("bf16", 1, 3953, 64, 11, 44, 339, 3953, 8, 1, 3),       # two terms, chunks
    ("bf16", 3, 10599, 128, 31, 88, 812, 10604, 3, 2, 3),
    ("bf16", 1, 2030, 256, 147, None, 170, 2035, 8, 1, 2),
    ("bf16", 34, 535, 64, 3, 57, 113, 540, 3, 2, 1),         # two terms, several tiles a workgroup
    ("bf16", 17, 525, 64, 15, 2, 525, 2100, 3, 4, 1),
    ("bf16", 105, 644, 64, 13, 61, 194, 2576, 8, 8, 1),
    ("bf16", 45, 527, 128, 104, 113, 71, 2108, 0, 2, 1),
    ("bf16", 96, 709, 128, 61, 100, 72, 709, 8, 4, 1),
    ("bf16", 12, 673, 256, 221, 91, 327, 2692, 3, 2, 1),
    ("bf16", 15, 608, 128, 40, 55, 1, 2432, 8, 1, 1),        # the mean alone
    ("bf16", 71, 151, 64, 23, 56, 151, 151, 3, 8, 1),        # three terms
    ("bf16", 102, 157, 128, 106, 48, 157, 157, 3, 8, 1),
    ("bf16", 86, 87, 256, 256, 59, 87, 92, 8, 4, 1),
    ("f32", 2, 9574, 64, 61, 64, 175, 9574, 3, 2, 19),
    ("f32", 10, 1725, 64, 39, None, 806, 1730, 3, 4, 3),
    ("f32", 10, 1111, 64, 29, 22, 965, 1111, 8, 8, 3),
    ("f32", 37, 1356, 128, 106, 15, 114, 1356, 3, 4, 3),
    ("f32", 50, 1411, 256, 157, 3, 35, 1416, 3, 2, 3),
    ("f32", 78, 37, 256, 8, 213, 37, 42, 0, 2, 1),
]
