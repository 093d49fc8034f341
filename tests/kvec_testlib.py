"""Shared helpers of the GPU parity tests: seeded inputs on the device, the
oracle on the same bytes, and the agreement / tolerance checks."""
from __future__ import annotations

import numpy as np

import oracle as orc
import synth

SCORE_RTOL = 2e-3      # score relative error bound (bf16 inputs, fp32 accumulation)
AGREE_MIN = 0.995      # end-to-end index agreement
CUT_RTOL = 4e-3        # a mismatch must sit within this of the cut (two score errors)


def torch_dtype(w):
    import torch
    return torch.bfloat16 if w.dtype == "bf16" else torch.float32


def to_device(a: np.ndarray, w):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a))
    if w.dtype == "bf16":
        t = t.view(torch.bfloat16)
    return t.cuda()


def layer_inputs(w, layer: int, b: int):
    """Host arrays of one (layer, sequence): q [HQ][Wn][d], k/v [H][T][d] (storage dtype)."""
    return synth.queries(w, layer, b), synth.keys(w, layer, b), synth.values(w, layer, b)


def model_tensors(w, layers=None):
    """Device tensors q [L][b][HQ][Wn][d], k/v [L][b][H][T][d] for the whole workload."""
    import torch
    L = w.n_layers if layers is None else layers
    dt = torch_dtype(w)
    q = torch.empty((L, w.batch, w.n_q_heads, w.rows, w.head_dim), dtype=dt, device="cuda")
    k = torch.empty((L, w.batch, w.n_kv_heads, w.seq_len, w.head_dim), dtype=dt, device="cuda")
    v = torch.empty_like(k)
    for l in range(L):
        for b in range(w.batch):
            qa, ka, va = layer_inputs(w, l, b)
            q[l, b].copy_(to_device(qa, w))
            k[l, b].copy_(to_device(ka, w))
            v[l, b].copy_(to_device(va, w))
    return q, k, v


def oracle_scores(w, layer: int, b: int, q=None, k=None):
    """Oracle fp32 scores (float64 computation on the exact input values)."""
    if q is None:
        q = synth.queries(w, layer, b)
        k = synth.keys(w, layer, b)
    qf = synth.to_f64(q, w.dtype)
    kf = synth.to_f64(k, w.dtype)
    p, pe, imp = orc.window_scores(qf, kf, w.window)
    return p, pe, imp


class StepPlan:
    """The library's geometry and the rules by which a model step picks its
    pipeline and its score work-groups, restated, so that a test can say which
    route its case takes (a case that left its route would test nothing)."""

    def __init__(self, cfg):
        self.cfg = cfg
        H, G, T, O, d = cfg.n_kv_heads, cfg.n_q_heads // cfg.n_kv_heads, cfg.seq_len, cfg.window, cfg.head_dim
        self.es = es = 2 if cfg.dtype == 0 else 4
        self.G, self.H, self.Wn, self.Tc = G, H, min(cfg.window_ext, T), T - O
        self.WR = WR = 16 * (1 if G >= 4 else 4 // G)
        self.delta = cfg.n_adjust_heads if self.Wn > O else 0
        self.n_rt, self.n_rt_base = _up(self.Wn, WR), _up(O, WR)
        self.nsum = 1 if O % WR == 0 else 2
        tpw = 8 // H
        self.n_rtg, self.n_rtg_base = _up(self.n_rt, tpw), _up(self.n_rt_base, tpw)
        self.n_rt_x = self.n_rt - self.n_rt_base if self.delta else 0
        tile = 512
        while tile > 128 and tile * 32 > T:
            tile //= 2
        self.tile1, step = tile, 16 * d * es
        ring = 8 * (4 if step <= 2048 else 3 if step <= 4096 else 1) * step

        def slot(nh, sk, tile, exchange):
            return ((1 if sk >= tile else 2) * WR * (sk + 4) if exchange else 0) + self.nsum * nh * tile + tile

        def periods(tile):
            sk, least = tile, 32 if tile == 512 else 16
            while sk >= least:
                yield sk
                sk = 128 if sk == tile and tile > 128 else sk // 2

        def fits(tile, sk):
            ext = 8 * slot(1, sk, tile, False) if self.n_rt_x else 0
            return ring + 4 * max(tpw * slot(H, sk, tile, H > 1), ext) <= 163840 - 1024

        self.tile2, self.SK = next((t, sk) for t in (512, 256, 128) if t <= tile for sk in periods(t) if fits(t, sk))
        self.n_kt1, self.n_kt2 = _up(T, self.tile1), _up(self.Tc, self.tile2)

    def wide(self, given, n_steps=1):
        """Whether a step runs the wide pipeline."""
        c, b, H = self.cfg, self.cfg.batch, self.H
        score = b * (self.n_kt2 + (0 if given else self.n_kt1)) * (self.n_rtg if self.delta else self.n_rtg_base)
        if score > 192:
            return False
        heavy = self.G >= 7 or self.es == 4
        if heavy and (c.head_dim == 128 or score <= 96):
            return True
        if not heavy and self.tile1 > 128:
            return n_steps == 1 or score <= 160
        pool, prep = b * H * _up(self.Tc, 8 * 512), b * H * _up(self.Tc, 8 * 1024)
        gather = b * _up(H * c.budget * c.head_dim * self.es // 16, 2048)
        others = sum(_up(n, 8) * 8 for n in (b * H, b * H, pool, prep, gather) + ((pool,) if self.delta else ()))
        return score + others // (4 if heavy else 2) <= 240

    def tiles(self, given):
        """Key tiles per score work-group of a step in the split pipeline."""
        b, d = self.cfg.batch, self.cfg.head_dim
        if self.es != 2 or self.tile1 != 512 or self.tile2 != 512:
            return 1

        def one_pass(n_kt):
            return b * n_kt * self.n_rtg_base + _up(b * n_kt * self.delta * self.n_rt_x, 8)

        n = one_pass(self.n_kt2) + (0 if given else one_pass(self.n_kt1))
        sub = 4 if n >= 2560 else 2 if n >= (640 if given else 896) else 1
        if not given and d == 128 and self.G >= 7:
            sub = 1 if self.G == 7 else min(sub, 2)
        return sub


def _up(n, m):
    return -(-n // m)


def rel_err(got: np.ndarray, ref: np.ndarray) -> float:
    got = np.asarray(got, np.float64)
    ref = np.asarray(ref, np.float64)
    return float(np.max(np.abs(got - ref) / np.maximum(np.abs(ref), 1e-30)))


def bits_to_bool(words: np.ndarray, T: int) -> np.ndarray:
    """uint64 bitmap row -> bool[T]."""
    u = np.asarray(words, dtype=np.uint64)
    bits = ((u[:, None] >> np.arange(64, dtype=np.uint64)[None, :]) & np.uint64(1)).astype(bool)
    return bits.reshape(-1)[:T]


def counts_before(bits_rows: np.ndarray, layer: int, T: int) -> np.ndarray:
    """n_t from bitmap rows [L][W] of the layers before `layer`."""
    n = np.zeros(T, dtype=np.int64)
    for l in range(layer):
        n += bits_to_bool(bits_rows[l], T)
    return n


def agreement(gpu_idx: np.ndarray, res: orc.LayerResult, M: int, kp: int):
    """Teacher-forced comparison of one layer for one sequence.

    Returns (matched, total, bad) where `bad` lists mismatched tokens that are
    NOT within CUT_RTOL of the oracle's cut (of P' for the final pick, or of
    P_sel for the preserve set)."""
    H = gpu_idx.shape[0]
    matched, total, bad = 0, 0, []
    for h in range(H):
        g = set(int(x) for x in gpu_idx[h, :M])
        o = set(int(x) for x in res.idx[h, :M])
        matched += len(g & o)
        total += M
        if g == o:
            continue
        padj = res.p_adj[h].astype(np.float64)
        cut = np.sort(padj)[::-1][M - 1]
        psel = res.p_sel[h].astype(np.float64)
        kcut = np.sort(psel)[::-1][kp - 1] if kp > 0 else None
        for t in g ^ o:
            near_cut = abs(padj[t] - cut) <= CUT_RTOL * abs(cut)
            near_keep = kcut is not None and abs(psel[t] - kcut) <= CUT_RTOL * abs(kcut)
            if not (near_cut or near_keep):
                bad.append((h, t, float(padj[t]), float(cut)))
    return matched, total, bad
