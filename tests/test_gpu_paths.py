"""The routes a model step can take give the same bytes: the wide pipeline
(small problems), the split pipeline (larger ones, and every call that hands its
scores out), and the per-layer entry points, which run the selection as one task.
Equality is exact: every route adds the same terms in the same order."""
import pytest

from kvec_testlib import StepPlan

pytestmark = pytest.mark.gpu


def _config(kv, T, H, G, d, dtype, batch=1, O=32, B=None, layers=4, beta=0.25, ext=None, adjust=3):
    return kv.Config(batch=batch, n_layers=layers, n_kv_heads=H, n_q_heads=H * G, head_dim=d, seq_len=T,
                     window=O, window_ext=ext or 2 * O, budget=B or O + T // 8, pool_kernel=7,
                     n_adjust_heads=min(adjust, H), lam=1.0, beta=beta, dtype=dtype)


class Step:
    def __init__(self, kv, cfg, dtype, seed, zero_q=False):
        import torch
        g = torch.Generator(device="cuda").manual_seed(seed)
        L, b, H, T, d, B = cfg.n_layers, cfg.batch, cfg.n_kv_heads, cfg.seq_len, cfg.head_dim, cfg.budget
        self.kv, self.cfg, W = kv, cfg, min(cfg.window_ext, T)
        self.q = torch.randn((L, b, cfg.n_q_heads, W, d), generator=g, device="cuda").to(dtype)
        if zero_q:
            self.q.zero_()
        self.k = torch.randn((L, b, H, T, d), generator=g, device="cuda").to(dtype)
        self.v = torch.randn((L, b, H, T, d), generator=g, device="cuda").to(dtype)
        x = torch.matmul(self.q.float().reshape(L, b, H, -1, d), self.k.float().transpose(-1, -2).contiguous())
        x = x.reshape(L, b, cfg.n_q_heads, W, T) / d ** 0.5
        hidden = torch.arange(T, device="cuda")[None] > torch.arange(T - W, T, device="cuda")[:, None]
        self.lse = x.masked_fill_(hidden, -float("inf")).logsumexp(-1)
        self.ws = torch.empty(kv.kvec_workspace_size(cfg), dtype=torch.uint8, device="cuda")

    def outputs(self):
        import torch
        c = self.cfg
        shape = (c.n_layers, c.batch, c.n_kv_heads, c.budget)
        return (torch.zeros((c.batch, c.n_layers, (c.seq_len + 63) // 64), dtype=torch.int64, device="cuda"),
                torch.full(shape, -7, dtype=torch.int32, device="cuda"),
                torch.zeros(shape + (c.head_dim,), dtype=self.k.dtype, device="cuda"),
                torch.zeros(shape + (c.head_dim,), dtype=self.k.dtype, device="cuda"))

    def model(self, given, timed=False):
        """The step as the library routes it; timed: with profiling events."""
        import torch
        o = self.outputs()
        ev = None
        if timed:
            n = (self.kv.kvec_profile_points_lse if given else self.kv.kvec_profile_points)(self.cfg)
            keep = [torch.cuda.Event(enable_timing=True) for _ in range(n)]
            for e in keep:
                e.record()
            torch.cuda.synchronize()
            ev = [e.cuda_event for e in keep]
        if given:
            self.kv.kvec_evict_model_lse(self.cfg, self.q, self.lse, self.k, self.v, *o, self.ws, events=ev)
        else:
            self.kv.kvec_evict_model(self.cfg, self.q, self.k, self.v, *o, self.ws, events=ev)
        torch.cuda.synchronize()
        if timed:  # every event was recorded, in order, with a launch in between
            assert all(a.elapsed_time(b) > 0.001 for a, b in zip(keep, keep[1:]))
        return o

    def split(self):
        """The step in the split pipeline, whatever its size."""
        import torch
        c, o = self.cfg, self.outputs()
        Tc = c.seq_len - c.window
        p, pe = (torch.zeros((c.n_layers, c.batch, c.n_kv_heads, Tc), device="cuda") for _ in range(2))
        imp = torch.zeros((c.n_layers, c.batch, Tc), device="cuda")
        htop = torch.zeros((c.n_layers, c.batch), dtype=torch.int32, device="cuda")
        self.kv.kvec_evict_model_scores(c, self.q, self.k, self.v, *o, p, pe, imp, htop, self.ws)
        torch.cuda.synchronize()
        return o

    def layers(self, given):
        import torch
        bits, idx, ko, vo = o = self.outputs()
        for l in range(self.cfg.n_layers):
            if given:
                self.kv.kvec_evict_layer_lse(self.cfg, l, self.q[l], self.lse[l], self.k[l], self.v[l], bits, idx[l],
                                             ko[l], vo[l], self.ws)
            else:
                self.kv.kvec_evict_layer(self.cfg, l, self.q[l], self.k[l], self.v[l], bits, idx[l], ko[l], vo[l],
                                         self.ws)
        torch.cuda.synchronize()
        return o


# (T, H, G, d, dtype, batch, O, wide with two passes and with given normalisers):
# both sides of the lines of the wide pipeline (score work-groups, what else a
# launch holds), ragged lengths, key tiles of 128, 256 and 512, one and two row
# tiles per work-group, row tiles that mix last-O and earlier rows
CASES = [
    (1024, 4, 2, 64, "f32", 1, 32, True, True),
    (777, 8, 4, 128, "bf16", 2, 32, True, True),
    (3071, 8, 4, 128, "bf16", 1, 32, True, True),
    (3073, 8, 4, 128, "bf16", 1, 32, False, True),
    (4096, 4, 7, 128, "bf16", 1, 32, True, True),
    (4096, 8, 4, 64, "bf16", 1, 32, False, True),
    (2048, 8, 4, 128, "bf16", 3, 32, False, False),
    (12001, 2, 4, 128, "bf16", 1, 32, True, True),
    (8200, 8, 1, 64, "bf16", 2, 40, False, True),
    (16384 + 77, 2, 6, 128, "bf16", 1, 16, True, True),
    (2000, 8, 4, 128, "bf16", 1, 20, True, True),
    (65, 2, 2, 64, "bf16", 3, 16, True, True),
    (1000, 8, 8, 64, "bf16", 5, 32, False, True),
    (1000, 8, 8, 64, "bf16", 6, 32, False, False),
    (300, 4, 2, 64, "f32", 16, 32, True, True),
    (1000, 8, 2, 64, "f32", 6, 32, False, True),
]


@pytest.mark.parametrize("given", [False, True], ids=["two-pass", "given"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"T{c[0]}-H{c[1]}-G{c[2]}-{c[4]}-b{c[5]}-O{c[6]}")
def test_routes_agree(gpu_lib, case, given):
    import torch
    T, H, G, d, dt, batch, O = case[:7]
    f32 = dt == "f32"
    cfg = _config(gpu_lib, T, H, G, d, gpu_lib.KVEC_F32 if f32 else gpu_lib.KVEC_BF16, batch, O)
    assert StepPlan(cfg).wide(given) == case[8 if given else 7]
    s = Step(gpu_lib, cfg, torch.float32 if f32 else torch.bfloat16, T)
    want = s.layers(given)
    for got in [s.model(given), s.model(given, timed=True)] + ([] if given else [s.split()]):
        for a, b in zip(got, want):
            assert torch.equal(a, b)


@pytest.mark.parametrize("ext,adjust", [(64, 0), (32, 3), (40, 1)], ids=["no-heads", "same-window", "mixed-tile"])
@pytest.mark.parametrize("given", [False, True], ids=["two-pass", "given"])
def test_routes_agree_few_extended_rows(gpu_lib, ext, adjust, given):
    """Without H_top heads or without rows of their own the wide pipeline scores
    the last-O rows only: the extended rows are not read (they hold NaN)."""
    import torch
    cfg = _config(gpu_lib, 1800, 8, 4, 128, gpu_lib.KVEC_BF16, ext=ext, adjust=adjust)
    assert StepPlan(cfg).wide(given)
    s = Step(gpu_lib, cfg, torch.bfloat16, ext)
    want = s.layers(given)
    if adjust == 0:
        s.q[..., :32, :] = float("nan")
        s.lse[..., :32] = float("nan")
    for got in [s.model(given)] + ([] if given else [s.split()]):
        for a, b in zip(got, want):
            assert torch.equal(a, b)


# (T, batch, layers, given): calls of several steps in the split pipeline, with
# layer counts below and above its depth (several steps in one launch, ring slots
# and count buffers reused across steps), and a prompt whose single step is wide
STEPS = [(3100, 3, 4, False), (3100, 3, 13, False), (3100, 3, 4, True), (3100, 3, 13, True), (12001, 1, 3, True)]


@pytest.mark.parametrize("T,batch,layers,given", STEPS)
def test_steps_in_the_split_pipeline(gpu_lib, T, batch, layers, given):
    import torch
    kv, n = gpu_lib, 3
    cfg = _config(kv, T, 8, 4, 128, kv.KVEC_BF16, batch, layers=layers)
    assert not StepPlan(cfg).wide(given, n) and StepPlan(cfg).wide(given) == (batch == 1)
    steps = [Step(kv, cfg, torch.bfloat16, 20 + i) for i in range(n)]
    q, k, v, lse = (torch.stack([getattr(s, x) for s in steps]) for x in ("q", "k", "v", "lse"))
    got = [torch.stack([o] * n) for o in steps[0].outputs()]
    if given:
        kv.kvec_evict_model_lse_steps(cfg, q, lse, k, v, *got, steps[0].ws)
    else:
        kv.kvec_evict_model_steps(cfg, q, k, v, *got, steps[0].ws)
    torch.cuda.synchronize()
    for i, s in enumerate(steps):
        for a, b in zip(got, s.layers(given)):
            assert torch.equal(a[i], b), f"step {i}"


@pytest.mark.parametrize("T", [11500, 13000], ids=["members-in-lds", "members-spilled"])
def test_routes_agree_all_members(gpu_lib, T):
    """Zero queries: all scores tie, so every token is a member; the longer
    prompt has more than a selection task holds in LDS (about 11.7 thousand)."""
    import torch
    cfg = _config(gpu_lib, T, 2, 2, 64, gpu_lib.KVEC_BF16, layers=3)
    s = Step(gpu_lib, cfg, torch.bfloat16, 5, zero_q=True)
    want = s.split()
    for got in (s.model(False), s.layers(False)):
        for a, b in zip(got, want):
            assert torch.equal(a, b)


# (T, H, G, d, batch, O, O', tiles with two passes and with given normalisers):
# batches whose launches hold enough score work-groups for two and for four key
# tiles each, ragged last tiles and last work-groups.  The heads' maxima are
# exchanged over LDS with one buffer (periods of the whole tile: H 8 with G 4, 3
# or 8, H 1 needs none) and with two (H 8 with O 20, G 1; H 4 with G 7; H 2 with
# G 6); row tiles mix last-O and earlier rows where O is no multiple of their 16 to
# 64 rows; seven and eight row blocks.  A tile of 256 keys (H 2, G 1) has none.
LONG = [
    (16384 + 77, 8, 4, 128, 10, 32, 64, 2, 2),
    (16384 + 77, 8, 4, 128, 30, 32, 64, 4, 4),
    (16384 + 77, 4, 7, 128, 12, 32, 64, 1, 2),
    (16384 + 77, 4, 7, 128, 46, 32, 64, 1, 4),
    (16384 + 77, 8, 8, 128, 6, 32, 64, 2, 1),
    (16384 + 77, 1, 8, 128, 40, 32, 64, 2, 2),
    (16900, 8, 1, 128, 30, 32, 64, 2, 2),
    (16384 + 77, 8, 4, 128, 10, 20, 40, 2, 2),
    (16384 + 77, 8, 3, 64, 10, 33, 71, 2, 2),
    (16384 + 77, 2, 6, 128, 24, 32, 64, 2, 2),
    (16384 + 77, 4, 2, 128, 16, 48, 120, 2, 2),
    (16384 + 77, 1, 4, 64, 12, 32, 64, 2, 1),
    (16384 + 77, 2, 1, 64, 24, 32, 64, 1, 1),
    (20011, 1, 4, 64, 44, 32, 64, 4, 2),
]


@pytest.mark.parametrize("case", LONG, ids=lambda c: f"T{c[0]}-H{c[1]}-G{c[2]}-d{c[3]}-b{c[4]}-O{c[5]}")
def test_long_score_work_groups(gpu_lib, case):
    """Steps and their scores are the bytes of the per-layer calls, whose score
    work-groups take one key tile each."""
    import torch
    kv = gpu_lib
    T, H, G, d, batch, O, ext = case[:7]
    cfg = _config(kv, T, H, G, d, kv.KVEC_BF16, batch, O, layers=1, B=512, ext=ext)
    plan = StepPlan(cfg)
    assert not plan.wide(False) and not plan.wide(True)
    assert (plan.tiles(False), plan.tiles(True)) == case[7:]
    s = Step(kv, cfg, torch.bfloat16, 11)
    for given in (False, True):
        for a, b in zip(s.model(given), s.layers(given)):
            assert torch.equal(a, b)
    _same_scores(kv, s)


def _same_scores(kv, s):
    import torch
    cfg, T, batch, H = s.cfg, s.cfg.seq_len, s.cfg.batch, s.cfg.n_kv_heads
    Tc = T - cfg.window
    p, pe = (torch.zeros((1, batch, H, Tc), device="cuda") for _ in range(2))
    imp = torch.zeros((1, batch, Tc), device="cuda")
    htop = torch.zeros((1, batch), dtype=torch.int32, device="cuda")
    kv.kvec_evict_model_scores(cfg, s.q, s.k, s.v, *s.outputs(), p, pe, imp, htop, s.ws)
    p1, pe1, imp1 = torch.empty_like(p[0]), torch.empty_like(p[0]), torch.empty_like(imp[0])
    kv.kvec_score(cfg, s.q[0], s.k[0], p1, pe1, imp1, s.ws)
    torch.cuda.synchronize()
    assert torch.equal(p[0], p1)
    top = (htop[0][:, None] >> torch.arange(H, device="cuda")) & 1  # the others' rows stay zero
    assert torch.equal(pe[0], pe1 * top[..., None])
    assert torch.equal(imp[0], imp1)


def test_long_score_work_groups_far_references(gpu_lib):
    """Logits spread over more than the float32 exponent range: with the
    references of another key tile, row sums lose terms or leave the range."""
    import torch
    kv = gpu_lib
    cfg = _config(kv, 20011, 8, 4, 128, kv.KVEC_BF16, 12, layers=1, B=512)
    assert StepPlan(cfg).tiles(False) == 4
    s = Step(kv, cfg, torch.bfloat16, 13)
    g = torch.Generator(device="cuda").manual_seed(14)
    s.q *= 6
    s.k *= 1 + 2 * (torch.rand(s.k.shape[:-1] + (1,), generator=g, device="cuda") < 0.01)
    _same_scores(kv, s)
