// The eviction step as a software pipeline of fused launches.
//
// Every stage of one layer depends only on earlier stages of the same layer,
// except the coverage-aware selection, which also needs the previous layer's
// selection (its bitmap row defines n_t).  The window rows split in two: the
// last-O rows (P and I, every head) and the rest of the extended window (P
// over O', needed only for the H_top heads, which are known once P is pooled).
// Launch j of the step therefore runs, side by side in one grid of 512-thread
// work-groups:
//
//   select B layer j-10  (one work-group per (sequence, head); the serial chain)
//   count    layer j-10  (running coverage counts for the next selection)
//   select A layer j-9   (members and preserve set; no earlier layer needed)
//   pass 2   layer j-2   last-O rows, every head: P, I
//   pass 2   layer j-6   extended rows, H_top heads: the rest of P over O'
//   pass 1   layer j     last-O rows: row-normaliser partials
//   pass 1   layer j-4   extended rows of the H_top heads
//   lse      layers j-1, j-5 (row normalisers of the two row sets)
//   pool     layer j-3   P: max-pool, sigma sums, histogram, I
//   pool     layer j-7   P over O' of the H_top heads
//   prep     layer j-8   (sigma, H_top, candidate members)
//   gather   layer j-11  (compacted cache)
//
// so L + 11 launches cover the whole step and the serial selection chain
// runs in the shadow of the score passes.  Per-layer scratch lives in a ring
// of kRing slots.
//
// When the caller supplies the window rows' normalisers (the log-sum-exp its
// prefill attention already computed for those query rows), pass 1 and the
// lse stages drop out and the step takes L + 7 launches: pass 2 of the
// last-O rows at j, their pool at j-1, pass 2 of the extended rows at j-2,
// their pool at j-3, prep at j-4, select A at j-5, select B and count at
// j-6, gather at j-7.
//
// Small problems run the wide pipeline: pass 1, lse, pass 2 and both pools of
// every row and head (of the last-O rows alone without H_top heads) at j .. j-3,
// prep at j-4, select A at j-5, select B and count at j-6, gather at j-7 (two
// less with given normalisers).
//
// Work-group IDs are dispatched round-robin over the 8 XCDs, each with its
// own L2.  Within a stage, consecutive tasks (e.g. the row tiles of one key
// tile, which read the same K rows) are mapped to work-groups on the same
// XCD so that K is fetched once per XCD L2.
#include <string.h>

#include "kvec_step.h"

namespace kvec {
namespace {

using namespace step;

// P, P over O', I of one layer from the score partials (fixed order).
__global__ void finalize_kernel(Problem P, const float* psum_base, const float* psum_all,
                                const float* ipart, float* p_raw, float* p_ext, float* imp) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y, b = blockIdx.z;
  if (t >= P.Tc) return;
  if (y < P.H) {
    float sb = 0.f, sa = 0.f;
    for (int rt = 0; rt < P.n_rt; ++rt) {
      const int64_t o = (((int64_t)b * P.n_rt + rt) * P.H + y) * P.Tc + t;
      if (rt < P.n_rt_base) sb += psum_base[o];
      sa += psum_all[o];
    }
    p_raw[((int64_t)b * P.H + y) * P.Tc + t] = sb * P.inv_go;
    p_ext[((int64_t)b * P.H + y) * P.Tc + t] = sa * P.inv_gwn;
  } else {
    float s = 0.f;
    for (int rt = 0; rt < P.n_rt_base; ++rt) s += ipart[((int64_t)b * P.n_rt + rt) * P.Tc + t];
    imp[(int64_t)b * P.Tc + t] = s * P.inv_go;
  }
}

__global__ void keep_all_kernel(int32_t* idx, uint64_t* bits, int H, int B, int T, int L, int W,
                                int layer) {
  const int b = blockIdx.y;
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < H * B) idx[(int64_t)b * H * B + i] = (i % B) < T ? (i % B) : -1;
  if (i < W) {
    const int t0 = i * 64;
    const int nb = min(64, T - t0);
    bits[((int64_t)b * L + layer) * W + i] = nb >= 64 ? ~0ull : ((1ull << nb) - 1ull);
  }
}

__global__ void coverage_kernel(const uint64_t* bits, int64_t* count, int L, int W, int upto) {
  __shared__ int64_t red[16];
  const int b = blockIdx.x;
  int64_t c = 0;
  for (int w = threadIdx.x; w < W; w += blockDim.x) {
    uint64_t u = 0;
    for (int l = 0; l <= upto; ++l) u |= bits[((int64_t)b * L + l) * W + w];
    c += __popcll(u);
  }
  for (int o = 32; o > 0; o >>= 1) c += __shfl_xor(c, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t s = 0;
    for (int w = 0; w < (int)(blockDim.x >> 6); ++w) s += red[w];
    count[b] = s;
  }
}

// Work-groups of an EXT pass over n_kt key tiles: its (sequence, key tile,
// H_top head, row tile) tasks packed eight to a work-group, one per wave.
int ext_wgs(const Problem& P, int n_kt) {
  return P.n_rt_x ? (int)(((int64_t)P.batch * n_kt * P.delta_eff * P.n_rt_x + 7) / 8) : 0;
}

int seg_count(const Problem& P, int st) {
  const bool ext = P.delta_eff > 0;
  switch (st) {
    case ST_SELECT:
    case ST_SELA:
    case ST_SELAB: return P.batch * P.H;
    case ST_COUNT: return P.batch * ((P.words + kCountWords - 1) / kCountWords);
    case ST_CNTB: return P.batch * ((P.words + kBitWords - 1) / kBitWords);
    case ST_PASS1: return P.batch * P.n_wt1 * P.n_rtg;
    case ST_P1B: return P.batch * P.n_wt1 * P.n_rtg_base;
    case ST_P1X: return ext_wgs(P, P.n_wt1);
    case ST_LSE:
    case ST_LSEB: return P.batch * lse_tasks_per_seq(P, st);
    case ST_LSEX: return P.n_rt_x ? P.batch * lse_tasks_per_seq(P, st) : 0;
    case ST_PASS2: return P.batch * P.n_wt2 * P.n_rtg;
    case ST_P2B: return P.batch * P.n_wt2 * P.n_rtg_base;
    case ST_P2X: return ext_wgs(P, P.n_wt2);
    case ST_POOL:
    case ST_POOLB:
    case ST_POOLE: return P.batch * P.H * ((P.n_pool + kPoolPer - 1) / kPoolPer);
    case ST_POOLX: return ext ? P.batch * P.delta_eff * ((P.n_pool + kPoolPer - 1) / kPoolPer) : 0;
    case ST_PREP: return P.batch * P.H * ((P.n_prep + kPrepPer - 1) / kPrepPer);
    case ST_GATHER: return P.batch * P.n_gather;
  }
  return 0;
}

// Work-groups of a stage in the grid (segments start at multiples of 8).
int padded(const Problem& P, int st) { return (seg_count(P, st) + 7) & ~7; }

StepFn pick(const Problem& P) {
  if (P.sub > 1) return P.D == 64 ? pick_g<BF16, 64, true>(P.G) : pick_g<BF16, 128, true>(P.G);
  if (P.esize == 2) return P.D == 64 ? pick_g<BF16, 64, false>(P.G) : pick_g<BF16, 128, false>(P.G);
  return P.D == 64 ? pick_g<F32, 64, false>(P.G) : pick_g<F32, 128, false>(P.G);
}

StepArgs base_args(const Geometry& g, char* ws, const Workspace& w) {
  StepArgs a;
  memset(&a, 0, sizeof(a));
  a.P = g.p;
  a.w = w;
  a.ws = ws;
  for (int s = 0; s < ST_N; ++s) a.seg[s] = Seg{-1, 0, 0, 0, 0};
  return a;
}

void set_model(StepArgs& a, const ModelIO& m) {
  a.q = static_cast<const char*>(m.q);
  a.k = static_cast<const char*>(m.k);
  a.v = static_cast<const char*>(m.v);
  for (int i = 0; i < 4; ++i) {
    a.qs[i] = m.qs[i];
    a.ks[i] = m.ks[i];
    a.vs[i] = m.vs[i];
  }
  a.lse = m.lse;
  for (int i = 0; i < 3; ++i) a.ls[i] = m.ls[i];
  a.bits = m.bits;
  a.idx = m.idx;
  a.k_out = static_cast<char*>(m.k_out);
  a.v_out = static_cast<char*>(m.v_out);
  a.sc_p = m.sc_p;
  a.sc_pe = m.sc_pe;
  a.sc_imp = m.sc_imp;
  a.sc_htop = m.sc_htop;
  a.q_step = m.q_step;
  a.k_step = m.k_step;
  a.v_step = m.v_step;
  a.lse_step = m.lse_step;
  a.bits_step = m.bits_step;
  a.idx_step = m.idx_step;
  a.out_step = m.out_step;
}

hipError_t launch(StepArgs& a, const Workspace& w, hipStream_t s) {
  int total = 0;
  for (int st = 0; st < ST_N; ++st) {
    a.seg[st].first = total;
    a.end[st] = total += (a.seg[st].count + 7) & ~7;
  }
  if (total == 0) return hipSuccess;
  StepFn fn = pick(a.P);
  static_assert(sizeof(StepArgs) < 4096, "kernel argument block too large");
  hipLaunchKernelGGL(fn, dim3(total), dim3(kThreads), w.lds_bytes, s, a);
  return hipGetLastError();
}

// Stage st of pipeline layer v (layer v % L of step v / L); v outside the
// call's n_steps x L layers leaves the stage out of the launch.
void set_seg(StepArgs& a, int st, int v, int n_steps = 1) {
  if (v < 0 || v >= n_steps * a.P.L) {
    a.seg[st] = Seg{-1, 0, 0, 0, 0};
    return;
  }
  a.seg[st] = Seg{v % a.P.L, v % kRing, seg_count(a.P, st), v / a.P.L, 0};
}

// Pass 1, row normalisers and pass 2 of one layer into ring slot 0 (pass 2
// alone when the caller gives the row normalisers).  count_layer >= 0: the
// last launch also counts the caller's bitmap rows before that layer.
hipError_t score_stages(StepArgs a, const Workspace& w, hipStream_t s, int count_layer = -1) {
  const int order[3] = {ST_PASS1, ST_LSE, ST_PASS2};
  for (int i = a.lse ? 2 : 0; i < 3; ++i) {
    for (int st = 0; st < ST_N; ++st) a.seg[st] = Seg{-1, 0, 0, 0, 0};
    a.seg[order[i]] = Seg{0, 0, seg_count(a.P, order[i]), 0, 0};
    if (i == 2 && count_layer >= 0) a.seg[ST_CNTB] = Seg{count_layer, 0, seg_count(a.P, ST_CNTB), 0, 0};
    const hipError_t e = launch(a, w, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

constexpr int kCus = 256;

// A stage of the wide pipeline: without H_top heads nothing needs the extended rows.
int wide_stage(const Problem& P, int all, int base) { return P.delta_eff > 0 ? all : base; }

// Whether a model step runs the wide pipeline: all window rows that some head
// needs at once (four stages and launches shorter, two with given normalisers),
// instead of the extended rows of the H_top heads four launches later.  It scores
// more rows (all heads'), which costs nothing on compute units that would idle,
// so the line depends on what else a launch holds; P over O' has pool work-groups
// of its own, since one that pools both scores is the longest of a small launch.
//
// Keys in tiles of 128 (below 8k tokens) make score work-groups about twice as
// long as the launch's others (selection, pool, prep, gather), which have to fit
// beside them; seven or eight row blocks or float32 make them four times as long
// at d = 64, and at d = 128 so long that the others do not matter.  Larger key tiles
// leave room for the others too, but the more score work-groups there are the
// longer they run, which in a call of several steps, where only the last pays for
// the closing launches, no longer pays.
//
// Measured, us per step split / wide (score work-groups, others).  8 KV heads, G
// 4, d 128: 1k tokens 586 / 532 (64, 48), 2k 589 / 545 (128, 48), 3k 588 / 552
// (192, 48), two of 1k 647 / 610 (128, 104); given normalisers 4k 638 / 611 (128,
// 48), 12k 836 / 819 (188, 104), 24k 1240 / 1230 (188, 184), four of 1k 712 / 683
// (128, 200).  d 64, 4k given 555 / 532.  Qwen heads 16k 2027 / 1878 (128); 24 of
// 200 1212 / 1117 (192, 528).  float32, d 64: 1k 1095 / 974, 16 of 300 1273 / 1040
// (96, 384), five of 1k 1215 / 1125 (160, 256).  Over the line: two of 1.5k 655 /
// 697 (192, 112), given normalisers two of 3k 719 / 801 (192, 136), five of 1k 724 /
// 794 (160, 256), 4k 611 / 872 (256); float32, d 64, six of 1k 1229 / 1277 (192,
// 304).  Calls of six steps, given normalisers 16k 1102 / 1103 (128), 12k 763 / 773
// (188), 24k 1149 / 1193 (188).
bool wide_pays(const Problem& P, bool lse, int n_steps) {
  const int score = seg_count(P, wide_stage(P, ST_PASS2, ST_P2B)) +
                    (lse ? 0 : seg_count(P, wide_stage(P, ST_PASS1, ST_P1B)));
  if (score > kCus * 3 / 4) return false;
  const bool heavy = P.G >= 7 || P.esize == 4;
  if (heavy && (P.D == 128 || score <= kCus * 3 / 8)) return true;
  if (!heavy && P.tile1 > kTileMin) return n_steps == 1 || score <= kCus * 5 / 8;
  int others = P.delta_eff > 0 ? padded(P, ST_POOLE) : 0;
  for (int st : {ST_SELA, ST_SELECT, ST_POOLB, ST_PREP, ST_GATHER}) others += padded(P, st);
  return score + others / (heavy ? 4 : 2) <= kCus * 15 / 16;
}

// Key tiles per score work-group of a split-pipeline step.  About 10 of the 30-odd
// us that a work-group takes for 512 keys are fixed (code and first keys from
// memory, queries, normalisers, write-out), so where a launch has many rounds of
// work-groups, each takes two or four tiles in a row; with few rounds the coarser
// last round costs more than that saves.  The lines are in rounds of one
// work-group per compute unit, over the passes of a launch: two tiles from 2.5
// rounds (given normalisers: one pass) or 3.5 (two, which fill each other's last
// round) on, four from 10 on.  Pass 1 with seven row blocks at d = 128 spills more
// when it stores tile by tile, and with eight blocks four tiles never beat two.
//
// Measured, time against one tile by the work-groups of one tile in a launch; G 1 to
// 8, d 64 and 128, one long prompt and batches.  Given normalisers: 500 to 600 0.92
// to 1.20, 601 to 639 0.94 to 1.02, 640 to 700 0.93 to 1.01, 701 to 1000 0.84 to
// 1.02, 1001 to 1500 0.70 to 0.97 (four 0.81 to 1.10), 1501 to 2300 0.88 to 0.92
// (four 0.82 to 0.90), 2816 0.71 to 0.93 (four 0.71 to 0.89).  Two passes: 616 1.11,
// 704 0.94 to 1.09, 750 to 895 0.98 to 1.01, 896 to 990 0.95 to 1.02, 1000 to 1300
// 0.94 to 1.03, 1301 to 1600 0.89 to 0.98 (four 0.94 to 1.10), 1601 to 2300 0.93 to
// 0.96 (four 0.95 to 1.05), 2500 to 2900 0.92 to 0.97 (four 0.89 to 0.94).  Two passes
// at d = 128 with G 7 1.20 to 1.9 at any count, with G 8 0.83 at 2816 (four 0.94).
void lengthen_tiles(Problem& P, bool lse) {
  if (P.esize != 2 || P.tile1 != kTileMax || P.tile2 != kTileMax) return;
  auto pass = [&](int n_kt) { return (int64_t)P.batch * n_kt * P.n_rtg_base + ext_wgs(P, n_kt); };
  const int64_t n = pass(P.n_kt2) + (lse ? 0 : pass(P.n_kt1));
  int sub = n >= 10 * kCus ? 4 : 2 * n >= (lse ? 5 : 7) * kCus ? 2 : 1;
  if (!lse && P.D == 128 && P.G >= 7) sub = P.G == 7 ? 1 : sub > 2 ? 2 : sub;
  P.sub = sub;
  P.n_wt1 = (P.n_kt1 + sub - 1) / sub;
  P.n_wt2 = (P.n_kt2 + sub - 1) / sub;
}

hipError_t set_lds_limit(const Problem& P, const Workspace& w) {
  static_assert(kThreads == 512, "task code assumes 512-thread work-groups");
  if (w.lds_bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(pick(P)),
                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)w.lds_bytes);
}

int launches(const Problem& P, bool lse, int n_steps, bool wide) {
  return n_steps * P.L + (wide ? kPipeDepthWide - (lse ? 2 : 0) : lse ? kPipeDepthLse : kPipeDepth);
}

}  // namespace

int step_launches(const Problem& P, bool lse) { return launches(P, lse, 1, wide_pays(P, lse, 1)); }

hipError_t run_model(const Geometry& g, const ModelIO& m, char* ws, const Workspace& w,
                     hipStream_t s, hipEvent_t* ev) {
  const Problem& P = g.p;
  hipError_t e = set_lds_limit(P, w);
  if (e != hipSuccess) return e;
  StepArgs a = base_args(g, ws, w);
  set_model(a, m);
  a.idx_layer_stride = (int64_t)P.batch * P.H * P.B;
  a.out_layer = 1;
  a.standalone_counts = 0;
  // several steps: one pipeline over their n_steps x L layers in order (a
  // layer's selection chain only links layers of its own step)
  const int ns = m.n_steps > 0 ? m.n_steps : 1;
  // (the caller's score outputs hold the extended rows' scores of the H_top heads
  // only, as the split pipeline has them)
  const bool wide = !m.sc_p && wide_pays(P, m.lse != nullptr, ns);
  const int n_launch = launches(P, m.lse != nullptr, ns, wide);
  if (wide) {
    const int d = m.lse ? 2 : 0;  // stages that the given normalisers save
    for (int j = 0; j < n_launch; ++j) {
      if (!m.lse) {
        set_seg(a, wide_stage(P, ST_PASS1, ST_P1B), j, ns);
        set_seg(a, wide_stage(P, ST_LSE, ST_LSEB), j - 1, ns);
      }
      set_seg(a, wide_stage(P, ST_PASS2, ST_P2B), j - 2 + d, ns);
      set_seg(a, ST_POOLB, j - 3 + d, ns);
      if (P.delta_eff > 0) set_seg(a, ST_POOLE, j - 3 + d, ns);
      set_seg(a, ST_PREP, j - 4 + d, ns);
      set_seg(a, ST_SELA, j - 5 + d, ns);
      set_seg(a, ST_SELECT, j - 6 + d, ns);
      set_seg(a, ST_COUNT, j - 6 + d, ns);
      set_seg(a, ST_GATHER, j - 7 + d, ns);
      if (ev) (void)hipEventRecord(ev[j], s);
      if ((e = launch(a, w, s)) != hipSuccess) return e;
    }
    if (ev) (void)hipEventRecord(ev[n_launch], s);
    return hipSuccess;
  }
  lengthen_tiles(a.P, m.lse != nullptr);
  if ((e = set_lds_limit(a.P, w)) != hipSuccess) return e;
  if (m.lse) {
    // The row normalisers come from the caller (the log-sum-exp of the
    // layer's prefill attention): no pass 1, a shorter pipeline.
    for (int j = 0; j < n_launch; ++j) {
      set_seg(a, ST_P2B, j, ns);
      set_seg(a, ST_POOLB, j - 1, ns);
      set_seg(a, ST_P2X, j - 2, ns);
      set_seg(a, ST_POOLX, j - 3, ns);
      set_seg(a, ST_PREP, j - 4, ns);
      set_seg(a, ST_SELA, j - 5, ns);
      set_seg(a, ST_SELECT, j - 6, ns);
      set_seg(a, ST_COUNT, j - 6, ns);
      set_seg(a, ST_GATHER, j - 7, ns);
      if (ev) (void)hipEventRecord(ev[j], s);
      if ((e = launch(a, w, s)) != hipSuccess) return e;
    }
    if (ev) (void)hipEventRecord(ev[n_launch], s);
    return hipSuccess;
  }
  for (int j = 0; j < n_launch; ++j) {
    set_seg(a, ST_P1B, j, ns);
    set_seg(a, ST_LSEB, j - 1, ns);
    set_seg(a, ST_P2B, j - 2, ns);
    set_seg(a, ST_POOLB, j - 3, ns);
    set_seg(a, ST_P1X, j - 4, ns);
    set_seg(a, ST_LSEX, j - 5, ns);
    set_seg(a, ST_P2X, j - 6, ns);
    set_seg(a, ST_POOLX, j - 7, ns);
    set_seg(a, ST_PREP, j - 8, ns);
    set_seg(a, ST_SELA, j - 9, ns);
    set_seg(a, ST_SELECT, j - 10, ns);
    set_seg(a, ST_COUNT, j - 10, ns);
    set_seg(a, ST_GATHER, j - 11, ns);
    if (ev) (void)hipEventRecord(ev[j], s);
    if ((e = launch(a, w, s)) != hipSuccess) return e;
  }
  if (ev) (void)hipEventRecord(ev[n_launch], s);
  return hipSuccess;
}

hipError_t run_score(const Geometry& g, const void* q, const int64_t qs[3], const void* k,
                     const int64_t ks[3], const float* lse, const int64_t ls[2], float* p_raw,
                     float* p_ext, float* imp, char* ws, const Workspace& w, hipStream_t s) {
  const Problem& P = g.p;
  hipError_t e = set_lds_limit(P, w);
  if (e != hipSuccess) return e;
  StepArgs a = base_args(g, ws, w);
  a.q = static_cast<const char*>(q);
  a.k = static_cast<const char*>(k);
  for (int i = 0; i < 3; ++i) {
    a.qs[i + 1] = qs[i];
    a.ks[i + 1] = ks[i];
  }
  a.lse = lse;
  if (lse) {
    a.ls[1] = ls[0];
    a.ls[2] = ls[1];
  }
  if ((e = score_stages(a, w, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(finalize_kernel, dim3((P.Tc + 255) / 256, P.H + 1, P.batch), dim3(256), 0, s, P,
                     reinterpret_cast<const float*>(ws + w.psum_base),
                     reinterpret_cast<const float*>(ws + w.psum_all),
                     reinterpret_cast<const float*>(ws + w.ipart), p_raw, p_ext, imp);
  return hipGetLastError();
}

// Selection stages of one layer; scores from the caller (p_raw != null) or
// from the workspace partials of ring slot 0, whose last launch has counted
// the earlier layers' bitmap rows.
static hipError_t select_stages(const Geometry& g, int layer, const float* p_raw, const float* p_ext,
                                const float* imp, uint64_t* bits, int32_t* idx, uint32_t* htop,
                                char* ws, const Workspace& w, hipStream_t s) {
  const Problem& P = g.p;
  StepArgs a = base_args(g, ws, w);
  a.p_raw = p_raw;
  a.p_ext = p_ext;
  a.imp_in = imp;
  a.bits = bits;
  a.idx = idx;
  a.htop = htop;
  a.standalone_counts = 1;
  const int order[4] = {ST_CNTB, ST_POOL, ST_PREP, ST_SELAB};
  for (int i = p_raw ? 0 : 1; i < 4; ++i) {
    for (int st = 0; st < ST_N; ++st) a.seg[st] = Seg{-1, 0, 0, 0, 0};
    a.seg[order[i]] = Seg{layer, 0, seg_count(P, order[i]), 0, 0};
    const hipError_t e = launch(a, w, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t run_select(const Geometry& g, int layer, const float* p_raw, const float* p_ext,
                      const float* imp, uint64_t* bits, int32_t* idx, uint32_t* htop, char* ws,
                      const Workspace& w, hipStream_t s) {
  hipError_t e = set_lds_limit(g.p, w);
  if (e != hipSuccess) return e;
  return select_stages(g, layer, p_raw, p_ext, imp, bits, idx, htop, ws, w, s);
}

hipError_t run_evict_layer(const Geometry& g, int layer, const ModelIO& m, char* ws,
                           const Workspace& w, hipStream_t s) {
  const Problem& P = g.p;
  hipError_t e = set_lds_limit(P, w);
  if (e != hipSuccess) return e;
  StepArgs a = base_args(g, ws, w);
  set_model(a, m);
  // scores of this layer into ring slot 0 (the tensors carry no layer dimension)
  if ((e = score_stages(a, w, s, layer)) != hipSuccess) return e;
  if ((e = select_stages(g, layer, nullptr, nullptr, nullptr, m.bits, m.idx, nullptr, ws, w, s)) !=
      hipSuccess)
    return e;
  return run_compact(g, 1, m, s);
}

hipError_t run_compact(const Geometry& g, int n_layers, const ModelIO& m, hipStream_t s) {
  Workspace none;
  memset(&none, 0, sizeof(none));
  StepArgs a = base_args(g, nullptr, none);
  set_model(a, m);
  a.idx_layer_stride = (int64_t)g.p.batch * g.p.H * g.p.B;
  a.out_layer = 1;
  for (int l = 0; l < n_layers; ++l) {
    a.seg[ST_GATHER] = Seg{l, 0, seg_count(g.p, ST_GATHER), 0, 0};
    hipError_t e = launch(a, none, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t run_keep_all(const Geometry& g, int layer, uint64_t* bits, int32_t* idx, hipStream_t s) {
  const Problem& P = g.p;
  const int n = max(P.H * P.B, P.words);
  hipLaunchKernelGGL(keep_all_kernel, dim3((n + 255) / 256, P.batch), dim3(256), 0, s, idx, bits,
                     P.H, P.B, P.T, P.L, P.words, layer);
  return hipGetLastError();
}

hipError_t run_coverage(const Geometry& g, const uint64_t* bits, int upto, int64_t* count,
                        hipStream_t s) {
  hipLaunchKernelGGL(coverage_kernel, dim3(g.p.batch), dim3(256), 0, s, bits, count, g.p.L,
                     g.p.words, upto);
  return hipGetLastError();
}

}  // namespace kvec
