// Device side of a plan: workspace layout, batch execution (leaf gather ->
// contraction steps -> FP64 slice sum), hipGraph capture and replay, the
// adjoint sweep for gradients, tile autotuning and per-step profiling.
//
// Everything runs on the stream given to ltn_bind; the library allocates no
// device memory of its own (the caller's workspace holds leaf data,
// descriptors, slice ids, the per-slice arenas and gradient accumulators).
#include <algorithm>
#include <array>
#include <chrono>
#include <cstring>
#include <fstream>
#include <map>
#include <mutex>
#include <sstream>
#include <unordered_map>

#include "kernels.h"
#include "plan.h"

using namespace ltn;

#define HIPCHECK(x)                                                                     \
  do {                                                                                  \
    hipError_t e_ = (x);                                                                \
    if (e_ != hipSuccess)                                                               \
      fail(LTN_E_HIP, std::string(#x) + ": " + hipGetErrorString(e_) + " (" +         \
                          std::to_string((int)e_) + ")");                               \
  } while (0)

struct Layout {
  size_t leafdata, gd_fwd, gd_grad, gd_gcot, pl, angles, leafgrad, ids, scales, arena, split, gscr,
      gscr_c, skinny, splitk, gdesc, fdesc, total;
};

struct ltn_plan_impl {
  hipStream_t st = nullptr;
  hipStream_t cap = nullptr;  // capture stream (the null stream cannot be captured)
  char* ws = nullptr;
  size_t bytes = 0;
  int grad = 0;
  int B = 0;
  Layout lay{};
  int n_pl = 0;
  int max_leaf_elems = 1;
  int64_t gather_chunks = 0;  // blocks per slice of the leaf gather
  std::vector<GatherDesc> gd_fwd, gd_grad, gd_gcot;
  std::vector<ParamLeaf> pl;
  std::vector<int32_t> sl_bits, out_bits;
  bool fuse = true;  // run fused sub-paths in forward passes
  // kernel choice per mode and step: kind 0 = generic (tk threads per
  // output), 1 = complex64 MFMA GEMM, 2 = split MFMA GEMM (cfg, swap),
  // 3 = narrow-step kernel (swap: rows taken from the B operand), 4 = split
  // sum over k for steps with few outputs, 5 = split-K complex64 MFMA GEMM
  // (cfg, swap) for long sums with too few columns for a full tile, 6 =
  // complex64 product from three bf16 parts (cfg, swap)
  struct Choice {
    int kind = 0, cfg = -1, swap = 0, tk = 1;
  };
  std::vector<Choice> choice[3];
  // adjoint products (forward-form GEMMs of the gradient sweep) by shape
  // (m | k << 8 | n << 16): kind 1 = a complex64 tile, kind 5 = a split-K
  // tile, kind 6 = a three-part tile (cfg, swap) chosen by ltn_autotune;
  // absent = the fixed rule of enqueue_nt
  std::map<uint32_t, Choice> adj;
  std::vector<char> needs_grad;
  hipGraphExec_t graph[3] = {nullptr, nullptr, nullptr};
  hipGraph_t graph_src[3] = {nullptr, nullptr, nullptr};
  // gradients, full batches: recomputed forward and adjoint sweep
  hipGraphExec_t ggraph[2] = {nullptr, nullptr};
  hipGraph_t ggraph_src[2] = {nullptr, nullptr};
  // gradient launch sequence: runs of independent generic contractions of
  // consecutive steps share one launch (descriptors in the workspace)
  struct GradItem {
    // 0: forward step, 1: independent generic steps in one launch, 2: large
    // adjoint step, 3: fused group, 4: run of small steps (step 1: of adjoint
    // products; tk 2: with large inputs)
    int what = 0;
    int step = -1, off = 0, count = 0, tk = 1, lds = 0;
    uint64_t max_outs = 0;
    RunGroups groups{};
  };
  // forward kept in the gradient arena by the last ltn_execute (plan bound
  // for gradients, complex64, one batch) and its slice ids: ltn_execute_grad
  // on the same ids skips recomputing it; ltn_set_params and every other use
  // of the arena drop it
  bool fwd_kept = false;
  std::vector<uint64_t> fwd_ids;
  bool gseq_valid = false;
  std::vector<GenericDesc> gseq_descs;
  std::vector<GradItem> gseq_fwd, gseq_bwd;
  // forward launch sequence per mode, and whether any leaf has to be gathered
  // for it (runs of small steps read leaves where they lie)
  bool fseq_valid[3] = {false, false, false}, fseq_gather[3] = {true, true, true};
  std::vector<GenericDesc> fseq_descs[3];
  std::vector<GradItem> fseq[3];
  std::vector<uint64_t> host_ids;
};

namespace {

size_t al(size_t x) { return (x + 255) / 256 * 256; }

Layout layout(const ltn_plan* p, int B, int grad) {
  Layout l{};
  size_t o = 0;
  int npl = 0;
  for (auto& lp : p->leaves) npl += lp.param >= 0;
  l.leafdata = o;
  o = al(o + (size_t)p->leaf_elems * 8);
  l.gd_fwd = o;
  o = al(o + p->leaves.size() * sizeof(GatherDesc));
  l.fdesc = o;  // forward runs: one descriptor per step and mode
  o = al(o + 3 * std::max<size_t>(1, p->steps.size()) * sizeof(GenericDesc));
  l.gd_grad = o;
  o = al(o + (grad ? p->leaves.size() * sizeof(GatherDesc) : 0));
  l.gd_gcot = o;
  o = al(o + (grad ? p->leaves.size() * sizeof(GatherDesc) : 0));
  l.pl = o;
  o = al(o + (size_t)npl * sizeof(ParamLeaf));
  l.angles = o;
  o = al(o + (size_t)p->n_params * sizeof(double));
  l.leafgrad = o;
  o = al(o + (size_t)npl * 8 * sizeof(double));
  l.ids = o;
  o = al(o + (size_t)B * 8);
  l.scales = o;  // per tensor and slice: max |Re|, |Im|; then split_f16 bounds
  o = al(o + (size_t)B * p->tensors.size() * 8);
  l.arena = o;
  o = al(o + (size_t)B * (grad ? p->garena : p->arena));
  l.split = o;
  o = al(o + (size_t)B * p->split_scratch);
  // adjoint scratch: a permuted copy of an output cotangent and of one operand
  size_t sc = 0, so = 0;
  if (grad)
    for (auto& sp : p->steps) {
      sc = std::max<size_t>(sc, p->tensors[sp.out].bytes());
      so = std::max<size_t>(so, std::max(p->tensors[sp.a].bytes(), p->tensors[sp.b].bytes()));
    }
  l.gscr = o;
  o = al(o + (size_t)B * so);
  l.gscr_c = o;
  o = al(o + (size_t)B * sc);
  // partial sums of the few-output steps (largest over the steps that fit)
  int64_t sk = 0;
  for (auto& sp : p->steps)
    if (skinny_fits(sp.m, sp.k, sp.n)) sk = std::max<int64_t>(sk, skinny_part_elems(sp.m, sp.k, sp.n));
  l.skinny = o;
  o = al(o + (size_t)B * (size_t)sk * 8);
  // split-K partials (largest over the steps a split-K tile fits and, on
  // plans bound for gradients, over the adjoint products)
  int64_t kp = 0;
  for (auto& sp : p->steps) {
    kp = std::max<int64_t>(kp, splitk_part_elems(sp.m, sp.k, sp.n));
    if (grad) {
      kp = std::max<int64_t>(kp, splitk_part_elems(sp.m, sp.n, sp.k));
      kp = std::max<int64_t>(kp, splitk_part_elems(sp.n, sp.m, sp.k));
    }
  }
  l.splitk = o;
  o = al(o + (size_t)B * (size_t)kp * 8);
  l.gdesc = o;  // gradient runs: at most one descriptor per step forward, two backward
  if (grad) o = al(o + 3 * p->steps.size() * sizeof(GenericDesc));
  l.total = o;
  return l;
}

ltn_plan_impl& rt(ltn_plan* p) {
  if (!p || !p->rt || !p->rt->ws) fail(LTN_E_STATE, "plan is not bound (call ltn_bind first)");
  return *p->rt;
}

float2* arena_ptr(ltn_plan* p, uint64_t off_bytes) {
  auto& r = *p->rt;
  return reinterpret_cast<float2*>(r.ws + r.lay.arena + off_bytes * (uint64_t)r.B);
}

// Untuned FP32 tiles: the three-product tiles first, then the direct tiles
// 0-7 (sums shorter than 16).
int default_cfg(int m, int k, int n) {
  static const int c64_order[] = {10, 15, 13, 0, 1, 2, 3, 4, 5, 6, 7};
  for (int c : c64_order)
    if (gemm_config_fits(c, m, k, n, LTN_C64)) return c;
  return -1;
}

// Untuned split tiles for nb slices. Sums of 64 and more: the DMA-staged
// tiles, the largest of which every CU gets one ((13,12,11) fp16: 1.54 ms
// against 1.65 on the register-staged 128 x 128 tile; (11,10,10), 256 tiles
// of 128 x 64: 0.074 against 0.114; (10,10,10), 64 x 64: 0.056 against 0.107).
// Shorter sums with many tiles write more than they multiply: the register-
// staged 128 x 64 tile ((14,4,12): 0.113 against 0.118 for 128 x 128 and
// 0.129 with DMA). fp16 tiles raise a slice's maximum once a wave, and the waves of
// several slices queue at neighbouring slots: there the largest register-staged
// tiles ((10,4,8) x 32: 0.044 against 0.076 ms for 128 x 64, (9,4,8) x 256 0.095 against
// 0.120, (9,4,7) x 16 0.023 against 0.031 for 64 x 64; at 2^18 outputs 64 x 64 is 5 %
// faster), and for one slice from 2^22 outputs, where they are even. Sums of 2^6 are
// touched at 2^20 outputs only ((8,6,7) x 32: 0.027 against 0.032; 0.90 and 1.00 of the
// time a factor of two below and above).
int default_split_cfg(int m, int k, int n, int64_t nb, int mode) {
  const int64_t outs = m + n > 40 ? int64_t(1) << 40 : (int64_t(1) << (m + n)) * nb;
  const bool many = outs >> 14 >= 256, half = outs >> 13 >= 256;
  const bool queued = mode == LTN_SPLIT_F16 && (k < 6 ? (nb > 1 ? outs >> 19 : outs >> 22) > 0
                                                      : k == 6 && nb > 1 && !half && outs >> 20 > 0);
  static const int large[] = {10, 11, 12, 13}, middle[] = {11, 12, 13}, small_[] = {13}, brief[] = {1, 2, 3};
  const int* order = k >= 6 ? (many ? large : half ? middle : small_) : (many ? brief : small_);
  const int len = k >= 6 ? (many ? 4 : half ? 3 : 1) : (many ? 3 : 1);
  for (int i = 0; i < len && !queued; ++i)
    if (gemm_config_fits(order[i], m, k, n, mode)) return order[i];
  for (int c = 0; c < gemm_config_count(mode); ++c)
    if (gemm_config_fits(c, m, k, n, mode)) return c;
  return -1;
}

int default_tk(int k, uint64_t outs) {
  int tk = k <= 3 ? 1 : (k <= 6 ? 8 : 64);
  if (outs < (1u << 16) && k >= 3) tk = std::max(tk, 8);
  if (outs < (1u << 12) && k >= 5) tk = 64;
  return tk;
}

uint32_t* slot(ltn_plan* p, int tensor) {
  auto& r = *p->rt;
  return reinterpret_cast<uint32_t*>(r.ws + r.lay.scales) + (size_t)tensor * r.B;
}

// split_f16: the bound whose scale a producer used to write the tensor in
// the split layout (read by the consumer in place of the tensor's maximum)
uint32_t* bound_slot(ltn_plan* p, int tensor) {
  return slot(p, (int)p->tensors.size() + tensor);
}

// Split modes: a tensor that a matrix-core step produces and a split step
// consumes is written by its producer in the split layout, and the
// conversion pass before the consumer is skipped. bf16 needs no scale; for
// fp16 the producer cannot know its output's maximum before writing, so it
// scales by the bound 2 K max|a| max|b| taken from its operands' recorded
// maxima (stored for the consumer). Steps run inside a fused sub-path read
// and write complex64, and the gradient's recomputed forward stays complex64.
bool split_direct(ltn_plan* p, int t, int mode, bool gradarena) {
  if (mode == LTN_C64 || gradarena) return false;
  auto& r = *p->rt;
  const TensorPlan& T = p->tensors[t];
  if (T.producer < 0 || T.consumer < 0) return false;
  auto fused = [&](int s) { return r.fuse && p->step_group[s] >= 0; };
  if (fused(T.producer) || fused(T.consumer)) return false;
  const auto& pc = r.choice[mode][T.producer];
  const bool writes = pc.kind == 1 || pc.kind == 2 || (pc.kind == 6 && !parts_config_splitk(pc.cfg));
  return writes && r.choice[mode][T.consumer].kind == 2;
}

// The generic kernel's descriptor for forward step s.
GenericDesc step_generic_desc(ltn_plan* p, int s, int nb, bool gradarena, int mode) {
  const StepPlan& sp = p->steps[s];
  const TensorPlan &ta = p->tensors[sp.a], &tb = p->tensors[sp.b], &tc = p->tensors[sp.out];
  const uint64_t cm = sp.c_mask_a, full = (sp.m + sp.n) >= 64 ? ~0ull : ((1ull << (sp.m + sp.n)) - 1);
  GenericDesc g{};
  g.P = arena_ptr(p, gradarena ? ta.goff : ta.off);
  g.Q = arena_ptr(p, gradarena ? tb.goff : tb.off);
  g.out = arena_ptr(p, gradarena ? tc.goff : tc.off);
  g.sP = int64_t(1) << ta.rank;
  g.sQ = int64_t(1) << tb.rank;
  g.sO = int64_t(1) << tc.rank;
  g.set_shape(sp.m, sp.n, sp.k, false);
  g.px = ((1ull << sp.m) - 1) << sp.k;
  g.pz = (1ull << sp.k) - 1;
  g.qy = ((1ull << sp.n) - 1) << sp.k;
  g.qz = (1ull << sp.k) - 1;
  g.ox = cm;
  g.oy = ~cm & full;
  g.nb = nb;
  if (mode == LTN_SPLIT_F16) g.scale_out = slot(p, sp.out);
  return g;
}

void enqueue_step(ltn_plan* p, int s, int nb, bool gradarena, int mode) {
  auto& r = *p->rt;
  const StepPlan& sp = p->steps[s];
  const TensorPlan &ta = p->tensors[sp.a], &tb = p->tensors[sp.b], &tc = p->tensors[sp.out];
  float2* A = arena_ptr(p, gradarena ? ta.goff : ta.off);
  float2* B = arena_ptr(p, gradarena ? tb.goff : tb.off);
  float2* C = arena_ptr(p, gradarena ? tc.goff : tc.off);
  const uint64_t cm = sp.c_mask_a, full = (sp.m + sp.n) >= 64 ? ~0ull : ((1ull << (sp.m + sp.n)) - 1);
  const auto& ch = r.choice[mode][s];
  const bool split = mode != LTN_C64;
  if (ch.kind == 4) {
    SkinnyDesc d{};
    d.A = A;
    d.B = B;
    d.C = C;
    d.sA = int64_t(1) << ta.rank;
    d.sB = int64_t(1) << tb.rank;
    d.sC = int64_t(1) << tc.rank;
    d.m = sp.m;
    d.k = sp.k;
    d.n = sp.n;
    d.cmask = cm;
    d.nb = nb;
    d.part = reinterpret_cast<float2*>(r.ws + r.lay.skinny);
    if (mode == LTN_SPLIT_F16) d.scale_c = slot(p, sp.out);
    launch_skinny(d, r.st);
    return;
  }
  if (ch.kind == 5) {
    GemmDesc d{};
    const bool sw = ch.swap;
    d.A = sw ? B : A;
    d.B = sw ? A : B;
    d.C = C;
    d.sA = int64_t(1) << (sw ? tb.rank : ta.rank);
    d.sB = int64_t(1) << (sw ? ta.rank : tb.rank);
    d.sC = int64_t(1) << tc.rank;
    d.m = sw ? sp.n : sp.m;
    d.n = sw ? sp.m : sp.n;
    d.k = sp.k;
    d.cmask = sw ? (~cm & full) : cm;
    d.nb = nb;
    d.cfg = ch.cfg;
    d.part = reinterpret_cast<float2*>(r.ws + r.lay.splitk);
    if (mode == LTN_SPLIT_F16) d.scale_c = slot(p, sp.out);
    launch_cgemm_splitk(d, r.st);
    return;
  }
  if (ch.kind == 3) {
    NarrowDesc d{};
    const bool sw = ch.swap;
    d.A = sw ? B : A;
    d.B = sw ? A : B;
    d.C = C;
    d.sA = int64_t(1) << (sw ? tb.rank : ta.rank);
    d.sB = int64_t(1) << (sw ? ta.rank : tb.rank);
    d.sC = int64_t(1) << tc.rank;
    d.m = sw ? sp.n : sp.m;
    d.n = sw ? sp.m : sp.n;
    d.k = sp.k;
    d.cmask = sw ? (~cm & full) : cm;
    d.nb = nb;
    d.cfg = ch.cfg;
    if (mode == LTN_SPLIT_F16) d.scale_c = slot(p, sp.out);
    launch_narrow(d, r.st);
    return;
  }
  if (ch.kind > 0) {
    GemmDesc d{};
    bool sw = ch.swap;
    d.A = sw ? B : A;
    d.B = sw ? A : B;
    d.C = C;
    d.sA = int64_t(1) << (sw ? tb.rank : ta.rank);
    d.sB = int64_t(1) << (sw ? ta.rank : tb.rank);
    d.sC = int64_t(1) << tc.rank;
    d.m = sw ? sp.n : sp.m;
    d.n = sw ? sp.m : sp.n;
    d.k = sp.k;
    d.cmask = sw ? (~cm & full) : cm;
    d.nb = nb;
    d.cfg = ch.cfg;
    const bool f16 = mode == LTN_SPLIT_F16;
    if (f16) d.scale_c = slot(p, sp.out);
    if (split_direct(p, sp.out, mode, gradarena)) {
      d.split_out = f16 ? 2 : 1;
      if (f16) {
        d.max_a = slot(p, sw ? sp.b : sp.a);
        d.max_b = slot(p, sw ? sp.a : sp.b);
        d.bound_c = bound_slot(p, sp.out);
      }
    }
    if (ch.kind == 2) {
      // split-layout copies of both operands in the per-batch scratch area,
      // unless the producer wrote them so
      float2* As = reinterpret_cast<float2*>(r.ws + r.lay.split);
      float2* Bs = As + (((ta.bytes() + 255) / 256 * 256) / 8) * (uint64_t)r.B;
      if (split_direct(p, sp.a, mode, gradarena))
        As = A;
      else
        launch_split_convert(A, As, ta.rank, nb, f16 ? slot(p, sp.a) : nullptr, mode, r.st);
      if (split_direct(p, sp.b, mode, gradarena))
        Bs = B;
      else
        launch_split_convert(B, Bs, tb.rank, nb, f16 ? slot(p, sp.b) : nullptr, mode, r.st);
      d.A = sw ? Bs : As;
      d.B = sw ? As : Bs;
      if (f16) {
        // the maximum the operand's split copy was scaled by, or the bound
        // its producer used
        const int ra = sw ? sp.b : sp.a, rb = sw ? sp.a : sp.b;
        d.scale_a = split_direct(p, ra, mode, gradarena) ? bound_slot(p, ra) : slot(p, ra);
        d.scale_b = split_direct(p, rb, mode, gradarena) ? bound_slot(p, rb) : slot(p, rb);
      }
    }
    if (ch.kind == 6) {
      if (f16) {
        d.scale_a = slot(p, sw ? sp.b : sp.a);
        d.scale_b = slot(p, sw ? sp.a : sp.b);
      }
      d.part = reinterpret_cast<float2*>(r.ws + r.lay.splitk);
      launch_cgemm_parts(d, r.st);
    } else {
      launch_cgemm(d, ch.kind == 2 ? mode : LTN_C64, r.st);
    }
  } else {
    GenericDesc g = step_generic_desc(p, s, nb, gradarena, mode);
    launch_generic(g, ch.tk, r.st);
  }
}

// A fused sub-path at its last step (the plan keeps T_0 and the small
// tensors live until then).
void enqueue_group(ltn_plan* p, int g, int nb, int mode) {
  auto& r = *p->rt;
  const FuseGroup& G = p->groups[g];
  FusedDesc d{};
  d.X0 = arena_ptr(p, p->tensors[G.t0].off);
  d.XL = arena_ptr(p, p->tensors[G.tl].off);
  d.sX0 = int64_t(1) << p->tensors[G.t0].rank;
  d.sXL = int64_t(1) << p->tensors[G.tl].rank;
  d.a = G.a;
  d.nsig = G.nsig;
  d.c = G.c;
  d.rmax = G.rmax;
  d.nstages = (int32_t)G.st.size();
  d.nb = nb;
  d.sig_out = G.sig_out;
  d.w_out = G.w_out;
  if (mode == LTN_SPLIT_F16) d.scale_c = slot(p, G.tl);
  int yoff = 0;
  for (int j = 0; j < d.nstages; ++j) {
    const FuseStage& s = G.st[j];
    FusedStage& f = d.st[j];
    f.Y = arena_ptr(p, p->tensors[s.other].off);
    f.sY = int64_t(1) << p->tensors[s.other].rank;
    f.m = s.m;
    f.k = s.k;
    f.n = s.n;
    f.cmask = s.cmask;
    f.yoff = yoff;
    yoff += 1 << (s.k + s.n);
  }
  d.y_elems = yoff;
  launch_fused(d, r.st);
}

// A launch of generic contractions (what 1 or 4) from descriptors in memory.
void enqueue_generic(ltn_plan* p, const GenericDesc* dd, const ltn_plan_impl::GradItem& it, int nb) {
  if (it.what == 4)
    launch_small_run(dd + it.off, it.groups, it.step == 1, it.tk == 2, it.lds,
                     reinterpret_cast<const float2*>(p->rt->ws + p->rt->lay.leafdata),
                     reinterpret_cast<const uint64_t*>(p->rt->ws + p->rt->lay.ids), nb, p->rt->st);
  else
    launch_generic_multi(dd + it.off, it.count, it.max_outs, nb, it.tk, p->rt->st);
}

void enqueue_forward(ltn_plan* p, int nb, bool gradarena, int mode) {
  auto& r = *p->rt;
  const GatherDesc* gd = reinterpret_cast<const GatherDesc*>(r.ws + (gradarena ? r.lay.gd_grad : r.lay.gd_fwd));
  uint32_t* scales = nullptr;
  if (mode == LTN_SPLIT_F16) {
    scales = reinterpret_cast<uint32_t*>(r.ws + r.lay.scales);
    launch_fill_zero(scales, al((size_t)r.B * p->tensors.size() * 4), r.st);
  }
  if (gradarena || !r.fseq_valid[mode] || r.fseq_gather[mode])
    launch_gather(gd, (int)p->leaves.size(), r.gather_chunks, r.max_leaf_elems,
                  reinterpret_cast<const float2*>(r.ws + r.lay.leafdata), arena_ptr(p, 0),
                  reinterpret_cast<const uint64_t*>(r.ws + r.lay.ids), nb, scales, r.B, r.st);
  if (gradarena && r.gseq_valid) {
    const GenericDesc* dd = reinterpret_cast<const GenericDesc*>(r.ws + r.lay.gdesc);
    for (const auto& it : r.gseq_fwd) {
      if (it.what == 0)
        enqueue_step(p, it.step, nb, true, mode);
      else
        enqueue_generic(p, dd, it, nb);
    }
    return;
  }
  if (!gradarena && r.fseq_valid[mode]) {
    const GenericDesc* dd =
        reinterpret_cast<const GenericDesc*>(r.ws + r.lay.fdesc) + (size_t)mode * p->steps.size();
    for (const auto& it : r.fseq[mode]) {
      if (it.what == 0)
        enqueue_step(p, it.step, nb, false, mode);
      else if (it.what == 3)
        enqueue_group(p, it.step, nb, mode);
      else
        enqueue_generic(p, dd, it, nb);
    }
    return;
  }
  for (int s = 0; s < (int)p->steps.size(); ++s) {
    const int g = p->step_group[s];
    if (g >= 0 && r.fuse && !gradarena) {
      if (s == p->groups[g].st.back().step) enqueue_group(p, g, nb, mode);
      continue;
    }
    enqueue_step(p, s, nb, gradarena, mode);
  }
}

// A generic contraction in a launch sequence: what it reads and writes (ids:
// tensor t, or n_tensors + t for its cotangent; per-slice byte ranges of the
// arena), the step whose contractions consume its output (-1: not one of this
// sequence), and whether the output is needed in memory even so.
struct SeqOp {
  GenericDesc g;
  int tk = 1, step = -1, consumer = -1;
  int in[2] = {-1, -1}, out = -1;
  struct Range {
    uint64_t lo, hi;
    bool meets(const Range& o) const { return lo < o.hi && o.lo < hi; }
  } rin[2], rout;
  bool keep = false;
  const GatherDesc* leaf[2] = {nullptr, nullptr};  // device descriptor of an operand that is a leaf
  int work() const { return g.xb() + g.yb() + g.zb(); }
};

// Runs of small steps: at most 2^15 multiply-adds a step (one block's work of
// about a launch: 512 threads take 3.5 us), 64 KiB of LDS (two blocks per CU).
// Up to 2^11 a step is one wave's when others share its level.
// Adjoint steps from 2^13 multiply-adds on take k_rowsum where it fits: 256 slices
// of (6,2,6) 13 us a product, 25 in a launch of several generic ones; between 2^11
// and 2^14 the line makes no difference.
constexpr int kRowsumWork = 13;
constexpr int kRunWork = 15, kWaveWork = 11, kRunSteps = 96, kRunLds = 8192;

// Which step of ops[i .. j) produces an operand (-1: none), and which outputs are
// needed in memory.
struct RunLinks {
  std::vector<std::array<int, 2>> from;
  std::vector<char> ext;
  RunLinks(const std::vector<SeqOp>& ops, int i, int j) : from(j - i, {-1, -1}), ext(j - i, 1) {
    std::unordered_map<int, int> made, step_of;
    for (int k = 0; k < j - i; ++k) {
      const SeqOp& o = ops[i + k];
      for (int q = 0; q < 2; ++q)
        if (auto it = made.find(o.in[q]); it != made.end()) from[k][q] = it->second;
      made[o.out] = k;
      step_of[o.step] = k;
    }
    for (int k = 0; k < j - i; ++k)
      if (auto it = step_of.find(ops[i + k].consumer); !ops[i + k].keep && it != step_of.end() && it->second > k)
        ext[k] = 0;
  }
};

// Whether a block of the run ops[i .. j) could write memory that another block
// of it still reads or writes: the arena reuses memory across tensors, whose
// slices then overlap.
bool run_clashes(const std::vector<SeqOp>& ops, int i, int j, const RunLinks& l) {
  for (int k = 0; k < j - i; ++k) {
    if (!l.ext[k]) continue;
    const auto& w = ops[i + k].rout;
    for (int m = 0; m < j - i; ++m) {
      if (m != k && l.ext[m] && w.meets(ops[i + m].rout)) return true;
      for (int q = 0; q < 2; ++q)
        if (l.from[m][q] < 0 && !ops[i + m].leaf[q] && w.meets(ops[i + m].rin[q])) return true;
    }
  }
  return false;
}

// Plan ops as the run of one block: levels by dependence, places in LDS by first
// fit over the levels a tensor is needed in, waves. False when LDS does not hold
// it.
bool plan_run(const std::vector<SeqOp>& ops, std::vector<GenericDesc>& out, int& lds) {
  constexpr int i = 0;
  const int j = (int)ops.size();
  const int n = j - i;
  struct Place {
    int off, size, from, to;
  };
  std::vector<Place> placed;
  // the lowest gap among those placed (in order of place) that are needed at
  // the same time
  auto place = [&](int size, int from, int to) {
    int off = 0;
    for (const Place& q : placed) {
      if (q.from > to || from > q.to) continue;
      if (off + size <= q.off) break;
      off = std::max(off, q.off + q.size);
    }
    placed.insert(std::upper_bound(placed.begin(), placed.end(), off,
                                   [](int o, const Place& q) { return o < q.off; }),
                  {off, size, from, to});
    lds = std::max(lds, off + size);
    return off;
  };
  const RunLinks links(ops, i, j);
  const auto& from = links.from;
  const auto& ext = links.ext;
  std::vector<int> level(n, 1), last(n, 0);
  for (int k = 0; k < n; ++k) {
    for (int q = 0; q < 2; ++q)
      if (from[k][q] >= 0) level[k] = std::max(level[k], level[from[k][q]] + 1);
    for (int q = 0; q < 2; ++q)
      if (from[k][q] >= 0) last[from[k][q]] = std::max(last[from[k][q]], level[k]);
  }
  lds = 0;
  std::vector<std::array<int, 3>> at(n, {-1, -1, -1});
  for (int k = 0; k < n; ++k) {
    const GenericDesc& g = ops[i + k].g;
    const int size[2] = {1 << (g.xb() + g.zb()), 1 << (g.yb() + g.zb())};
    for (int q = 0; q < 2; ++q)
      if (from[k][q] >= 0)
        at[k][q] = at[from[k][q]][2];
      else
        at[k][q] = place(size[q], 0, level[k]);
    if (last[k]) at[k][2] = place(1 << (g.xb() + g.yb()), level[k], last[k]);
    if (lds > kRunLds) return false;
  }
  // address tables behind the tensors, 16 bits an entry
  std::vector<int> table(n);
  int words = 4 * lds;
  for (int k = 0; k < n; ++k) {
    const GenericDesc& g = ops[i + k].g;
    table[k] = words;
    words += (1 << g.xb()) + (1 << (g.conjQ() ? g.zb() : g.yb()));
  }
  lds = (words + 3) / 4;
  if (lds > kRunLds) return false;
  std::vector<int> order(n);
  for (int k = 0; k < n; ++k) order[k] = k;
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return level[a] < level[b]; });
  const int waves = small_run_waves();
  for (int a = 0; a < n;) {
    int e = a;
    while (e < n && level[order[e]] == level[order[a]]) ++e;
    int w = 0;
    for (int x = a; x < e; ++x) {
      const int k = order[x];
      GenericDesc g = ops[i + k].g;
      // a step of the block's own unless several share the level
      const bool own = e - a >= 2 && ops[i + k].work() <= (e - a >= waves / 2 ? kWaveWork : 9);
      if (from[k][0] >= 0) g.P = nullptr;
      if (from[k][1] >= 0) g.Q = nullptr;
      const SeqOp& o = ops[i + k];
      if (o.leaf[0]) g.P = reinterpret_cast<const float2*>(o.leaf[0]);
      if (o.leaf[1]) g.Q = reinterpret_cast<const float2*>(o.leaf[1]);
      if (!ext[k]) {
        g.out = nullptr;
        g.scale_out = nullptr;  // only matrix-core consumers read the maxima
      }
      // the step's partial sums per output, one lane each while there are threads
      const int tk = o.tk == 1 ? 0 : (o.tk == 8 ? 3 : 6);
      const int sums = tk == 0 ? 0 : (tk == 3 ? 1 : 3) + (g.xb() + g.yb() + tk > (own ? 6 : 9));
      g.nb = table[k];
      g.places = (uint32_t)(at[k][0] + 1) | (uint32_t)(at[k][1] + 1) << 16;
      g.plan = (uint32_t)(at[k][2] + 1) | (own ? (uint32_t)(w++ % waves) + 1u : 0u) << 16 | (uint32_t)sums << 20 |
               (x == a ? 1u << 23 : 0u) | (o.leaf[0] ? 1u << 24 : 0u) | (o.leaf[1] ? 1u << 25 : 0u);
      out.push_back(g);
    }
    a = e;
  }
  return true;
}

// Plan ops[i .. j) as one run of nb slices: steps that depend on each other stay
// together, and what does not is spread over up to eight blocks per slice while
// that gives no more than two blocks a CU (a run is a chain of latencies: 64
// slices of a 20-qubit circuit's first 96 steps on one block each 42 us). `reused`:
// the arena's memory serves several tensors; with one block, which has read its
// inputs before it writes, that does not matter.
bool plan_groups(const std::vector<SeqOp>& ops, int i, int j, int nb, bool reused, std::vector<GenericDesc>& out,
                 RunGroups& groups, int& lds) {
  const int n = j - i;
  const RunLinks links(ops, i, j);
  // trees of the run: the last step of a tree stands for it
  std::vector<int> root(n);
  for (int k = 0; k < n; ++k) root[k] = k;
  auto find = [&](int k) {
    while (root[k] != k) k = root[k] = root[root[k]];
    return k;
  };
  for (int k = 0; k < n; ++k)
    for (int q = 0; q < 2; ++q)
      if (links.from[k][q] >= 0) root[find(links.from[k][q])] = find(k);
  std::vector<std::pair<int, int>> trees;  // cost, root
  std::vector<int> cost(n, 0);
  for (int k = 0; k < n; ++k) cost[find(k)] += 2 + (1 << std::max(0, ops[i + k].work() - 9));
  for (int k = 0; k < n; ++k)
    if (root[k] == k) trees.push_back({cost[k], k});
  int G = std::max(1, std::min({(int)trees.size(), kRunGroups, 512 / nb}));
  if (reused && (nb > 1 || G > 1) && run_clashes(ops, i, j, links)) {
    if (nb > 1) return false;
    G = 1;
  }
  std::sort(trees.begin(), trees.end(), [](auto& a, auto& b) { return a.first > b.first; });
  std::vector<int> load(G, 0), group(n, 0);
  for (auto& t : trees) {
    const int g = (int)(std::min_element(load.begin(), load.end()) - load.begin());
    load[g] += t.first;
    group[t.second] = g;
  }
  groups = RunGroups{};
  groups.n = G;
  lds = 0;
  for (int g = 0; g < G; ++g) {
    std::vector<SeqOp> mine;
    for (int k = 0; k < n; ++k)
      if (group[find(k)] == g) mine.push_back(ops[i + k]);
    int size = 0;
    if (!plan_run(mine, out, size)) return false;
    lds = std::max(lds, size);
    groups.off[g + 1] = (int)out.size();
  }
  return true;
}

// Launches of consecutive generic contractions: runs of small steps where two
// or more fit one, else launches of independent steps (a step joins the launch
// unless it reads, or writes over, what a member writes, or writes over what a
// member reads).
void sequence_generic(const std::vector<SeqOp>& ops, int nb, bool reused, std::vector<GenericDesc>& descs,
                      std::vector<ltn_plan_impl::GradItem>& seq) {
  using Item = ltn_plan_impl::GradItem;
  std::vector<const SeqOp*> group;
  auto flush = [&]() {
    for (int tk : {1, 8, 64}) {
      Item it;
      it.what = 1;
      it.tk = tk;
      it.off = (int)descs.size();
      for (auto* e : group)
        if (e->tk == tk) {
          descs.push_back(e->g);
          it.max_outs = std::max<uint64_t>(it.max_outs, 1ull << (e->g.xb() + e->g.yb()));
        }
      it.count = (int)descs.size() - it.off;
      if (it.count) seq.push_back(it);
    }
    group.clear();
  };
  const int n = (int)ops.size();
  for (int i = 0; i < n;) {
    int j = i;
    while (j < n && j - i < kRunSteps && ops[j].work() <= kRunWork) ++j;
    // the longest run, by bisection; contractions of one step (the two of an
    // adjoint step) stay together
    std::vector<GenericDesc> run, longer;
    int lds = 0, fits = i, fails = j + 1;
    RunGroups groups{}, more;
    for (int t = j; fails - fits > 1; t = (fits + fails) / 2) {
      int e = t;
      while (e < n && e > fits && ops[e].step == ops[e - 1].step) --e;
      longer.clear();
      int size = 0;
      if (e <= i + 1) {
        fails = t;  // too short
      } else if (e > fits && plan_groups(ops, i, e, nb, reused, longer, more, size)) {
        fits = t;
        j = e;
        lds = size;
        groups = more;
        run.swap(longer);
      } else {
        fails = t;
      }
    }
    if (run.empty()) j = i;
    if (j - i >= 2) {
      flush();
      Item it;
      it.what = 4;
      it.off = (int)descs.size();
      it.count = j - i;
      it.lds = lds;
      it.groups = groups;
      it.step = run[0].conjQ() ? 1 : 0;
      for (auto& g : run) {
        const int p = g.P ? 1 << (g.xb() + g.zb()) : 0, q = g.Q ? 1 << (g.yb() + g.zb()) : 0;
        if (std::max(p, q) > small_run_side()) it.tk = 2;
      }
      descs.insert(descs.end(), run.begin(), run.end());
      seq.push_back(it);
      i = j;
      continue;
    }
    const SeqOp& o = ops[i++];
    bool clash = false;
    for (auto* e : group)
      clash = clash || e->rout.meets(o.rin[0]) || e->rout.meets(o.rin[1]) || e->rout.meets(o.rout) ||
              e->rin[0].meets(o.rout) || e->rin[1].meets(o.rout);
    if (clash) flush();
    group.push_back(&o);
  }
  flush();
}

SeqOp step_seq_op(ltn_plan* p, int s, bool gradarena, int mode) {
  const StepPlan& sp = p->steps[s];
  SeqOp o;
  o.g = step_generic_desc(p, s, p->rt->B, gradarena, mode);
  o.tk = p->rt->choice[mode][s].tk;
  o.step = s;
  o.consumer = p->tensors[sp.out].consumer;
  o.keep = gradarena;  // the adjoint sweep reads it
  auto range = [&](int t) {
    const TensorPlan& T = p->tensors[t];
    const uint64_t off = gradarena ? T.goff : T.off;
    return SeqOp::Range{off, off + T.bytes()};
  };
  const int in[2] = {sp.a, sp.b};
  for (int q = 0; q < 2; ++q) {
    o.in[q] = in[q];
    o.rin[q] = range(in[q]);
    // a run reads leaves where they lie; the adjoint sweep wants them gathered
    if (in[q] < p->L && !gradarena)
      o.leaf[q] = reinterpret_cast<const GatherDesc*>(p->rt->ws + p->rt->lay.gd_fwd) + in[q];
  }
  o.out = sp.out;
  o.rout = range(sp.out);
  return o;
}

// Forward launch sequence of a mode. Fused sub-paths keep their launch at
// their last step. Descriptors (for the bound batch size) are copied to the
// workspace here, outside any capture.
void build_fwd_seq(ltn_plan* p, int mode, bool upload = true) {
  auto& r = *p->rt;
  using Item = ltn_plan_impl::GradItem;
  auto& seq = r.fseq[mode];
  auto& descs = r.fseq_descs[mode];
  seq.clear();
  descs.clear();
  std::vector<SeqOp> ops;
  auto single = [&](int what, int step) {
    sequence_generic(ops, r.B, true, descs, seq);
    ops.clear();
    Item it;
    it.what = what;
    it.step = step;
    seq.push_back(it);
  };
  for (int s = 0; s < (int)p->steps.size(); ++s) {
    const int g = p->step_group[s];
    if (g >= 0 && r.fuse) {
      if (s == p->groups[g].st.back().step) single(3, g);
    } else if (r.choice[mode][s].kind != 0) {
      single(0, s);
    } else {
      ops.push_back(step_seq_op(p, s, false, mode));
    }
  }
  sequence_generic(ops, r.B, true, descs, seq);
  int from_leaves = 0;  // leaf operands that runs read themselves
  for (const Item& it : seq)
    for (int i = 0; i < it.count && it.what == 4; ++i)
      from_leaves += descs[it.off + i].leafP() + descs[it.off + i].leafQ();
  r.fseq_gather[mode] = from_leaves < (int)p->leaves.size();
  require(descs.size() <= p->steps.size(), "forward descriptor area too small");
  if (!descs.empty() && upload) {
    char* dst = r.ws + r.lay.fdesc + (size_t)mode * p->steps.size() * sizeof(GenericDesc);
    HIPCHECK(hipMemcpyAsync(dst, descs.data(), descs.size() * sizeof(GenericDesc), hipMemcpyHostToDevice, r.st));
    // the host array may be rebuilt by a later call: let the copy finish
    HIPCHECK(hipStreamSynchronize(r.st));
  }
  r.fseq_valid[mode] = true;
}

void enqueue_reduce(ltn_plan* p, int nb, bool gradarena, double* out) {
  auto& r = *p->rt;
  const TensorPlan& root = p->tensors[p->root];
  launch_reduce(arena_ptr(p, gradarena ? root.goff : root.off), root.rank, p->out_mask,
                r.sl_bits.data(), r.out_bits.data(), (int)r.sl_bits.size(),
                reinterpret_cast<const uint64_t*>(r.ws + r.lay.ids), nb, out, r.st);
}

void set_ids(ltn_plan* p, const uint64_t* ids, uint64_t base, int n, bool range) {
  auto& r = *p->rt;
  uint64_t* d = reinterpret_cast<uint64_t*>(r.ws + r.lay.ids);
  if (range)
    launch_set_range(d, base, n, r.st);
  else
    launch_set_ids(d, ids, n, r.st);
}

void check_launch() {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) fail(LTN_E_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
}

// Launch the work `enqueue` issues as one graph on the bound stream,
// capturing it (on a stream of our own) the first time. The captured
// kernels keep their arguments, so only work whose pointers and shapes are
// fixed for the bound workspace goes in.
template <typename F>
void launch_captured(ltn_plan* p, hipGraphExec_t& exec, hipGraph_t& src, F&& enqueue) {
  auto& r = *p->rt;
  if (!exec) {
    if (!r.cap) HIPCHECK(hipStreamCreateWithFlags(&r.cap, hipStreamNonBlocking));
    hipGraph_t g;
    hipStream_t bound = r.st;
    r.st = r.cap;
    hipError_t e = hipStreamBeginCapture(r.cap, hipStreamCaptureModeThreadLocal);
    if (e == hipSuccess) {
      try {
        enqueue();
      } catch (...) {
        r.st = bound;
        (void)hipStreamEndCapture(r.cap, &g);
        throw;
      }
      e = hipStreamEndCapture(r.cap, &g);
    }
    r.st = bound;
    if (e != hipSuccess) fail(LTN_E_HIP, std::string("graph capture: ") + hipGetErrorString(e));
    HIPCHECK(hipGraphInstantiate(&exec, g, nullptr, nullptr, 0));
    src = g;
  }
  HIPCHECK(hipGraphLaunch(exec, r.st));
}

void run_batch(ltn_plan* p, int nb, int mode, double* out) {
  auto& r = *p->rt;
  if (!r.fseq_valid[mode]) build_fwd_seq(p, mode);
  // A graph pays from about ten launches: one costs 3 us directly and 10 us as a
  // graph, calls of six to eight in a row 60 -> 54 and 77 -> 73 us directly, and at
  // 16 a call alone takes longer (95 -> 99 us).
  if (nb == r.B && r.fseq[mode].size() > 8) {
    launch_captured(p, r.graph[mode], r.graph_src[mode], [&] { enqueue_forward(p, nb, false, mode); });
  } else {
    enqueue_forward(p, nb, false, mode);
  }
  enqueue_reduce(p, nb, false, out);
  check_launch();
}

void check_mode(int mode) {
  require(mode == LTN_C64 || mode == LTN_SPLIT_F16 || mode == LTN_SPLIT_BF16, "unknown mode");
}

}  // namespace

void runtime_describe(const ltn_plan* p, ltn_plan_info* o) {
  if (p->rt) o->batch = p->rt->B;
  o->const_bytes = layout(p, 0, 0).total;
}

void runtime_free(ltn_plan* p) {
  if (!p->rt) return;
  for (int m = 0; m < 3; ++m) {
    if (p->rt->graph[m]) (void)hipGraphExecDestroy(p->rt->graph[m]);
    if (p->rt->graph_src[m]) (void)hipGraphDestroy(p->rt->graph_src[m]);
  }
  for (int m = 0; m < 2; ++m) {
    if (p->rt->ggraph[m]) (void)hipGraphExecDestroy(p->rt->ggraph[m]);
    if (p->rt->ggraph_src[m]) (void)hipGraphDestroy(p->rt->ggraph_src[m]);
  }
  if (p->rt->cap) (void)hipStreamDestroy(p->rt->cap);
  delete p->rt;
  p->rt = nullptr;
}

extern "C" ltn_status ltn_workspace_size(const ltn_plan* p, int32_t batch, int32_t grad,
                                         size_t* bytes) {
  return guarded([&] {
    require(p && bytes, "NULL argument");
    require(batch >= 1, "batch must be >= 1");
    *bytes = layout(p, batch, grad).total;
  });
}

namespace {

// Largest batch whose workspace fits in `bytes`, at most `cap` (0 when not
// even one slice fits).
int fit_batch(const ltn_plan* p, size_t bytes, int grad, int cap) {
  int B = std::min(p->opt.batch > 0 ? p->opt.batch : 4096, 4096);
  if (p->sliced.size() < 12) B = std::min(B, 1 << p->sliced.size());
  B = std::max(1, std::min(B, cap));
  while (B > 1 && layout(p, B, grad).total > bytes) {
    size_t per = grad ? p->garena : p->arena;
    size_t fixed = layout(p, 0, grad).total;
    size_t fit = bytes > fixed ? (bytes - fixed) / (per + 8 + 4 * p->tensors.size() + 512) : 0;
    B = (int)std::max<size_t>(1, std::min<size_t>(fit, (size_t)B - 1));
    if (layout(p, B, grad).total <= bytes) break;
  }
  return layout(p, B, grad).total <= bytes ? B : 0;
}

// Fill a device-side state for the workspace d_ws (batch B): gather
// descriptors, default kernel choices, and the uploads of leaf data and
// descriptors, synchronised on `st` before returning. With `only`, a state for
// one mode whose caller uploads leaf data and descriptors.
void bind_state(ltn_plan* p, ltn_plan_impl* r, char* d_ws, size_t bytes, int grad, hipStream_t st,
                int B, int only = -1) {
  r->st = st;
  r->ws = d_ws;
  r->bytes = bytes;
  r->grad = grad;
  r->B = B;
  r->lay = layout(p, B, grad);
  // descriptors
  int gi = 0;
  for (auto& lp : p->leaves) {
    require(lp.rank_src <= kMaxLeafRank, "leaf rank above 32 is not supported");
    GatherDesc g{};
    g.src_off = lp.src_off;
    g.chunk0 = r->gather_chunks;
    r->gather_chunks += ((int64_t(1) << lp.rank) + kGatherChunk - 1) / kGatherChunk;
    g.rank = lp.rank;
    g.nsl = (int32_t)lp.sl_bit.size();
    for (int j = 0; j < lp.rank; ++j) g.src_bit[j] = (int8_t)lp.src_bit[j];
    for (int j = 0; j < g.nsl; ++j) {
      g.sl_src_bit[j] = (int8_t)lp.sl_src_bit[j];
      g.sl_bit[j] = (int8_t)lp.sl_bit[j];
    }
    const TensorPlan& t = p->tensors[lp.tensor];
    g.tensor = lp.tensor;
    g.dst_off = (int64_t)(t.off * (uint64_t)B / 8);
    r->gd_fwd.push_back(g);
    g.dst_off = (int64_t)(t.goff * (uint64_t)B / 8);
    r->gd_grad.push_back(g);
    g.dst_off = (int64_t)(t.gcot * (uint64_t)B / 8);
    r->gd_gcot.push_back(g);
    r->max_leaf_elems = lp.rank >= 30 ? (1 << 30) : std::max(r->max_leaf_elems, 1 << lp.rank);
    if (lp.param >= 0) r->pl.push_back(ParamLeaf{lp.src_off, lp.param, gi});
    ++gi;
  }
  r->n_pl = (int)r->pl.size();
  for (auto& pr : p->out_sliced) {
    r->sl_bits.push_back(pr.first);
    r->out_bits.push_back(pr.second);
  }
  require(r->sl_bits.size() <= 32, "more than 32 sliced open indices");
  // kernel choice per mode and step (refined by ltn_autotune)
  for (int mode = 0; mode < 3; ++mode)
    for (auto& sp : p->steps) {
      ltn_plan_impl::Choice ch;
      if (only >= 0 && mode != only) {
        r->choice[mode].push_back(ch);
        continue;
      }
      ch.tk = default_tk(sp.k, (1ull << (sp.m + sp.n)) * (uint64_t)B);
      if (sp.kernel == LTN_K_MFMA) {
        // MFMA columns follow the output's lowest bits when possible.
        // Gradient plans keep the FP32 tiles in their forward: a loss with the
        // logarithm of small amplitudes magnifies any change of rounding
        // there (3e-5 in the 20-qubit gradient, more than this path's own
        // error on most inputs); their adjoint products do take the parts.
        bool nat = (sp.c_mask_a & 1) != 0;
        if (mode != LTN_C64 || !grad)
          for (bool sw : {nat, !nat}) {
            const int c = ch.kind ? -1 : parts_config_default(sw ? sp.n : sp.m, sp.k, sw ? sp.m : sp.n, B, mode);
            if (c >= 0) {
              ch.kind = 6;
              ch.cfg = c;
              ch.swap = sw;
            }
          }
        for (int kind : {mode == LTN_C64 ? 1 : 2, 1}) {
          for (bool sw : {nat, !nat}) {
            const int m = sw ? sp.n : sp.m, n = sw ? sp.m : sp.n;
            const int c = kind == 2 ? default_split_cfg(m, sp.k, n, B, mode) : default_cfg(m, sp.k, n);
            if (c >= 0 && ch.kind == 0) {
              ch.kind = kind;
              ch.cfg = c;
              ch.swap = sw;
            }
          }
        }
      }
      // no full tile but a long sum: the split-K tile (the small side as columns)
      if (ch.kind == 0) {
        const bool sw = sp.n > sp.m;
        for (int c = 0; c < splitk_config_count() && ch.kind == 0; ++c)
          if (sw ? splitk_config_fits(c, sp.n, sp.k, sp.m) : splitk_config_fits(c, sp.m, sp.k, sp.n)) {
            ch.kind = 5;
            ch.cfg = c;
            ch.swap = sw;
          }
      }
      // few outputs and a long sum: split the sum over blocks
      if (ch.kind == 0 && skinny_fits(sp.m, sp.k, sp.n) && sp.k >= 10) {
        ch.kind = 4;
        ch.cfg = 0;
      }
      // short sums of 2 and 4 with many outputs: the direct tiles 64 x 32 x 2
      // and x 4 (64 slices of (7,2,7): 0.009 ms against 0.019 on the generic
      // kernel, (8,1,6): 0.009 against 0.011 on the narrow one, (13,1,10): 0.029
      // against 0.151; at 2^17 outputs, (6,2,6) x 32, no gain). Not from 2^21 outputs
      // on where the narrow kernel fits, the rows hold the output's lowest bit and no
      // maxima are recorded: (16,1,6) 16.6 us narrow and 18.4 here, (11,1,6) x 256 76 and
      // 89, (17,2,6) x 4 85 and 98; lowest bit from the columns, (12,2,5) x 256, 111 and 93.
      const bool nat = (sp.c_mask_a & 1) != 0, tall = sp.m >= sp.n;
      const int64_t outs = sp.m + sp.n < 40 ? (int64_t(1) << (sp.m + sp.n)) * B : 0;
      const bool narrow = mode != LTN_SPLIT_F16 && nat == tall && outs >> 21 > 0 &&
                          narrow_fits(tall ? sp.m : sp.n, sp.k, tall ? sp.n : sp.m);
      if (ch.kind == 0 && (mode != LTN_C64 || !grad) && (sp.k == 1 || sp.k == 2) && outs >> 18 > 0 && !narrow) {
        const int c = sp.k == 1 ? 7 : 6;
        for (bool sw : {nat, !nat})
          if (ch.kind == 0 && gemm_config_fits(c, sw ? sp.n : sp.m, sp.k, sw ? sp.m : sp.n, LTN_C64)) {
            ch.kind = 1;
            ch.cfg = c;
            ch.swap = sw;
          }
      }
      // steps with many output rows and no MFMA tile: the narrow kernel
      if (ch.kind == 0 && sp.m + sp.n >= 12) {
        const bool sw = sp.n > sp.m;
        const int c = sw ? narrow_config_default(sp.n, sp.k, sp.m, ~sp.c_mask_a)
                         : narrow_config_default(sp.m, sp.k, sp.n, sp.c_mask_a);
        if (c >= 0) {
          ch.kind = 3;
          ch.cfg = c;
          ch.swap = sw;
        }
      }
      r->choice[mode].push_back(ch);
    }
  r->needs_grad.assign(p->tensors.size(), 0);
  for (size_t v = 0; v < p->tensors.size(); ++v) {
    if ((int)v < p->L)
      r->needs_grad[v] = p->leaves[v].param >= 0;
    else {
      const StepPlan& sp = p->steps[v - p->L];
      r->needs_grad[v] = r->needs_grad[sp.left] || r->needs_grad[sp.right];
    }
  }
  if (only >= 0) return;
  // uploads (host vectors live in the plan / impl; synchronised below)
  HIPCHECK(hipMemcpyAsync(r->ws + r->lay.leafdata, p->leaf_data.data(), (size_t)p->leaf_elems * 8,
                          hipMemcpyHostToDevice, r->st));
  HIPCHECK(hipMemcpyAsync(r->ws + r->lay.gd_fwd, r->gd_fwd.data(), r->gd_fwd.size() * sizeof(GatherDesc),
                          hipMemcpyHostToDevice, r->st));
  if (grad) {
    HIPCHECK(hipMemcpyAsync(r->ws + r->lay.gd_grad, r->gd_grad.data(),
                            r->gd_grad.size() * sizeof(GatherDesc), hipMemcpyHostToDevice, r->st));
    HIPCHECK(hipMemcpyAsync(r->ws + r->lay.gd_gcot, r->gd_gcot.data(),
                            r->gd_gcot.size() * sizeof(GatherDesc), hipMemcpyHostToDevice, r->st));
  }
  if (r->n_pl)
    HIPCHECK(hipMemcpyAsync(r->ws + r->lay.pl, r->pl.data(), r->pl.size() * sizeof(ParamLeaf),
                            hipMemcpyHostToDevice, r->st));
  HIPCHECK(hipStreamSynchronize(r->st));
}

}  // namespace

extern "C" ltn_status ltn_bind(ltn_plan* p, void* d_ws, size_t bytes, int32_t grad, void* stream) {
  return guarded([&] {
    require(p != nullptr, "plan is NULL");
    require(d_ws != nullptr, "workspace is NULL");
    require(((uintptr_t)d_ws & 255) == 0, "workspace must be 256-byte aligned");
    // grid.y limit of the gather; no batch larger than the slice count
    const int B = fit_batch(p, bytes, grad, 4096);
    if (B == 0)
      fail(LTN_E_NOMEM, "workspace of " + std::to_string(bytes) + " bytes is below the " +
                            std::to_string(layout(p, 1, grad).total) + " needed for one slice");
    runtime_free(p);
    auto r = new ltn_plan_impl();
    p->rt = r;
    bind_state(p, r, reinterpret_cast<char*>(d_ws), bytes, grad, reinterpret_cast<hipStream_t>(stream), B);
  });
}

static void build_grad_seq(ltn_plan* p);

static ltn_status execute_impl(ltn_plan* p, const uint64_t* ids, uint64_t begin, uint64_t n,
                               bool range, int32_t mode, void* d_out) {
  return guarded([&] {
    auto& r = rt(p);
    check_mode(mode);
    require(d_out != nullptr, "d_out is NULL");
    const int ns = (int)p->sliced.size();
    if (range) {
      require(begin <= n, "range end before begin");
      require(ns >= 64 || n <= (1ull << ns), "slice range beyond 2^|S|");
      n = n - begin;
    } else {
      require(n == 0 || ids != nullptr, "slice_ids is NULL");
      if (ns < 64)
        for (uint64_t i = 0; i < n; ++i)
          require(ids[i] < (1ull << ns), "slice id " + std::to_string(ids[i]) + " is not below 2^|S|");
    }
    r.fwd_kept = false;
    if (r.grad && mode == LTN_C64 && n >= 1 && n <= (uint64_t)r.B) {
      // a plan bound for gradients runs a one-batch forward in its gradient
      // arena, whose tensors then stay for ltn_execute_grad on the same ids
      const int nb = (int)n;
      if (!r.gseq_valid) build_grad_seq(p);
      set_ids(p, range ? nullptr : ids, begin, nb, range);
      if (nb == r.B)
        launch_captured(p, r.ggraph[0], r.ggraph_src[0], [&] { enqueue_forward(p, nb, true, LTN_C64); });
      else
        enqueue_forward(p, nb, true, LTN_C64);
      enqueue_reduce(p, nb, true, reinterpret_cast<double*>(d_out));
      check_launch();
      r.fwd_ids.resize(n);
      for (uint64_t i = 0; i < n; ++i) r.fwd_ids[i] = range ? begin + i : ids[i];
      r.fwd_kept = true;
      return;
    }
    for (uint64_t off = 0; off < n; off += (uint64_t)r.B) {
      int nb = (int)std::min<uint64_t>((uint64_t)r.B, n - off);
      set_ids(p, range ? nullptr : ids + off, begin + off, nb, range);
      run_batch(p, nb, mode, reinterpret_cast<double*>(d_out));
    }
  });
}

extern "C" ltn_status ltn_execute(ltn_plan* p, const uint64_t* ids, uint64_t n, int32_t mode,
                                  void* d_out) {
  return execute_impl(p, ids, 0, n, false, mode, d_out);
}

extern "C" ltn_status ltn_execute_range(ltn_plan* p, uint64_t begin, uint64_t end, int32_t mode,
                                        void* d_out) {
  return execute_impl(p, nullptr, begin, end, true, mode, d_out);
}

// Device memory of the library's own, for callers that cannot allocate:
// one fixed array per GPU, held until the process ends. Host code never
// uses the array's name as an address (on the host it is only a handle);
// it uses the device address hipGetSymbolAddress returns for the current
// device, fetched once per device.
static __device__ __align__(256) char scratch[LTN_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
char* g_scratch_ptr[kMaxDevices] = {};

char* scratch_ptr() {
  int dev = 0;
  HIPCHECK(hipGetDevice(&dev));
  require(dev >= 0 && dev < kMaxDevices, "device ordinal above 63");
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    HIPCHECK(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
    require(ptr != nullptr, "no device address for the scratch array");
    g_scratch_ptr[dev] = reinterpret_cast<char*>(ptr);
  }
  return g_scratch_ptr[dev];
}

}  // namespace

extern "C" ltn_status ltn_execute_scratch(ltn_plan* p, const uint64_t* ids, uint64_t n, int32_t mode,
                                          void* d_out, void* stream) {
  return guarded([&] {
    require(p != nullptr, "plan is NULL");
    check_mode(mode);
    require(d_out != nullptr, "d_out is NULL");
    require(n == 0 || ids != nullptr, "slice_ids is NULL");
    const int ns = (int)p->sliced.size();
    if (ns < 64)
      for (uint64_t i = 0; i < n; ++i)
        require(ids[i] < (1ull << ns), "slice id " + std::to_string(ids[i]) + " is not below 2^|S|");
    if (n == 0) return;
    const int B = fit_batch(p, LTN_SCRATCH_BYTES, 0, (int)std::min<uint64_t>(n, 4096));
    if (B == 0)
      fail(LTN_E_NOMEM, "one slice needs " + std::to_string(layout(p, 1, 0).total) +
                            " bytes of workspace; the library's scratch holds " +
                            std::to_string((size_t)LTN_SCRATCH_BYTES));
    char* ws = scratch_ptr();
    // a state of this call only: the plan's own binding (if any) is kept
    ltn_plan_impl tmp;
    ltn_plan_impl* bound = p->rt;
    p->rt = &tmp;
    try {
      bind_state(p, &tmp, ws, LTN_SCRATCH_BYTES, 0, reinterpret_cast<hipStream_t>(stream), B, mode);
      build_fwd_seq(p, mode, false);
      // leaf data and descriptors, which lie in a row, in one copy (three with
      // two waits took 20 of a 12-qubit amplitude's 64 us); leaf data above 1 MiB
      // from where they are, as gathering them on the host costs more (512 KiB: 72
      // against 84 us a call, 2 MiB: 180 against 134, 8 MiB: 530 against 306)
      const auto& descs = tmp.fseq_descs[mode];
      const size_t fdesc = tmp.lay.fdesc + (size_t)mode * p->steps.size() * sizeof(GenericDesc);
      const size_t leaf_bytes = (size_t)p->leaf_elems * 8, from = leaf_bytes > (1 << 20) ? tmp.lay.gd_fwd : 0;
      std::vector<char> host(fdesc - from + descs.size() * sizeof(GenericDesc));
      if (from)
        HIPCHECK(hipMemcpyAsync(ws + tmp.lay.leafdata, p->leaf_data.data(), leaf_bytes, hipMemcpyHostToDevice, tmp.st));
      else
        std::memcpy(host.data() + tmp.lay.leafdata, p->leaf_data.data(), leaf_bytes);
      std::memcpy(host.data() + (tmp.lay.gd_fwd - from), tmp.gd_fwd.data(), tmp.gd_fwd.size() * sizeof(GatherDesc));
      std::memcpy(host.data() + (fdesc - from), descs.data(), descs.size() * sizeof(GenericDesc));
      HIPCHECK(hipMemcpyAsync(ws + from, host.data(), host.size(), hipMemcpyHostToDevice, tmp.st));
      HIPCHECK(hipStreamSynchronize(tmp.st));
      for (uint64_t off = 0; off < n; off += (uint64_t)B) {
        const int nb = (int)std::min<uint64_t>((uint64_t)B, n - off);
        set_ids(p, ids + off, 0, nb, false);
        enqueue_forward(p, nb, false, mode);
        enqueue_reduce(p, nb, false, reinterpret_cast<double*>(d_out));
        check_launch();
      }
    } catch (...) {
      p->rt = bound;
      throw;
    }
    p->rt = bound;
  });
}

extern "C" ltn_status ltn_set_params(ltn_plan* p, const double* d_angles) {
  return guarded([&] {
    auto& r = rt(p);
    require(r.n_pl == 0 || d_angles != nullptr, "d_angles is NULL");
    if (r.n_pl == 0) return;
    r.fwd_kept = false;
    double* ang = reinterpret_cast<double*>(r.ws + r.lay.angles);
    HIPCHECK(hipMemcpyAsync(ang, d_angles, (size_t)p->n_params * sizeof(double),
                            hipMemcpyDeviceToDevice, r.st));
    launch_u3_build(reinterpret_cast<const ParamLeaf*>(r.ws + r.lay.pl), r.n_pl, ang,
                    reinterpret_cast<float2*>(r.ws + r.lay.leafdata), r.st);
    check_launch();
  });
}

// One adjoint product in the forward form: C[merge(m, n)] = sum_k
// X[m 2^k + k] Y[n 2^k + k] over a batch of nb slices, on the complex64
// MFMA GEMM when a tile fits (either operand role), else the narrow kernel,
// else the generic kernel. Kinds: 1 a full FP32 tile, 5 a split-K tile (partials
// in the workspace's split-K buffer, which the layout sizes for the adjoint
// products of gradient plans), 6 a three-part tile.
uint32_t adj_key(int m, int k, int n) { return (uint32_t)m | (uint32_t)k << 8 | (uint32_t)n << 16; }

static void nt_gemm(ltn_plan* p, const float2* X, int64_t sX, const float2* Y, int64_t sY, float2* C,
                    int64_t sC, int m, int k, int n, uint64_t cmask, int nb, int kind, int sw, int cfg) {
  auto& r = *p->rt;
  const uint64_t full = (m + n) >= 64 ? ~0ull : ((1ull << (m + n)) - 1);
  GemmDesc d{};
  d.A = sw ? Y : X;
  d.B = sw ? X : Y;
  d.C = C;
  d.sA = sw ? sY : sX;
  d.sB = sw ? sX : sY;
  d.sC = sC;
  d.m = sw ? n : m;
  d.n = sw ? m : n;
  d.k = k;
  d.cmask = sw ? (~cmask & full) : cmask;
  d.nb = nb;
  d.cfg = cfg;
  d.part = reinterpret_cast<float2*>(r.ws + r.lay.splitk);
  if (kind == 1)
    launch_cgemm(d, LTN_C64, r.st);
  else if (kind == 5)
    launch_cgemm_splitk(d, r.st);
  else
    launch_cgemm_parts(d, r.st);
}

static void enqueue_nt(ltn_plan* p, const float2* X, int64_t sX, const float2* Y, int64_t sY,
                       float2* C, int64_t sC, int m, int k, int n, uint64_t cmask, int nb) {
  auto& r = *p->rt;
  const uint64_t full = (m + n) >= 64 ? ~0ull : ((1ull << (m + n)) - 1);
  const auto tuned = r.adj.find(adj_key(m, k, n));
  if (tuned != r.adj.end() && tuned->second.kind > 0) {
    const auto& t = tuned->second;
    nt_gemm(p, X, sX, Y, sY, C, sC, m, k, n, cmask, nb, t.kind, t.swap, t.cfg);
    return;
  }
  for (int sw = 0; sw < 2; ++sw) {
    const int cfg = parts_config_default(sw ? n : m, k, sw ? m : n, nb, LTN_C64);
    if (cfg >= 0) {
      nt_gemm(p, X, sX, Y, sY, C, sC, m, k, n, cmask, nb, 6, sw, cfg);
      return;
    }
  }
  for (int sw = 0; sw < 2; ++sw) {
    const int mm = sw ? n : m, nn = sw ? m : n;
    const int cfg = default_cfg(mm, k, nn);
    if (cfg >= 0 && mm >= 5 && nn >= 5) {
      nt_gemm(p, X, sX, Y, sY, C, sC, m, k, n, cmask, nb, 1, sw, cfg);
      return;
    }
  }
  if (m + n >= 12) {
    const bool sw = n > m;
    const int cfg = narrow_config_default(sw ? n : m, k, sw ? m : n, sw ? ~cmask : cmask);
    if (cfg >= 0) {
      NarrowDesc d{};
      d.A = sw ? Y : X;
      d.B = sw ? X : Y;
      d.C = C;
      d.sA = sw ? sY : sX;
      d.sB = sw ? sX : sY;
      d.sC = sC;
      d.m = sw ? n : m;
      d.n = sw ? m : n;
      d.k = k;
      d.cmask = sw ? (~cmask & full) : cmask;
      d.nb = nb;
      d.cfg = cfg;
      launch_narrow(d, r.st);
      return;
    }
  }
  GenericDesc g{};
  g.P = X;
  g.Q = Y;
  g.out = C;
  g.sP = sX;
  g.sQ = sY;
  g.sO = sC;
  g.set_shape(m, n, k, false);
  g.px = ((1ull << m) - 1) << k;
  g.pz = (1ull << k) - 1;
  g.qy = ((1ull << n) - 1) << k;
  g.qz = (1ull << k) - 1;
  g.ox = cmask;
  g.oy = ~cmask & full;
  g.nb = nb;
  launch_generic(g, default_tk(k, (1ull << (m + n)) * (uint64_t)nb), r.st);
}

// Whether a parts tile reads the operands of an adjoint product where they lie: the
// product itself then takes 12-30 % longer, so it pays where there is enough to
// permute. The cotangent has 2^-cols of the product's multiply-adds in elements (none
// to move if its rows are the upper bits already), the other operand 2^-rows; in
// place from 2^-8 on. 256 slices, permuted against in place, us: (rows 10, cols 10,
// sum 7) 1558 and 1728, (11,9,6) 522 and 550, (9,7,7) in order 119 and 129, (10,6,10)
// in order 820 and 1077; (8,7,8) in order 113 and 106, (11,7,5) 238 and 218, (9,7,7)
// 162 and 125, (10,6,10) 1604 and 1020.
static bool in_place_pays(int rows, int cols, bool in_order) {
  return rows <= 8 || (!in_order && (cols <= 8 || (rows == 9 && cols == 9)));
}

// The adjoint product of step s for one operand (which 0: A, 1: B) on a parts
// tile that reads the output's cotangent and the other operand where they lie;
// false where the product takes another kernel.
static bool adj_parts_in_place(ltn_plan* p, int s, int which, int nb) {
  auto& r = *p->rt;
  const StepPlan& sp = p->steps[s];
  const TensorPlan &ta = p->tensors[sp.a], &tb = p->tensors[sp.b], &tc = p->tensors[sp.out];
  const TensorPlan &self = which ? tb : ta, &other = which ? ta : tb;
  const int m = which ? sp.n : sp.m, k = which ? sp.m : sp.n, n = sp.k;
  bool sw = false;
  int cfg = -1;
  const auto tuned = r.adj.find(adj_key(m, k, n));
  if (tuned != r.adj.end() && tuned->second.kind > 0) {
    if (tuned->second.kind != 6) return false;
    sw = tuned->second.swap;
    cfg = tuned->second.cfg;
  } else {
    cfg = parts_config_default(m, k, n, nb, LTN_C64, true);
    if (cfg < 0) {
      sw = true;
      cfg = parts_config_default(n, k, m, nb, LTN_C64, true);
    }
  }
  const uint64_t cfull = (1ull << (sp.m + sp.n)) - 1, ofull = (1ull << (m + n)) - 1;
  const uint64_t xrow = which ? ~sp.c_mask_a & cfull : sp.c_mask_a, yrow = (1ull << n) - 1;
  if (cfg < 0 || !parts_config_in_place(cfg) || !in_place_pays(m, n, (cfull & ~xrow) == (1ull << k) - 1)) return false;
  const uint64_t ysum = ((1ull << k) - 1) << n, cmask = ((1ull << m) - 1) << n;
  const float2 *X = arena_ptr(p, tc.gcot), *Y = arena_ptr(p, other.goff);
  GemmDesc d{};
  d.A = sw ? Y : X;
  d.B = sw ? X : Y;
  d.C = arena_ptr(p, self.gcot);
  d.sA = int64_t(1) << (sw ? other.rank : tc.rank);
  d.sB = int64_t(1) << (sw ? tc.rank : other.rank);
  d.sC = int64_t(1) << self.rank;
  d.m = sw ? n : m;
  d.n = sw ? m : n;
  d.k = k;
  d.cmask = sw ? ~cmask & ofull : cmask;
  d.nb = nb;
  d.cfg = cfg;
  d.arow = sw ? yrow : xrow;
  d.asum = sw ? ysum : ~xrow & cfull;
  d.brow = sw ? xrow : yrow;
  d.bsum = sw ? ~xrow & cfull : ysum;
  d.conj_a = sw;
  d.conj_b = !sw;
  launch_cgemm_parts(d, r.st);
  return true;
}

static PermuteDesc plan_permute(int32_t rank, const int32_t* perm, int64_t batch, bool conj);

// Bit permutation of a batch of nb tensors (slice stride 2^rank), optionally
// conjugated, into `out`; returns the tensor to read (the input itself for
// the identity without conjugation).
static const float2* enqueue_perm(ltn_plan* p, const float2* in, float2* out,
                                  const std::vector<int32_t>& perm, int nb, bool conj) {
  bool ident = !conj;
  for (size_t j = 0; j < perm.size() && ident; ++j) ident = perm[j] == (int32_t)j;
  if (ident) return in;
  PermuteDesc d = plan_permute((int32_t)perm.size(), perm.data(), nb, conj);
  launch_permute(in, out, d, p->rt->st);
  return out;
}

// Adjoint of a small step for one operand (which 0: A, 1: B) on the
// generic kernel: the output cotangent times the other operand, conjugated,
// summed over the other operand's free bits; operands read in place.
static GenericDesc adj_generic_desc(ltn_plan* p, int s, int which, int nb, int* tk) {
  const StepPlan& sp = p->steps[s];
  const TensorPlan &ta = p->tensors[sp.a], &tb = p->tensors[sp.b], &tc = p->tensors[sp.out];
  const uint64_t cm = sp.c_mask_a, full = (1ull << (sp.m + sp.n)) - 1;
  GenericDesc g{};
  g.P = arena_ptr(p, tc.gcot);
  g.sP = int64_t(1) << tc.rank;
  g.qy = (1ull << sp.k) - 1;
  g.oy = (1ull << sp.k) - 1;
  g.nb = nb;
  if (which == 0) {
    g.Q = arena_ptr(p, tb.goff);
    g.out = arena_ptr(p, ta.gcot);
    g.sQ = int64_t(1) << tb.rank;
    g.sO = int64_t(1) << ta.rank;
    g.set_shape(sp.m, sp.k, sp.n, true);
    g.px = cm;
    g.pz = ~cm & full;
    g.qz = ((1ull << sp.n) - 1) << sp.k;
    g.ox = ((1ull << sp.m) - 1) << sp.k;
    *tk = default_tk(sp.n, (1ull << (sp.m + sp.k)) * (uint64_t)nb);
  } else {
    g.Q = arena_ptr(p, ta.goff);
    g.out = arena_ptr(p, tb.gcot);
    g.sQ = int64_t(1) << ta.rank;
    g.sO = int64_t(1) << tb.rank;
    g.set_shape(sp.n, sp.k, sp.m, true);
    g.px = ~cm & full;
    g.pz = cm;
    g.qz = ((1ull << sp.m) - 1) << sp.k;
    g.ox = ((1ull << sp.n) - 1) << sp.k;
    *tk = default_tk(sp.m, (1ull << (sp.n + sp.k)) * (uint64_t)nb);
  }
  return g;
}

// The adjoint product of step s for one operand (which 0: A, 1: B), on the kernel
// that the sweep takes for it.
static void enqueue_adjoint_product(ltn_plan* p, int s, int which, int nb) {
  auto& r = *p->rt;
  const StepPlan& sp = p->steps[s];
  const TensorPlan &ta = p->tensors[sp.a], &tb = p->tensors[sp.b], &tc = p->tensors[sp.out];
  const TensorPlan &self = which ? tb : ta, &other = which ? ta : tb;
  // small steps and products with few columns: one kernel, reading the operands
  // in place (strided) and conjugating the second one
  int tk = 1;
  const GenericDesc g = adj_generic_desc(p, s, which, nb, &tk);
  RowsumDesc d;
  if (rowsum_fits(g, d)) {
    launch_rowsum(d, r.st);
    return;
  }
  if (sp.m + sp.n + sp.k <= 16) {
    launch_generic(g, tk, r.st);
    return;
  }
  if (adj_parts_in_place(p, s, which, nb)) return;
  // forward form: the output cotangent and the other operand are permuted so that
  // the summed bits are lowest (and the operand conjugated), then one GEMM:
  // dA[m][k] = sum_n dC[merge(m, n)] conj(B[n][k]), dB[n][k] = sum_m dC[merge(m, n)]
  // conj(A[m][k])
  const int rows = which ? sp.n : sp.m, sum = which ? sp.m : sp.n, rc = sp.m + sp.n;
  std::vector<int32_t> pc(rc), po(sp.k + sum);
  int row = 0, at = 0;
  for (int j = 0; j < rc; ++j) pc[j] = (int)((sp.c_mask_a >> j) & 1) != which ? sum + row++ : at++;
  for (int j = 0; j < sp.k; ++j) po[j] = sum + j;
  for (int i = 0; i < sum; ++i) po[sp.k + i] = i;
  float2* Xs = reinterpret_cast<float2*>(r.ws + r.lay.gscr_c);
  float2* Ys = reinterpret_cast<float2*>(r.ws + r.lay.gscr);
  const float2* X = enqueue_perm(p, arena_ptr(p, tc.gcot), Xs, pc, nb, false);
  enqueue_perm(p, arena_ptr(p, other.goff), Ys, po, nb, true);
  enqueue_nt(p, X, int64_t(1) << rc, Ys, int64_t(1) << other.rank, arena_ptr(p, self.gcot), int64_t(1) << self.rank,
             rows, sum, sp.k, ((1ull << rows) - 1) << sp.k, nb);
}

// Adjoint of step s (operand cotangents from the output's cotangent).
static void enqueue_adjoint_step(ltn_plan* p, int s, int nb) {
  const auto& need = p->rt->needs_grad;
  const StepPlan& sp = p->steps[s];
  if (!need[sp.out]) return;
  for (int which = 0; which < 2; ++which)
    if (need[which ? sp.b : sp.a]) enqueue_adjoint_product(p, s, which, nb);
}

// Adjoint sweep of one batch (steps in reverse order), then the leaf
// cotangents accumulated into the per-leaf FP64 sums. Every pointer is in
// the bound workspace, so a full batch can run from a captured graph.
static void enqueue_backward(ltn_plan* p, int nb) {
  auto& r = *p->rt;
  double* lg = reinterpret_cast<double*>(r.ws + r.lay.leafgrad);
  const GatherDesc* gcot = reinterpret_cast<const GatherDesc*>(r.ws + r.lay.gd_gcot);
  const uint64_t* dids = reinterpret_cast<const uint64_t*>(r.ws + r.lay.ids);
  if (r.gseq_valid) {
    const GenericDesc* dd = reinterpret_cast<const GenericDesc*>(r.ws + r.lay.gdesc);
    for (const auto& it : r.gseq_bwd) {
      if (it.what == 2)
        enqueue_adjoint_step(p, it.step, nb);
      else
        enqueue_generic(p, dd, it, nb);
    }
  } else {
    for (int s = (int)p->steps.size() - 1; s >= 0; --s) enqueue_adjoint_step(p, s, nb);
  }
  launch_leaf_cot_accumulate(reinterpret_cast<const ParamLeaf*>(r.ws + r.lay.pl), r.n_pl, gcot,
                             arena_ptr(p, 0), dids, nb, lg, r.st);
}

// Gradient launch sequences: the recomputed forward (outputs of small steps
// are kept in memory, where the adjoint sweep reads them) and the adjoint sweep
// in reverse order. The gradient arena gives every tensor and every cotangent
// a place of its own, so memory is never reused. The descriptors (for the
// bound batch size; the launch passes the actual one) are copied to the
// workspace here, outside any capture.
static void build_grad_seq(ltn_plan* p) {
  auto& r = *p->rt;
  using Item = ltn_plan_impl::GradItem;
  r.gseq_descs.clear();
  r.gseq_fwd.clear();
  r.gseq_bwd.clear();
  std::vector<SeqOp> ops;
  auto single = [&](std::vector<Item>& seq, int what, int s) {
    sequence_generic(ops, r.B, false, r.gseq_descs, seq);
    ops.clear();
    Item it;
    it.what = what;
    it.step = s;
    seq.push_back(it);
  };
  for (int s = 0; s < (int)p->steps.size(); ++s) {
    if (r.choice[LTN_C64][s].kind != 0)
      single(r.gseq_fwd, 0, s);
    else
      ops.push_back(step_seq_op(p, s, true, LTN_C64));
  }
  sequence_generic(ops, r.B, false, r.gseq_descs, r.gseq_fwd);
  ops.clear();
  const int nt = (int)p->tensors.size();
  auto range = [&](int t, bool cot) {
    const TensorPlan& T = p->tensors[t];
    const uint64_t off = cot ? T.gcot : T.goff;
    return SeqOp::Range{off, off + T.bytes()};
  };
  for (int s = (int)p->steps.size() - 1; s >= 0; --s) {
    const StepPlan& sp = p->steps[s];
    if (!r.needs_grad[sp.out]) continue;
    bool alone = sp.m + sp.n + sp.k > 16;
    if (!alone && sp.m + sp.n + sp.k >= kRowsumWork) {
      alone = true;
      for (int which = 0; which < 2; ++which) {
        int tk;
        RowsumDesc d;
        if (r.needs_grad[which ? sp.b : sp.a]) alone = alone && rowsum_fits(adj_generic_desc(p, s, which, r.B, &tk), d);
      }
    }
    if (alone) {
      single(r.gseq_bwd, 2, s);
      continue;
    }
    for (int which = 0; which < 2; ++which) {
      const int t = which ? sp.b : sp.a, other = which ? sp.a : sp.b;
      if (!r.needs_grad[t]) continue;
      SeqOp o;
      o.g = adj_generic_desc(p, s, which, r.B, &o.tk);
      o.step = s;
      o.consumer = p->tensors[t].producer;
      o.in[0] = nt + sp.out;
      o.rin[0] = range(sp.out, true);
      o.in[1] = other;
      o.rin[1] = range(other, false);
      o.out = nt + t;
      o.rout = range(t, true);
      ops.push_back(o);
    }
  }
  sequence_generic(ops, r.B, false, r.gseq_descs, r.gseq_bwd);
  require(r.gseq_descs.size() <= 3 * p->steps.size(), "gradient descriptor area too small");
  if (!r.gseq_descs.empty())
    HIPCHECK(hipMemcpyAsync(r.ws + r.lay.gdesc, r.gseq_descs.data(), r.gseq_descs.size() * sizeof(GenericDesc),
                            hipMemcpyHostToDevice, r.st));
  // the host array may be rebuilt by a later call: let the copy finish
  HIPCHECK(hipStreamSynchronize(r.st));
  r.gseq_valid = true;
}

extern "C" ltn_status ltn_execute_grad(ltn_plan* p, const uint64_t* ids, uint64_t n, int32_t mode,
                                       const void* d_cot, void* d_out, double* d_angle_grad) {
  return guarded([&] {
    auto& r = rt(p);
    check_mode(mode);
    if (mode != LTN_C64) fail(LTN_E_UNSUPPORTED, "gradients run in complex64 only");
    require(r.grad, "plan was bound without gradient workspace");
    require(d_cot && d_angle_grad, "NULL argument");
    require(n == 0 || ids, "slice_ids is NULL");
    const int ns = (int)p->sliced.size();
    if (ns < 64)
      for (uint64_t i = 0; i < n; ++i) require(ids[i] < (1ull << ns), "slice id is not below 2^|S|");
    double* lg = reinterpret_cast<double*>(r.ws + r.lay.leafgrad);
    if (!r.gseq_valid) build_grad_seq(p);
    // the forward of these very slices (same parameters) is still in the
    // gradient arena after a one-batch ltn_execute: it is not recomputed
    const bool kept = r.fwd_kept && n == r.fwd_ids.size() && std::equal(ids, ids + n, r.fwd_ids.begin());
    r.fwd_kept = false;
    launch_fill_zero(lg, al((size_t)r.n_pl * 64), r.st);
    const uint64_t* dids = reinterpret_cast<const uint64_t*>(r.ws + r.lay.ids);
    // full batches run the recomputed forward and the adjoint sweep from two
    // captured graphs; the cotangent and output pointers stay outside them
    for (uint64_t off = 0; off < n; off += (uint64_t)r.B) {
      int nb = (int)std::min<uint64_t>((uint64_t)r.B, n - off);
      if (!kept) {
        set_ids(p, ids + off, 0, nb, false);
        if (nb == r.B)
          launch_captured(p, r.ggraph[0], r.ggraph_src[0], [&] { enqueue_forward(p, nb, true, LTN_C64); });
        else
          enqueue_forward(p, nb, true, LTN_C64);
      }
      if (d_out) enqueue_reduce(p, nb, true, reinterpret_cast<double*>(d_out));
      const TensorPlan& root = p->tensors[p->root];
      launch_root_cotangent(reinterpret_cast<const double*>(d_cot), root.rank, p->out_mask,
                            r.sl_bits.data(), r.out_bits.data(), (int)r.sl_bits.size(), dids, nb,
                            arena_ptr(p, root.gcot), r.st);
      if (nb == r.B)
        launch_captured(p, r.ggraph[1], r.ggraph_src[1], [&] { enqueue_backward(p, nb); });
      else
        enqueue_backward(p, nb);
      check_launch();
    }
    launch_u3_adjoint(reinterpret_cast<const ParamLeaf*>(r.ws + r.lay.pl), r.n_pl,
                      reinterpret_cast<const double*>(r.ws + r.lay.angles), lg, d_angle_grad, r.st);
    check_launch();
  });
}

namespace {

// What a tuning was chosen from: a file keeps the entries of other sets, but a
// plan does not take its kernels from them.
constexpr char kCandidates[] = "_c2";

// The complex64 forward of a plan bound for gradients has candidates of its own
// (see bind_state), hence entries of its own.
std::string tune_key(int mode, const StepPlan& sp, int B, bool fp32_forward) {
  std::ostringstream o;
  o << "m" << mode << (fp32_forward ? "g" : "") << "_" << sp.m << "_" << sp.k << "_" << sp.n << "_"
    << (sp.c_mask_a & 1) << "_b" << B << kCandidates;
  return o.str();
}

// Why a kernel choice cannot run a step in a mode (null: it can).
const char* misfit(const ltn_plan_impl::Choice& c, const StepPlan& sp, int mode) {
  const int m = c.swap ? sp.n : sp.m, n = c.swap ? sp.m : sp.n;
  const int km = c.kind == 2 ? mode : LTN_C64;
  switch (c.kind) {
    case 0: return c.tk == 1 || c.tk == 8 || c.tk == 64 ? nullptr : "tk must be 1, 8 or 64";
    case 1:
    case 2:
      if (c.kind == 2 && mode == LTN_C64) return "split GEMM kernels need a split mode";
      return c.cfg >= 0 && c.cfg < gemm_config_count(km) && gemm_config_fits(c.cfg, m, sp.k, n, km)
                 ? nullptr
                 : "tile configuration does not fit the step";
    case 3:
      if (c.cfg != 0 && c.cfg != 1) return "narrow kernel configuration must be 0 or 1";
      return (c.cfg == 0 ? narrow_fits(m, sp.k, n) : narrow_rows_fits(m, sp.k, n))
                 ? nullptr
                 : "the narrow kernel does not fit the step";
    case 4: return skinny_fits(sp.m, sp.k, sp.n) ? nullptr : "the split-sum kernel needs m <= 3 and n <= 3";
    case 5:
      return splitk_config_fits(c.cfg, m, sp.k, n) ? nullptr : "split-K tile configuration does not fit the step";
    case 6: return parts_config_fits(c.cfg, m, sp.k, n, mode) ? nullptr : "tile configuration does not fit the step";
  }
  return "unknown kernel kind";
}

std::map<std::string, std::pair<int, int>> read_cache(const char* path) {
  std::map<std::string, std::pair<int, int>> c;
  if (!path) return c;
  std::ifstream f(path);
  if (!f) return c;
  std::stringstream ss;
  ss << f.rdbuf();
  std::string s = ss.str();
  // entries look like "key": [a, b]
  size_t pos = 0;
  while ((pos = s.find('"', pos)) != std::string::npos) {
    size_t e = s.find('"', pos + 1);
    if (e == std::string::npos) break;
    std::string key = s.substr(pos + 1, e - pos - 1);
    size_t lb = s.find('[', e), rb = s.find(']', e);
    if (lb == std::string::npos || rb == std::string::npos) break;
    int a = 0, b = 0;
    if (sscanf(s.c_str() + lb + 1, "%d , %d", &a, &b) == 2) c[key] = {a, b};
    pos = rb + 1;
  }
  return c;
}

void write_cache(const char* path, const std::map<std::string, std::pair<int, int>>& c) {
  if (!path) return;
  std::ofstream f(path);
  f << "{\n";
  size_t i = 0;
  for (auto& kv : c)
    f << "  \"" << kv.first << "\": [" << kv.second.first << ", " << kv.second.second << "]"
      << (++i < c.size() ? ",\n" : "\n");
  f << "}\n";
}

float time_step(ltn_plan* p, int s, int reps, int mode, bool warm = true) {
  auto& r = *p->rt;
  hipEvent_t a, b;
  HIPCHECK(hipEventCreate(&a));
  HIPCHECK(hipEventCreate(&b));
  if (warm) enqueue_step(p, s, r.B, false, mode);  // untimed warm-up launch
  HIPCHECK(hipEventRecord(a, r.st));
  for (int i = 0; i < reps; ++i) enqueue_step(p, s, r.B, false, mode);
  HIPCHECK(hipEventRecord(b, r.st));
  HIPCHECK(hipEventSynchronize(b));
  float ms = 0;
  HIPCHECK(hipEventElapsedTime(&ms, a, b));
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  check_launch();
  return ms / reps;
}

void drop_graphs(ltn_plan* p) {
  auto& r = *p->rt;
  for (int m = 0; m < 3; ++m) {
    if (r.graph[m]) (void)hipGraphExecDestroy(r.graph[m]);
    if (r.graph_src[m]) (void)hipGraphDestroy(r.graph_src[m]);
    r.graph[m] = nullptr;
    r.graph_src[m] = nullptr;
  }
  for (int m = 0; m < 2; ++m) {
    if (r.ggraph[m]) (void)hipGraphExecDestroy(r.ggraph[m]);
    if (r.ggraph_src[m]) (void)hipGraphDestroy(r.ggraph_src[m]);
    r.ggraph[m] = nullptr;
    r.ggraph_src[m] = nullptr;
  }
  r.gseq_valid = false;  // kernel choices or fusion may have changed
  r.fwd_kept = false;
  for (int m = 0; m < 3; ++m) r.fseq_valid[m] = false;
}

// Average duration of `launch` over reps launches (after one untimed launch
// when warm), with HIP events on the plan's stream.
template <typename F>
float time_launch(ltn_plan* p, F&& launch, int reps, bool warm) {
  auto& r = *p->rt;
  hipEvent_t a, b;
  HIPCHECK(hipEventCreate(&a));
  HIPCHECK(hipEventCreate(&b));
  if (warm) launch();
  HIPCHECK(hipEventRecord(a, r.st));
  for (int i = 0; i < reps; ++i) launch();
  HIPCHECK(hipEventRecord(b, r.st));
  HIPCHECK(hipEventSynchronize(b));
  float ms = 0;
  HIPCHECK(hipEventElapsedTime(&ms, a, b));
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  check_launch();
  return ms / reps;
}

// Tile choice for the adjoint products of the gradient sweep (plans bound for
// gradients, complex64): every complex64, split-K and three-part tile that fits a
// product's shape in either operand role, against the fixed rule, each timed as the
// sweep runs it (in place, or behind its permutations) on operands filled with
// numbers of order one: what an unused arena holds may be NaN, on which the
// three-part tiles take another way. Products that k_rowsum takes have no choice.
// Cache entries: [1000 kind + cfg, swap], or [-1, 0] for the fixed rule.
void tune_adjoint(ltn_plan* p, std::map<std::string, std::pair<int, int>>& cache, bool& dirty) {
  auto& r = *p->rt;
  using Choice = ltn_plan_impl::Choice;
  for (int s = 0; s < (int)p->steps.size(); ++s) {
    const StepPlan& sp = p->steps[s];
    if (!r.needs_grad[sp.out] || sp.m + sp.n + sp.k <= 16) continue;
    for (int which = 0; which < 2; ++which) {
      if (!r.needs_grad[which ? sp.b : sp.a]) continue;
      int tk;
      RowsumDesc rd;
      if (rowsum_fits(adj_generic_desc(p, s, which, r.B, &tk), rd)) continue;
      // dA: (m, n, k) with B's layout; dB: (n, m, k) with A's layout
      const int m = which ? sp.n : sp.m, k = which ? sp.m : sp.n, n = sp.k;
      const uint32_t key = adj_key(m, k, n);
      if (r.adj.count(key)) continue;
      std::ostringstream o;
      o << "g0_" << m << "_" << k << "_" << n << "_b" << r.B << kCandidates;
      const auto it = cache.find(o.str());
      Choice pick;  // kind 0: the fixed rule
      if (it != cache.end()) {
        const int kind = it->second.first >= 1000 ? it->second.first / 1000 : 0;
        const int cfg = it->second.first % 1000, sw = it->second.second != 0;
        const int rm = sw ? n : m, rn = sw ? m : n;
        if ((kind == 1 && gemm_config_fits(cfg, rm, k, rn, LTN_C64)) ||
            (kind == 5 && splitk_config_fits(cfg, rm, k, rn)) || (kind == 6 && parts_config_fits(cfg, rm, k, rn, LTN_C64))) {
          pick.kind = kind;
          pick.cfg = cfg;
          pick.swap = sw;
        }
      } else {
        const TensorPlan &tc = p->tensors[sp.out], &other = p->tensors[which ? sp.a : sp.b];
        launch_fill_spread(arena_ptr(p, tc.gcot), ((int64_t)r.B << tc.rank), r.st);
        launch_fill_spread(arena_ptr(p, other.goff), ((int64_t)r.B << other.rank), r.st);
        auto run = [&](const Choice& c) {
          r.adj[key] = c;
          enqueue_adjoint_product(p, s, which, r.B);
        };
        std::vector<Choice> cands(1);
        for (int sw = 0; sw < 2; ++sw)
          for (int c = 0; c < gemm_config_count(LTN_C64); ++c)
            if (sw ? gemm_config_fits(c, n, k, m, LTN_C64) : gemm_config_fits(c, m, k, n, LTN_C64)) {
              Choice ch;
              ch.kind = 1;
              ch.cfg = c;
              ch.swap = sw;
              cands.push_back(ch);
            }
        for (int sw = 0; sw < 2; ++sw)
          for (int c = 0; c < splitk_config_count(); ++c)
            if (sw ? splitk_config_fits(c, n, k, m) : splitk_config_fits(c, m, k, n)) {
              Choice ch;
              ch.kind = 5;
              ch.cfg = c;
              ch.swap = sw;
              cands.push_back(ch);
            }
        for (int sw = 0; sw < 2; ++sw)
          for (int c = 0; c < parts_config_count(LTN_C64); ++c)
            if (sw ? parts_config_fits(c, n, k, m, LTN_C64) : parts_config_fits(c, m, k, n, LTN_C64)) {
              Choice ch;
              ch.kind = 6;
              ch.cfg = c;
              ch.swap = sw;
              cands.push_back(ch);
            }
        float best = 1e30f;
        bool first = true;
        for (auto& c : cands) {
          float ms = time_launch(p, [&] { run(c); }, 1, first);
          first = false;
          if (ms > 2.0f * best) continue;
          if (ms < 2.0f)
            ms = std::min(ms, time_launch(p, [&] { run(c); }, 3, false));
          else if (ms < 1.05f * best)
            ms = std::min(ms, time_launch(p, [&] { run(c); }, 1, false));
          if (ms < best) {
            best = ms;
            pick = c;
          }
        }
        cache[o.str()] = pick.kind > 0 ? std::make_pair(1000 * pick.kind + pick.cfg, pick.swap) : std::make_pair(-1, 0);
        dirty = true;
      }
      r.adj[key] = pick;
    }
  }
}

}  // namespace

// Candidates: every MFMA tile configuration that fits the step in either
// operand role (split tiles first in the split modes, then complex64 tiles),
// the narrow-step kernel in either role (k + n <= 10), the split-sum kernel
// (m, n <= 3), and the generic kernel with 1, 8 or 64 threads per output on
// small steps.
// Cache entries: [kind * 1000 + cfg, swap] for MFMA kinds, [-tk, 0] for the
// generic kernel.
extern "C" ltn_status ltn_autotune(ltn_plan* p, int32_t mode, const char* cache_path) {
  return guarded([&] {
    auto& r = rt(p);
    check_mode(mode);
    auto cache = read_cache(cache_path);
    bool dirty = false;
    using Choice = ltn_plan_impl::Choice;
    const bool fp32_forward = r.grad && mode == LTN_C64;  // see bind_state
    auto encode = [](const Choice& c) {
      return c.kind > 0 ? std::make_pair(c.kind * 1000 + c.cfg, c.swap) : std::make_pair(-c.tk, 0);
    };
    auto decode = [](std::pair<int, int> e) {
      Choice c;
      if (e.first >= 0) {
        c.kind = e.first / 1000;
        c.cfg = e.first % 1000;
        c.swap = e.second != 0;
      } else {
        c.kind = 0;
        c.tk = -e.first;
      }
      return c;
    };
    // a cached choice that does not fit its step is not there
    auto cached = [&](const StepPlan& sp, Choice& c) {
      const auto it = cache.find(tune_key(mode, sp, r.B, fp32_forward));
      if (it == cache.end()) return false;
      c = decode(it->second);
      return !misfit(c, sp, mode) && !(fp32_forward && c.kind == 6);
    };
    // the synchronising time_step below must not run inside a capture
    // and a stale graph would keep the old kernels
    drop_graphs(p);
    // time on realistic values (power and clocks depend on the data): one
    // forward pass over slices 0.. fills every tensor of the arena, and in
    // split-fp16 mode the per-slice maxima (not needed when every step's
    // choice comes from the cache)
    bool all_cached = true;
    Choice hit;
    for (auto& sp : p->steps) all_cached = all_cached && cached(sp, hit);
    if (!all_cached) {
      set_ids(p, nullptr, 0, r.B, true);
      enqueue_forward(p, r.B, false, mode == LTN_C64 ? LTN_C64 : mode);
    }
    for (int s = 0; s < (int)p->steps.size(); ++s) {
      const StepPlan& sp = p->steps[s];
      const bool found = cached(sp, hit);
      std::vector<Choice> cands;
      if (found) {
        cands.push_back(hit);
      } else if (sp.m + sp.k + sp.n <= kWaveWork && r.choice[mode][s].kind == 0) {
        // one launch of such a step takes its launch's 10 us on any kernel; in a
        // run it is one wave's microsecond
        cands.push_back(r.choice[mode][s]);
      } else {
        for (int kind : {2, 1}) {
          if (kind == 2 && mode == LTN_C64) continue;
          int km = kind == 2 ? mode : LTN_C64;
          for (int sw = 0; sw < 2; ++sw)
            for (int c = 0; c < gemm_config_count(km); ++c)
              if (sw ? gemm_config_fits(c, sp.n, sp.k, sp.m, km) : gemm_config_fits(c, sp.m, sp.k, sp.n, km)) {
                Choice ch;
                ch.kind = kind;
                ch.cfg = c;
                ch.swap = sw;
                cands.push_back(ch);
              }
        }
        for (int sw = 0; sw < 2; ++sw) {
          if (sw ? narrow_fits(sp.n, sp.k, sp.m) : narrow_fits(sp.m, sp.k, sp.n)) {
            Choice ch;
            ch.kind = 3;
            ch.cfg = 0;
            ch.swap = sw;
            cands.push_back(ch);
          }
          if (sw ? narrow_rows_fits(sp.n, sp.k, sp.m) : narrow_rows_fits(sp.m, sp.k, sp.n)) {
            Choice ch;
            ch.kind = 3;
            ch.cfg = 1;
            ch.swap = sw;
            cands.push_back(ch);
          }
        }
        if (skinny_fits(sp.m, sp.k, sp.n)) {
          Choice ch;
          ch.kind = 4;
          ch.cfg = 0;
          cands.push_back(ch);
        }
        for (int sw = 0; sw < 2; ++sw)
          for (int c = 0; c < splitk_config_count(); ++c)
            if (sw ? splitk_config_fits(c, sp.n, sp.k, sp.m) : splitk_config_fits(c, sp.m, sp.k, sp.n)) {
              Choice ch;
              ch.kind = 5;
              ch.cfg = c;
              ch.swap = sw;
              cands.push_back(ch);
            }
        for (int sw = 0; sw < 2 && !fp32_forward; ++sw)
          for (int c = 0; c < parts_config_count(mode); ++c)
            if ((sw ? parts_config_fits(c, sp.n, sp.k, sp.m, mode) : parts_config_fits(c, sp.m, sp.k, sp.n, mode)) &&
                !parts_config_yields(c, sw ? sp.n : sp.m, sp.k, sw ? sp.m : sp.n, mode)) {
              Choice ch;
              ch.kind = 6;
              ch.cfg = c;
              ch.swap = sw;
              cands.push_back(ch);
            }
        // the generic kernel only competes on small steps (or when no tile fits)
        if (cands.empty() || (cands.size() == 1 && cands[0].kind == 4) || sp.m + sp.k + sp.n <= 22)
          for (int tk : {1, 8, 64})
            if (tk == 1 || (1 << sp.k) >= tk) {
              Choice ch;
              ch.tk = tk;
              cands.push_back(ch);
            }
      }
      // one launch of each candidate; clearly slower ones get no repeats,
      // short launches (timer and launch noise) three more, long ones one
      // more only when they come within 5 % of the best so far
      float best = 1e30f;
      Choice pick = cands[0];
      bool first = true;
      for (auto& c : cands) {
        r.choice[mode][s] = c;
        if (cands.size() == 1) break;
        float ms = time_step(p, s, 1, mode, first);
        first = false;
        if (ms > 2.0f * best) continue;
        if (ms < 2.0f)
          ms = std::min(ms, time_step(p, s, 3, mode, false));
        else if (ms < 1.05f * best)
          ms = std::min(ms, time_step(p, s, 1, mode, false));
        // launches of 10 us vary by a few percent: of equals the first stays, so
        // that tunings agree (and with them the rounding of what they compute)
        if (ms < best * (ms < 0.05f ? 0.98f : 1.f)) {
          best = ms;
          pick = c;
        }
      }
      r.choice[mode][s] = pick;
      if (!found) {
        cache[tune_key(mode, sp, r.B, fp32_forward)] = encode(pick);
        dirty = true;
      }
    }
    if (mode == LTN_C64 && r.grad) tune_adjoint(p, cache, dirty);
    if (dirty) write_cache(cache_path, cache);
    HIPCHECK(hipStreamSynchronize(r.st));
  });
}

extern "C" ltn_status ltn_profile_steps(ltn_plan* p, uint64_t first, int32_t mode, float* ms_out) {
  return guarded([&] {
    auto& r = rt(p);
    check_mode(mode);
    require(ms_out != nullptr, "ms_out is NULL");
    r.fwd_kept = false;
    set_ids(p, nullptr, first, r.B, true);
    const GatherDesc* gd = reinterpret_cast<const GatherDesc*>(r.ws + r.lay.gd_fwd);
    uint32_t* scales = nullptr;
    if (mode == LTN_SPLIT_F16) {
      scales = reinterpret_cast<uint32_t*>(r.ws + r.lay.scales);
      launch_fill_zero(scales, al((size_t)r.B * p->tensors.size() * 4), r.st);
    }
    launch_gather(gd, (int)p->leaves.size(), r.gather_chunks, r.max_leaf_elems,
                  reinterpret_cast<const float2*>(r.ws + r.lay.leafdata), arena_ptr(p, 0),
                  reinterpret_cast<const uint64_t*>(r.ws + r.lay.ids), r.B, scales, r.B, r.st);
    std::vector<hipEvent_t> ev(p->steps.size() + 1);
    for (auto& e : ev) HIPCHECK(hipEventCreate(&e));
    HIPCHECK(hipEventRecord(ev[0], r.st));
    for (int s = 0; s < (int)p->steps.size(); ++s) {
      enqueue_step(p, s, r.B, false, mode);
      HIPCHECK(hipEventRecord(ev[s + 1], r.st));
    }
    HIPCHECK(hipEventSynchronize(ev.back()));
    for (int s = 0; s < (int)p->steps.size(); ++s) HIPCHECK(hipEventElapsedTime(&ms_out[s], ev[s], ev[s + 1]));
    for (auto& e : ev) (void)hipEventDestroy(e);
    check_launch();
  });
}

extern "C" ltn_status ltn_set_fusion(ltn_plan* p, int32_t enable) {
  return guarded([&] {
    require(p && p->rt, "plan is not bound", LTN_E_STATE);
    drop_graphs(p);
    p->rt->fuse = enable != 0;
  });
}

extern "C" ltn_status ltn_set_step_kernel(ltn_plan* p, int32_t step, int32_t mode, int32_t kind,
                                          int32_t cfg, int32_t swap, int32_t tk) {
  return guarded([&] {
    require(p && p->rt, "plan is not bound");
    require(step >= 0 && step < (int32_t)p->steps.size(), "step out of range");
    check_mode(mode);
    ltn_plan_impl::Choice c;
    c.kind = kind;
    if (kind == 0) {
      c.tk = tk;
    } else {
      c.cfg = kind == 4 ? 0 : cfg;
      c.swap = swap && kind != 4 ? 1 : 0;
    }
    const char* why = misfit(c, p->steps[step], mode);
    require(!why, why ? why : "");
    drop_graphs(p);
    p->rt->choice[mode][step] = c;
  });
}

extern "C" ltn_status ltn_step_kernel(const ltn_plan* p, int32_t step, int32_t mode, int32_t* kind,
                                      int32_t* cfg, int32_t* swap, int32_t* tk) {
  return guarded([&] {
    require(p && p->rt, "plan is not bound");
    require(step >= 0 && step < (int32_t)p->steps.size(), "step out of range");
    check_mode(mode);
    const auto& c = p->rt->choice[mode][step];
    if (kind) *kind = c.kind;
    if (cfg) *cfg = c.kind > 0 ? c.cfg : -1;
    if (swap) *swap = c.swap;
    if (tk) *tk = c.tk;
  });
}

extern "C" const char* ltn_kernel_name(int32_t kind, int32_t cfg, int32_t mode) {
  if (mode < LTN_C64 || mode > LTN_SPLIT_BF16) return "?";
  switch (kind) {
    case 0: return "generic";
    case 1: return gemm_config_name(cfg, LTN_C64);
    case 2: return mode == LTN_C64 ? "?" : gemm_config_name(cfg, mode);
    case 3: return cfg == 0 ? "narrow_tile" : (cfg == 1 ? "narrow_rows" : "?");
    case 4: return cfg == 0 ? "split_sum" : "?";
    case 5: return splitk_config_name(cfg);
    case 6: return parts_config_name(cfg, mode);
  }
  return "?";
}

// Tile plan of a bit permutation (see k_permute): the tile holds the lowest
// 5 source bits, the sources of the lowest 5 destination bits and then the
// next source bits up to 12; the LDS swizzle spreads one half-wave's reads
// in destination order over distinct banks.
static PermuteDesc plan_permute(int32_t rank, const int32_t* perm, int64_t batch, bool conj) {
  std::vector<int> inv(rank, -1);
  for (int j = 0; j < rank; ++j) {
    require(perm[j] >= 0 && perm[j] < rank && inv[perm[j]] < 0, "perm is not a permutation");
    inv[perm[j]] = j;
  }
  PermuteDesc d{};
  d.rank = rank;
  d.batch = batch;
  const int t = std::min(rank, 5);
  std::vector<char> in_tile(rank, 0);
  for (int j = 0; j < t; ++j) in_tile[j] = 1;          // lowest source bits
  for (int y = 0; y < t; ++y) in_tile[inv[y]] = 1;     // sources of the lowest destination bits
  int nt = 0;
  for (int j = 0; j < rank; ++j) nt += in_tile[j];
  // filled up to 4096 elements with the next source bits, to fewer (1024 at
  // least, so that runs stay long) while that leaves CUs without a tile: 2^19
  // elements 8.3 -> 5.3 us, 2^16 7.4 -> 4.3
  int fill = std::min(rank, 12);
  while (fill > 10 && (batch << (rank - fill)) < 256) --fill;
  for (int j = 0; j < rank && nt < fill; ++j)
    if (!in_tile[j]) {
      in_tile[j] = 1;
      ++nt;
    }
  std::vector<int> tsrc, outer;
  for (int j = 0; j < rank; ++j) (in_tile[j] ? tsrc : outer).push_back(j);
  d.n_tile = (int)tsrc.size();
  d.n_outer = (int)outer.size();
  for (int k = 0; k < d.n_tile; ++k) d.tile_src[k] = (int8_t)tsrc[k];
  // destination order of the tile bits
  std::vector<std::pair<int, int>> dt;
  for (int k = 0; k < d.n_tile; ++k) dt.push_back({perm[tsrc[k]], k});
  std::sort(dt.begin(), dt.end());
  for (int r = 0; r < d.n_tile; ++r) {
    d.tile_dst[r] = (int8_t)dt[r].first;
    d.dst_tile[r] = (int8_t)dt[r].second;
  }
  for (int k = 0; k < d.n_outer; ++k) {
    d.outer_src[k] = (int8_t)outer[k];
    d.outer_dst[k] = (int8_t)perm[outer[k]];
  }
  // LDS swizzle: the tile bits read by one half-wave in destination order
  // are dst_tile[0..4]; those at tile bit >= 5 each get a distinct low bit
  // not already among them, so the 32 slots differ in their low 5 bits.
  {
    const int nr = std::min(d.n_tile, 5);
    bool used[5] = {false, false, false, false, false};
    for (int r = 0; r < nr; ++r)
      if (d.dst_tile[r] < 5) used[d.dst_tile[r]] = true;
    int next = 0;
    for (int r = 0; r < nr; ++r)
      if (d.dst_tile[r] >= 5) {
        while (used[next]) ++next;
        used[next] = true;
        d.swz[d.dst_tile[r] - 5] = (uint8_t)(1u << next);
      }
  }
  d.flip = conj ? (1ull << 63) : 0;
  return d;
}

extern "C" ltn_status ltn_permute(const void* d_in, void* d_out, int32_t rank, const int32_t* perm,
                                  int64_t batch, void* stream) {
  return guarded([&] {
    require(d_in && d_out, "NULL buffer");
    require(d_in != d_out, "ltn_permute does not work in place");
    require(rank >= 0 && rank <= 40, "rank must be in 0..40");
    require(batch >= 1, "batch must be >= 1");
    require(rank == 0 || perm != nullptr, "perm is NULL");
    require(rank == 0 || ((uintptr_t)d_in % 16 == 0 && (uintptr_t)d_out % 16 == 0),
            "d_in and d_out must be 16-byte aligned");
    for (int j = 0; j < rank; ++j) require(perm[j] >= 0 && perm[j] < rank, "perm is not a permutation");
    std::vector<char> seen(rank, 0);
    for (int j = 0; j < rank; ++j) {
      require(!seen[perm[j]], "perm is not a permutation");
      seen[perm[j]] = 1;
    }
    PermuteDesc d = plan_permute(rank, perm, batch, false);
    launch_permute(reinterpret_cast<const float2*>(d_in), reinterpret_cast<float2*>(d_out), d,
                   reinterpret_cast<hipStream_t>(stream));
    check_launch();
  });
}
