// C ABI of the convolution library: argument validation, the per-shape plan
// cache and dispatch to the kernels.  The declarations and their contracts
// are in include/conv_fwd.h.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

#include "conv_internal.h"
#include "split_internal.h"

using namespace convfwd;

namespace {

const int64_t kMaxElems = (int64_t(1) << 31) - 1;

int validate_shape(int N, int C, int K, int H, int W, int R, int S) {
  if (N <= 0 || C <= 0 || K <= 0 || H <= 0 || W <= 0 || R <= 0 || S <= 0) return CONV_EINVAL;
  if (R > H || S > W) return CONV_EINVAL;
  const int64_t P = H - R + 1, Q = W - S + 1;
  if ((int64_t)N * C * H * W > kMaxElems) return CONV_ERANGE;
  if ((int64_t)K * C * R * S > kMaxElems) return CONV_ERANGE;
  if ((int64_t)N * K * P * Q > kMaxElems) return CONV_ERANGE;
  return CONV_OK;
}

// Per (shape, dtype, tensor alignment) the selected plan and its resolved launch.
struct Entry {
  conv_plan_t plan;
  const Variant* v = nullptr;  // none: no plan takes the shape (that is cached too)
  Geom g;
  int split = -1;  // the call takes the split-operand route: 1 yes, 0 no, -1 not looked up yet
};
typedef std::tuple<int, int, int, int, int, int, int, int, int> Key;
std::mutex g_mu;
std::map<Key, Entry> g_cache;

// Alignment bits of a call: vector loads of In (4 fp32) or Ker need a
// 16-byte aligned tensor; the transposing bf16 kernel loads In in dwords.
enum { ALIGN_KER = 1, ALIGN_IN = 2, ALIGN_IN4 = 4, ALIGN_ALL = 7 };

int alignment_of(const void* In, const void* Ker) {
  return ((reinterpret_cast<uintptr_t>(Ker) & 15) == 0 ? ALIGN_KER : 0) |
         ((reinterpret_cast<uintptr_t>(In) & 15) == 0 ? ALIGN_IN : 0) |
         ((reinterpret_cast<uintptr_t>(In) & 3) == 0 ? ALIGN_IN4 : 0);
}

// Does variant v run with tensors of this alignment?
bool variant_fits(const Variant& v, int dtype, int align) {
  const int elem = dtype == CONV_DTYPE_BF16 ? 2 : 4;
  if (v.ker_vec * elem > elem && v.family != FAMILY_BF16 && !(align & ALIGN_KER)) return false;
  if (v.family == FAMILY_DMA && v.in_vec > 1 && !(align & ALIGN_IN)) return false;
  if (v.family == FAMILY_BF16_TR && !(align & ALIGN_IN4)) return false;
  return true;
}

int select_entry(const Shape& s, int dtype, int align, Entry* e) {
  conv_plan_t p;
  int st = select_plan(s, dtype, &p);
  if (st != CONV_OK) return st;
  const Variant* v = find_variant(p.variant);
  if (v && !variant_fits(*v, dtype, align)) {
    // best plan of a variant whose loads suit the tensors' alignment
    std::vector<conv_plan_t> buf(4096);
    const int n = enumerate_plans(s, dtype, buf.data(), (int)buf.size());
    v = nullptr;
    for (int i = 0; i < n && i < (int)buf.size(); ++i) {
      const Variant* w = find_variant(buf[i].variant);
      if (w && variant_fits(*w, dtype, align)) {
        p = buf[i];
        v = w;
        break;
      }
    }
    if (!v) return CONV_ENOPLAN;
  }
  if (!v || !resolve_geom(s, *v, p, &e->g, nullptr)) return CONV_ENOPLAN;
  e->plan = p;
  e->v = v;
  return CONV_OK;
}

int cached_entry(const Shape& s, int dtype, int align, Entry* out) {
  const Key key{s.N, s.C, s.K, s.H, s.W, s.R, s.S, dtype, align};
  {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) {
      *out = it->second;
      return out->v ? CONV_OK : CONV_ENOPLAN;
    }
  }
  Entry e;
  const int st = select_entry(s, dtype, align, &e);
  if (st != CONV_OK && st != CONV_ENOPLAN) return st;
  if (st != CONV_OK) e.v = nullptr;
  std::lock_guard<std::mutex> lk(g_mu);
  *out = g_cache.emplace(key, e).first->second;  // (another thread may have tuned the layer meanwhile)
  return out->v ? CONV_OK : CONV_ENOPLAN;
}

// bf16 Out from the transposing bf16 kernel: its stores are 16 bytes only
// when the wave tile pairs neighbouring blocks (an even number of blocks per
// part, in rows of an even number of blocks); otherwise every output is a
// 2-byte store, eight times slower on the 226x226 layer.  Whether a tile
// pairs is fixed by the instance (rows max_ni, columns max_nk), as in the
// kernel's PAIRED.
bool pairs_bf16_out(const Variant& v) {
  if (v.family != FAMILY_BF16_TR) return true;
  const int cbr = v.max_nk / 16, wp = v.max_ni * cbr / 4;
  const int npart = wp % 2 == 0 ? 2 : 1, pb = wp / npart;
  return pb % 2 == 0 && cbr % 2 == 0;
}

// The plan of conv_fwd_bf16_out: the selected bf16 plan, unless 16-byte
// stores are possible (Q % 8 == 0, Out 16-byte aligned) and it does not pair
// them: then the best candidate that does.  Cached beside the other entries
// under its own dtype code.
constexpr int kBf16OutKey = 0x100;
int cached_entry_bf16_out(const Shape& s, int align, bool pair_possible, Entry* out) {
  Entry e;
  int st = cached_entry(s, CONV_DTYPE_BF16, align, &e);
  if (st != CONV_OK || !pair_possible || pairs_bf16_out(*e.v)) {
    *out = e;
    return st;
  }
  const Key key{s.N, s.C, s.K, s.H, s.W, s.R, s.S, CONV_DTYPE_BF16 | kBf16OutKey, align};
  {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) {
      *out = it->second;
      return CONV_OK;
    }
  }
  std::vector<conv_plan_t> buf(4096);
  const int n = std::min<int>(enumerate_plans(s, CONV_DTYPE_BF16, buf.data(), (int)buf.size()), (int)buf.size());
  for (int i = 0; i < n; ++i) {
    const Variant* w = find_variant(buf[i].variant);
    Geom g;
    if (!w || !variant_fits(*w, CONV_DTYPE_BF16, align) || !pairs_bf16_out(*w) ||
        !resolve_geom(s, *w, buf[i], &g, nullptr))
      continue;
    e.plan = buf[i];
    e.v = w;
    e.g = g;
    break;
  }
  {
    std::lock_guard<std::mutex> lk(g_mu);
    g_cache[key] = e;
  }
  *out = e;
  return CONV_OK;
}

int cached_plan(const Shape& s, int dtype, conv_plan_t* out) {
  Entry e;
  const int st = cached_entry(s, dtype, ALIGN_ALL, &e);
  if (st == CONV_OK) *out = e.plan;
  return st;
}

int run(const Shape& s, const void* In, const void* Ker, float* Out, const conv_plan_t& plan,
        void* stream) {
  const Variant* v = find_variant(plan.variant);
  if (!v || v->dtype != plan.dtype || v->phase_skip) return CONV_EINVAL;  // phase skip: conv_fwd_ex only
  if (!variant_fits(*v, plan.dtype, alignment_of(In, Ker))) return CONV_EINVAL;
  Geom g;
  if (!resolve_geom(s, *v, plan, &g, nullptr)) return CONV_EINVAL;
  return launch(*v, g, In, Ker, Out, stream);
}

// Selected plan for a call: cached per shape and tensor alignment.
// bf16 shapes that no bf16 kernel instance takes (other tap counts): the
// inputs are widened exactly to fp32 in a stream-ordered workspace and the
// fp32 plan runs -- the same products and fp32 sums.  out_bf16: Out is
// bf16, written by rounding an fp32 result kept in the workspace.
int run_bf16_widened(const Shape& s, const void* In, const void* Ker, void* Out, bool out_bf16, void* stream) {
  const size_t n_in = (size_t)s.N * s.C * s.H * s.W, n_ker = (size_t)s.K * s.C * s.R * s.S;
  const size_t n_out = out_bf16 ? (size_t)s.N * s.K * (s.H - s.R + 1) * (s.W - s.S + 1) : 0;
  const size_t a_in = (n_in * 4 + 255) / 256 * 256, a_ker = (n_ker * 4 + 255) / 256 * 256;
  Workspace w;
  int st = workspace_acquire(0, a_in + a_ker + n_out * 4, stream, &w);
  if (st != CONV_OK) return st;
  void* ws = w.ptr;
  float* in32 = static_cast<float*>(ws);
  float* ker32 = reinterpret_cast<float*>(static_cast<char*>(ws) + a_in);
  float* out32 = reinterpret_cast<float*>(static_cast<char*>(ws) + a_in + a_ker);
  st = launch_widen_bf16(In, in32, (int64_t)n_in, stream);
  if (st == CONV_OK) st = launch_widen_bf16(Ker, ker32, (int64_t)n_ker, stream);
  if (st == CONV_OK) {
    Entry e;
    st = cached_entry(s, CONV_DTYPE_F32, alignment_of(in32, ker32), &e);
    if (st == CONV_OK) st = launch(*e.v, e.g, in32, ker32, out_bf16 ? out32 : static_cast<float*>(Out), stream);
  }
  if (st == CONV_OK && out_bf16) st = launch_round_bf16(out32, Out, (int64_t)n_out, stream);
  const int freed = workspace_release(w, stream);
  return st == CONV_OK ? freed : st;
}

// The selected plan's kernel (the split-operand kernels are tried before).
int run_planned(const Shape& s, int dtype, const void* In, const void* Ker, float* Out, void* stream) {
  Entry e;
  const int st = cached_entry(s, dtype, alignment_of(In, Ker), &e);
  if (st == CONV_ENOPLAN && dtype == CONV_DTYPE_BF16) return run_bf16_widened(s, In, Ker, Out, false, stream);
  if (st != CONV_OK) return st;
  return launch(*e.v, e.g, In, Ker, Out, stream);
}

// conv_fwd_ex's plan for an fp32 strided or padded layer: the selector's
// plan of the inner problem (the best one whose loads suit the tensors as
// the kernel will see them), run reading In through the phase mapping when
// its kernel can.  Cached per layer, stride, padding and alignment.
struct ExEntry {
  Entry e;      // (its split field: of the strided layer)
  bool direct;  // e.g carries the phase mapping
};
typedef std::tuple<int, int, int, int, int, int, int, int, int, int, int, int> ExKey;
std::map<ExKey, ExEntry> g_ex_cache;

int select_ex_entry(const PhaseGeom& p, int align_direct, int align_split, ExEntry* out) {
  const Shape inner{p.N, p.C * p.na * p.nb, p.K, p.Hp, p.Wp, p.Rp, p.Sp};
  // (Ranking the candidates with the phase-split pass charged to plans that
  // cannot read In directly picked worse plans on the small layers, whose
  // predicted times are least reliable: Table 1's R1 28 -> 54 us.)
  // Stride-2 layers with odd taps also get the phase-skip variants, which
  // run only reading In directly.
  const bool skip_ok = p.na == 2 && p.nb == 2 && p.sh == 2 && p.sw == 2 && p.R == 2 * p.Rp - 1 &&
                       p.S == 2 * p.Sp - 1;
  std::vector<conv_plan_t> buf(4096);
  const int n =
      std::min<int>(enumerate_plans(inner, CONV_DTYPE_F32, buf.data(), (int)buf.size(), skip_ok), (int)buf.size());
  for (int i = 0; i < n; ++i) {
    const Variant* v = find_variant(buf[i].variant);
    Geom g;
    if (!v || !resolve_geom(inner, *v, buf[i], &g, nullptr)) continue;
    Geom gd = g;
    const bool direct = variant_fits(*v, CONV_DTYPE_F32, align_direct) && phase_direct(*v, p, CONV_DTYPE_F32, &gd);
    if (v->phase_skip && !direct) continue;
    if (!direct && !variant_fits(*v, CONV_DTYPE_F32, align_split)) continue;
    out->e.plan = buf[i];
    out->e.v = v;
    out->e.g = direct ? gd : g;
    out->direct = direct;
    return CONV_OK;
  }
  return CONV_ENOPLAN;
}

int cached_ex_entry(const PhaseGeom& p, int align_direct, int align_split, ExEntry* out) {
  const ExKey key{p.N, p.C, p.K, p.H, p.W, p.R, p.S, p.sh, p.sw, p.ph, p.pw, align_direct * 8 + align_split};
  {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_ex_cache.find(key);
    if (it != g_ex_cache.end()) {
      *out = it->second;
      return CONV_OK;
    }
  }
  ExEntry e;
  const int st = select_ex_entry(p, align_direct, align_split, &e);
  if (st != CONV_OK) return st;
  std::lock_guard<std::mutex> lk(g_mu);
  g_ex_cache[key] = e;
  *out = e;
  return CONV_OK;
}

// Inner stride-1 problem of a strided, padded convolution (polyphase rewrite).
int phase_geom(int N, int C, int K, int H, int W, int R, int S, int sh, int sw, int ph, int pw,
               PhaseGeom* p) {
  if (N <= 0 || C <= 0 || K <= 0 || H <= 0 || W <= 0 || R <= 0 || S <= 0) return CONV_EINVAL;
  if (sh < 1 || sw < 1 || ph < 0 || pw < 0 || sh > 64 || sw > 64 || ph > 4096 || pw > 4096) return CONV_EINVAL;
  if (H + 2 * ph < R || W + 2 * pw < S) return CONV_EINVAL;
  PhaseGeom q;
  q.N = N; q.C = C; q.K = K; q.H = H; q.W = W; q.R = R; q.S = S;
  q.sh = sh; q.sw = sw; q.ph = ph; q.pw = pw;
  q.P = (H + 2 * ph - R) / sh + 1;
  q.Q = (W + 2 * pw - S) / sw + 1;
  q.na = std::min(sh, R);
  q.nb = std::min(sw, S);
  q.Rp = (R + sh - 1) / sh;
  q.Sp = (S + sw - 1) / sw;
  q.Hp = q.P + q.Rp - 1;
  q.Wp = q.Q + q.Sp - 1;
  if ((int64_t)C * q.na * q.nb > kMaxElems) return CONV_ERANGE;
  const int st = validate_shape(N, C * q.na * q.nb, K, q.Hp, q.Wp, q.Rp, q.Sp);
  if (st != CONV_OK) return st;
  if ((int64_t)N * C * H * W > kMaxElems) return CONV_ERANGE;
  *p = q;
  return CONV_OK;
}

// Workspaces that the planned route takes for a call: their bytes summed, each
// rounded up to the 256-byte alignment of the arena's bump allocation, and
// the bytes of each level's kept buffer (a level's second workspace in one
// call is a fresh allocation).  Mirrors the dispatch of run_ex, run_planned,
// run_bf16_widened, launch (split partial sums) and launch_bf16_out; any
// workspace the library carves is 256-byte aligned, which is what the
// alignment of the plans that run on workspaces is computed with.
size_t up256(size_t b) { return (b + 255) / 256 * 256; }

struct Need {
  size_t total = 0;
  size_t level[3] = {0, 0, 0};
  void add(int l, size_t bytes) {
    total += up256(bytes);
    if (level[l] == 0) level[l] = bytes;
  }
  void add_split(const Geom& g) {
    if (g.split > 1) add(2, (size_t)g.split * g.N * g.K * g.P * g.Q * sizeof(float));
  }
};

// run_bf16_widened: exact fp32 copies of In and Ker (and for bf16 Out the
// fp32 one), then the fp32 plan
int widened_need(const Shape& s, bool out_bf16, Need* need) {
  const size_t n_in = (size_t)s.N * s.C * s.H * s.W, n_ker = (size_t)s.K * s.C * s.R * s.S;
  const size_t n_out = out_bf16 ? (size_t)s.N * s.K * (s.H - s.R + 1) * (s.W - s.S + 1) : 0;
  Entry e;
  const int st = cached_entry(s, CONV_DTYPE_F32, ALIGN_ALL, &e);
  if (st != CONV_OK) return st;
  need->add(0, up256(n_in * 4) + up256(n_ker * 4) + n_out * 4);
  need->add_split(e.g);
  return CONV_OK;
}

int selected_need(const Shape& s, int dtype, int align, Need* need) {
  Entry e;
  const int st = cached_entry(s, dtype, align, &e);
  if (st == CONV_ENOPLAN && dtype == CONV_DTYPE_BF16) return widened_need(s, false, need);
  if (st == CONV_OK) need->add_split(e.g);
  return st;
}

int bf16_out_need(const Shape& s, int align, bool pair_possible, Need* need) {
  Entry e;
  const int st = cached_entry_bf16_out(s, align, pair_possible, &e);
  if (st == CONV_ENOPLAN) return widened_need(s, true, need);
  if (st != CONV_OK) return st;
  if (bf16_out_staged(*e.v)) {
    need->add(1, (size_t)e.g.N * e.g.K * e.g.P * e.g.Q * sizeof(float));
    need->add_split(e.g);
  }
  return CONV_OK;
}

int ex_need(const PhaseGeom& p, int dtype, int align, Need* need) {
  const Shape s{p.N, p.C, p.K, p.H, p.W, p.R, p.S};
  if (p.sh == 1 && p.sw == 1 && p.ph == 0 && p.pw == 0) return selected_need(s, dtype, align, need);
  const size_t e = dtype == CONV_DTYPE_BF16 ? 2 : 4;
  const int Cp = p.C * p.na * p.nb;
  const bool ker_moves = p.na * p.nb > 1;
  const Shape inner{p.N, Cp, p.K, p.Hp, p.Wp, p.Rp, p.Sp};
  // the plan runs on (aligned) phase images and the rearranged or the
  // caller's Ker
  const int ker_al = ker_moves ? ALIGN_KER : (align & ALIGN_KER);
  const int al_split = ALIGN_IN | ALIGN_IN4 | ker_al;
  const size_t ker_ws = ker_moves ? (size_t)p.K * Cp * p.Rp * p.Sp * e : 0;
  const size_t in_ws = up256((size_t)p.N * Cp * p.Hp * p.Wp * e);
  if (dtype == CONV_DTYPE_F32) {
    ExEntry x;
    const int st = cached_ex_entry(p, (align & (ALIGN_IN | ALIGN_IN4)) | ker_al, al_split, &x);
    if (st != CONV_OK) return st;
    need->add(0, (x.direct ? 0 : in_ws) + ker_ws);
    need->add_split(x.e.g);
    return CONV_OK;
  }
  need->add(0, in_ws + ker_ws);
  return selected_need(inner, dtype, al_split, need);
}

// ---------------------------------------------------------------------------
// Split-operand route: layers that the kernels of split_kernels.hip run
// faster than the tile plan.  The two are compared by their estimates: the
// plan's ranking time plus its passes over In, Ker and Out, and the split
// plan's (split_choose).  The choice depends on the layer alone, not on the
// type of Out, so bf16 Out stays the rounded fp32 Out.
struct SplitEntry {
  bool use = false;
  SplitPlan p;
  // what the planned route keeps for 16-byte aligned tensors; bf16 Out
  // without and with 16-byte stores
  Need need, out_need[2];
};
typedef std::tuple<int, int, int, int, int, int, int, int, int, int, int> SplitKey;
std::map<SplitKey, SplitEntry> g_split_cache;

// Estimated time of the planned route for 16-byte aligned tensors.  The extra
// passes are charged what they measured: the phase split 0.2 elements per ns
// (3x3 C128 bf16 layer at batch 32: 19 us), the rearranged Ker 4.5 us, the
// widening and rounding passes 0.4 elements per ns.
int planned_time(const SplitShape& s, double* us) {
  const auto selected = [](const Shape& q, int dtype, double* t) {
    Entry e;
    int st = cached_entry(q, dtype, ALIGN_ALL, &e);
    double extra = 0;
    if (st == CONV_ENOPLAN && dtype == CONV_DTYPE_BF16) {
      st = cached_entry(q, CONV_DTYPE_F32, ALIGN_ALL, &e);
      extra = 6 + ((double)q.N * q.C * q.H * q.W + (double)q.K * q.C * q.R * q.S) / 0.4e6;
    }
    // (the transposing bf16 kernel's ranking times were taken between events:
    // 73 us for the 226x226 layer that runs in 59-70 us, 16.0 us for a
    // 166x106 one that runs in 12.3 us.  Of 61 wide layers of up to 32 channels
    // 8 keep their plans with this: five ran faster there, by 2% to 27%, and
    // three, 163x172 at batch 2, 163x144 at batch 8 and 128x96 at batch 4, would
    // have been 1.4 to 1.7 times as fast on the split kernels.  bf16 Out of the
    // 226x226 layer too: 63.5 against 58.0 us, with fp32 Out 59.6 against 65.0.)
    if (st == CONV_OK) *t = e.plan.rank_us * (e.v->family == FAMILY_BF16_TR ? 0.7 : 1.0) + extra;
    return st;
  };
  if (s.sh == 1 && s.sw == 1 && s.ph == 0 && s.pw == 0) {
    const Shape q{s.N, s.C, s.K, s.H, s.W, s.R, s.S};
    return selected(q, s.dtype, us);
  }
  PhaseGeom p;
  int st = phase_geom(s.N, s.C, s.K, s.H, s.W, s.R, s.S, s.sh, s.sw, s.ph, s.pw, &p);
  if (st != CONV_OK) return st;
  const double inner = (double)p.N * p.C * p.na * p.nb * p.Hp * p.Wp;
  double extra = p.na * p.nb > 1 ? 4.5 : 0.0;
  if (s.dtype == CONV_DTYPE_F32) {
    ExEntry x;
    st = cached_ex_entry(p, ALIGN_ALL, ALIGN_ALL, &x);
    if (st != CONV_OK) return st;
    *us = x.e.plan.rank_us;
    if (!x.direct) extra += 3 + inner / 0.2e6;
  } else {
    st = selected(Shape{p.N, p.C * p.na * p.nb, p.K, p.Hp, p.Wp, p.Rp, p.Sp}, s.dtype, us);
    if (st != CONV_OK) return st;
    extra += 3 + inner / 0.2e6;
  }
  *us += extra;
  return CONV_OK;
}

SplitShape split_shape(int N, int C, int K, int H, int W, int R, int S, int sh, int sw, int ph, int pw, int dtype) {
  return SplitShape{N, C, K, H, W, R, S, sh, sw, ph, pw, (H + 2 * ph - R) / sh + 1, (W + 2 * pw - S) / sw + 1, dtype};
}

// Is the split plan p to run instead of a plan estimated at us?  Estimates of
// grids that fill half the chip are within a few percent of each other's
// errors; for fewer tiles both are less reliable (a 672 x 814 1x1 layer on 6
// tiles: estimate 30 against 32 us, measured 30.0 against 23.3).
//
// The shorter layers need more: the plans of fp32 layers with taps measure 2 us
// less than their estimates below 20 us, the split kernels up to 2 us more
// (two launches, the sum of the channel groups).  The lines were drawn on 1400
// random layers of which 26 were slower than their plans by more than 1.5%,
// by up to 13%; of 2000 others that they route 16 are (8 of 886 fp32, 8 of 1114
// bf16; worst 3x3 stride 2 C19 K16 91x91 at batch 9, 18.8 -> 21.5 us), and all
// run 1.55 times (fp32) and 2.56 times (bf16) as fast as their plans in the
// geometric mean.
bool split_wins(const SplitShape& s, const SplitPlan& p, double us) {
  double share = p.g.num_tiles >= 128 ? 0.97 : 0.9;
  if (s.dtype == CONV_DTYPE_BF16) {
    // Of one-chunk layers this short half were faster on their plans (14 layers
    // in 0.91 to 1.12 times their plans' speed, 1.00 in the mean).
    if (p.cfg->vec > 1 && us < 13.2) return false;
  } else if (s.R * s.S > 1) {
    // The rearranged Ker of strided layers below 25 us costs them 2.0 us (66
    // layers: 1.2 to 2.1 in the mean of each 4 us), not 4.5.
    if (p.cfg->mode == SPLIT_CONV && (s.sh > 1 || s.sw > 1) && us < 30) us -= 2.5;
    // (strided image layers: 1.06 to 1.42 times their plans' speed here)
    if (us < 20 && (p.cfg->mode == SPLIT_CONV || (s.sh == 1 && s.sw == 1))) share = 0.77;
    else if (us < 27) share = 0.88;
  } else if (us < 26) {
    share = 0.88;
  }
  return p.us < share * us;
}

SplitEntry split_entry(const SplitShape& s) {
  const SplitKey key{s.N, s.C, s.K, s.H, s.W, s.R, s.S, s.sh * 64 + s.sw, s.ph, s.pw, s.dtype};
  {
    std::lock_guard<std::mutex> lk(g_mu);
    auto it = g_split_cache.find(key);
    if (it != g_split_cache.end()) return it->second;
  }
  SplitEntry e;
  double us = 0;
  // The packed operand also has to fit the allocation-free entry point's
  // scratch, so that it takes the same route.
  e.use = planned_time(s, &us) == CONV_OK && split_choose(s, &e.p) &&
          e.p.pk_bytes <= (size_t)CONV_NOALLOC_SCRATCH_BYTES && split_wins(s, e.p, us);
  PhaseGeom p;
  if (e.use && phase_geom(s.N, s.C, s.K, s.H, s.W, s.R, s.S, s.sh, s.sw, s.ph, s.pw, &p) == CONV_OK) {
    (void)ex_need(p, s.dtype, ALIGN_ALL, &e.need);
    if (s.dtype == CONV_DTYPE_BF16 && s.sh == 1 && s.sw == 1 && s.ph == 0 && s.pw == 0)
      for (int pair = 0; pair < 2; ++pair)
        (void)bf16_out_need(Shape{s.N, s.C, s.K, s.H, s.W, s.R, s.S}, ALIGN_ALL, pair != 0, &e.out_need[pair]);
  }
  std::lock_guard<std::mutex> lk(g_mu);
  g_split_cache[key] = e;
  return e;
}

// The route of a call whose plan entry does not know it yet: not where
// 16-byte loads of Ker or dword loads of bf16 In meet an unaligned tensor.
int split_route(const SplitShape& s, int align) {
  const SplitEntry e = split_entry(s);
  if (!e.use) return 0;
  if (e.p.cfg->mode == SPLIT_POINT && !(align & ALIGN_KER)) return 0;
  return s.dtype == CONV_DTYPE_BF16 && e.p.cfg->vec > 1 && !(align & ALIGN_IN4) ? 0 : 1;
}

// Does the call take the split-operand route?  Unless its workspace is the
// static scratch, not under graph capture: a graph would keep the address of
// a workspace that later calls may replace.
bool takes_split(const Entry& e, void* stream, bool static_scratch) {
  return e.split == 1 && (static_scratch || !stream_capturing(stream));
}

// cached_entry with the route looked up.  A bf16 layer without a bf16 plan
// has a route too (its planned one widens the inputs).
int routed_entry(const Shape& s, int dtype, int align, Entry* e) {
  const int st = cached_entry(s, dtype, align, e);
  if (st != CONV_OK && (st != CONV_ENOPLAN || dtype != CONV_DTYPE_BF16)) return st;
  if (e->split >= 0) return st;
  e->split = split_route(split_shape(s.N, s.C, s.K, s.H, s.W, s.R, s.S, 1, 1, 0, 0, dtype), align);
  std::lock_guard<std::mutex> lk(g_mu);
  Entry& kept = g_cache[Key{s.N, s.C, s.K, s.H, s.W, s.R, s.S, dtype, align}];
  if (kept.split < 0) kept.split = e->split;
  e->split = kept.split;  // (conv_fwd_tune on another thread may have decided meanwhile)
  return st;
}

int run_split(const SplitEntry& e, bool out_bf16, const void* In, const void* Ker, void* Out, void* stream) {
  Workspace w;
  int st = workspace_acquire(3, e.p.pk_bytes, stream, &w);
  if (st != CONV_OK) return st;
  st = split_launch(e.p, out_bf16, In, Ker, w.ptr, Out, stream);
  const int freed = workspace_release(w, stream);
  return st == CONV_OK ? freed : st;
}

// A call on the split-operand route keeps the buffers of its planned route
// too: under graph capture the same call runs that, and a program that has
// called the layer on this stream before captures no allocation.
void reserve_planned(const Need& need, void* stream) {
  for (int l = 0; l < 3; ++l)
    if (need.level[l] > 0) workspace_reserve(l, need.level[l], stream);
}

int run_selected(const Shape& s, int dtype, const void* In, const void* Ker, float* Out, void* stream) {
  Entry e;
  const int align = alignment_of(In, Ker), st = routed_entry(s, dtype, align, &e);
  if (takes_split(e, stream, false)) {
    SplitEntry se = split_entry(split_shape(s.N, s.C, s.K, s.H, s.W, s.R, s.S, 1, 1, 0, 0, dtype));
    if (align != ALIGN_ALL) (void)selected_need(s, dtype, align, &(se.need = Need()));
    reserve_planned(se.need, stream);
    return run_split(se, false, In, Ker, Out, stream);
  }
  if (st == CONV_ENOPLAN && dtype == CONV_DTYPE_BF16) return run_bf16_widened(s, In, Ker, Out, false, stream);
  if (st != CONV_OK) return st;
  return launch(*e.v, e.g, In, Ker, Out, stream);
}

// The fields of conv_fwd_geometry, in the header's order.
int export_geometry(const Variant& vr, const Geom& g, int lds, int32_t* out, int cap) {
  const Variant* v = &vr;
  const int32_t f[CONV_GEOM_FIELDS] = {
      g.N, g.C, g.K, g.H, g.W, g.R, g.S, g.P, g.Q,
      g.tr, g.tw, g.tiles_rows, g.tiles_cols, g.tiles_k,
      g.in_rows, g.in_wp, g.in_cstride, g.ker_rstride,
      g.nwk, g.nwp, g.order, g.num_tiles,
      g.lds_in_elems, g.lds_ker_elems, g.ni_in, g.ni_ker, g.nchunks,
      v->wk, v->wp, v->tc, v->rc, v->sc, v->max_ni, v->max_nk, v->ker_vec, v->threads, lds,
      v->family, v->in_vec, v->stages, g.stage_elems, g.in_region, (int32_t)g.in_bytes,
      (int32_t)g.ker_bytes, g.grid, v->phase_skip, 0, 0, g.split, g.cps, v->mfma32, v->groups(),
      g.nph, g.na, g.nb, g.sh, g.sw, g.ph, g.pw, g.C0, g.H0, g.W0, g.Wi,
      (int32_t)g.dv_in_cstride.m, g.dv_in_cstride.s, (int32_t)g.dv_in_wp.m, g.dv_in_wp.s,
      (int32_t)g.dv_H.m, g.dv_H.s, (int32_t)g.dv_ker_rstride.m, g.dv_ker_rstride.s,
      (int32_t)g.dv_tw.m, g.dv_tw.s, (int32_t)g.dv_P.m, g.dv_P.s, (int32_t)g.dv_nph.m, g.dv_nph.s,
      (int32_t)g.dv_nb.m, g.dv_nb.s, (int32_t)g.dv_Wi.m, g.dv_Wi.s, (int32_t)g.dv_tiles_k.m, g.dv_tiles_k.s,
      (int32_t)g.dv_tiles_cols.m, g.dv_tiles_cols.s, (int32_t)g.dv_tiles_rows.m, g.dv_tiles_rows.s};
  for (int i = 0; i < cap && i < CONV_GEOM_FIELDS; ++i) out[i] = f[i];
  return CONV_GEOM_FIELDS;
}

}  // namespace

extern "C" {

int conv_fwd(int N, int C, int K, int H, int W, int R, int S, const float* In, const float* Ker,
             float* Out, void* stream) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!In || !Ker || !Out) return CONV_ENULL;
  return run_selected(Shape{N, C, K, H, W, R, S}, CONV_DTYPE_F32, In, Ker, Out, stream);
}

int conv_fwd_bf16(int N, int C, int K, int H, int W, int R, int S, const uint16_t* In,
                  const uint16_t* Ker, float* Out, void* stream) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!In || !Ker || !Out) return CONV_ENULL;
  return run_selected(Shape{N, C, K, H, W, R, S}, CONV_DTYPE_BF16, In, Ker, Out, stream);
}

int conv_fwd_bf16_out(int N, int C, int K, int H, int W, int R, int S, const uint16_t* In,
                      const uint16_t* Ker, uint16_t* Out, void* stream) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!In || !Ker || !Out) return CONV_ENULL;
  Entry e;
  const Shape sh{N, C, K, H, W, R, S};
  const int align = alignment_of(In, Ker);
  routed_entry(sh, CONV_DTYPE_BF16, align, &e);
  const bool pair_possible = (W - S + 1) % 8 == 0 && (reinterpret_cast<uintptr_t>(Out) & 15) == 0;
  if (takes_split(e, stream, false)) {
    SplitEntry se = split_entry(split_shape(N, C, K, H, W, R, S, 1, 1, 0, 0, CONV_DTYPE_BF16));
    Need& need = se.out_need[pair_possible];
    if (align != ALIGN_ALL) (void)bf16_out_need(sh, align, pair_possible, &(need = Need()));
    reserve_planned(need, stream);
    return run_split(se, true, In, Ker, Out, stream);
  }
  st = cached_entry_bf16_out(sh, align, pair_possible, &e);
  if (st == CONV_ENOPLAN) return run_bf16_widened(sh, In, Ker, Out, true, stream);
  if (st != CONV_OK) return st;
  return launch_bf16_out(*e.v, e.g, In, Ker, Out, stream);
}

}  // extern "C"

namespace {

bool rewrites(const PhaseGeom& p) { return p.sh > 1 || p.sw > 1 || p.ph > 0 || p.pw > 0; }

// The plan entry of a strided or padded fp32 layer for these tensors (a
// strided Ker is rearranged into an aligned workspace, phase images too).
int ex_entry(const PhaseGeom& p, const void* In, const void* Ker, ExEntry* x) {
  const int ker_al = p.na * p.nb > 1 ? ALIGN_KER : (alignment_of(In, Ker) & ALIGN_KER);
  return cached_ex_entry(p, (alignment_of(In, Ker) & (ALIGN_IN | ALIGN_IN4)) | ker_al, ALIGN_IN | ALIGN_IN4 | ker_al, x);
}

// Route of a conv_fwd_ex call: CONV_OK with *split set where the
// split-operand kernels run, else with *x the plan entry of a strided or
// padded fp32 layer.
int ex_route(const PhaseGeom& p, int dtype, const void* In, const void* Ker, void* stream, bool static_scratch,
             bool* split, ExEntry* x) {
  const int align = alignment_of(In, Ker);
  const SplitShape q = split_shape(p.N, p.C, p.K, p.H, p.W, p.R, p.S, p.sh, p.sw, p.ph, p.pw, dtype);
  *split = false;
  if (!rewrites(p)) {
    routed_entry(Shape{p.N, p.C, p.K, p.H, p.W, p.R, p.S}, dtype, align, &x->e);
  } else if (dtype == CONV_DTYPE_F32) {
    const int st = ex_entry(p, In, Ker, x);
    if (st != CONV_OK) return st;
    if (x->e.split < 0) {
      x->e.split = split_route(q, align);
      const int ker_al = p.na * p.nb > 1 ? ALIGN_KER : (align & ALIGN_KER);
      const int al = ((align & (ALIGN_IN | ALIGN_IN4)) | ker_al) * 8 + (ALIGN_IN | ALIGN_IN4 | ker_al);
      std::lock_guard<std::mutex> lk(g_mu);
      g_ex_cache[ExKey{p.N, p.C, p.K, p.H, p.W, p.R, p.S, p.sh, p.sw, p.ph, p.pw, al}].e.split = x->e.split;
    }
  } else {
    x->e.split = split_route(q, align);
  }
  *split = takes_split(x->e, stream, static_scratch);
  return CONV_OK;
}

// The planned route of conv_fwd_ex (arguments already validated).
int run_ex(const PhaseGeom& p, int dtype, const void* In, const void* Ker, float* Out, void* stream, const ExEntry& x) {
  const int N = p.N, C = p.C, K = p.K, H = p.H, W = p.W, R = p.R, S = p.S;
  int st = CONV_OK;
  if (p.sh == 1 && p.sw == 1 && p.ph == 0 && p.pw == 0)
    return run_planned(Shape{N, C, K, H, W, R, S}, dtype, In, Ker, static_cast<float*>(Out), stream);
  const size_t e = dtype == CONV_DTYPE_BF16 ? 2 : 4;
  const int Cp = C * p.na * p.nb;
  // The rearranged Ker differs from Ker only with more than one phase (one
  // phase per axis means stride 1 or a single tap along it).
  const bool ker_moves = p.na * p.nb > 1;
  const Shape inner{N, Cp, K, p.Hp, p.Wp, p.Rp, p.Sp};
  if (dtype == CONV_DTYPE_F32) {
    // The plan either reads the caller's In through the phase mapping
    // (direct-to-LDS kernel: no pass over In) or runs on phase-split copies
    // in a workspace; a strided Ker is rearranged first either way.  The
    // workspaces are 256-byte aligned.
    const size_t in_ws = x.direct ? 0 : ((size_t)N * Cp * p.Hp * p.Wp * e + 255) / 256 * 256;
    const size_t ker_ws = ker_moves ? (size_t)K * Cp * p.Rp * p.Sp * e : 0;
    if (in_ws + ker_ws == 0) return launch(*x.e.v, x.e.g, In, Ker, Out, stream);
    Workspace w;
    st = workspace_acquire(0, in_ws + ker_ws, stream, &w);
    if (st != CONV_OK) return st;
    char* ws = static_cast<char*>(w.ptr);
    void* Kp = ker_moves ? ws + in_ws : nullptr;
    st = launch_phase_split(p, dtype, In, Ker, x.direct ? nullptr : ws, Kp, stream);
    if (st == CONV_OK)
      st = launch(*x.e.v, x.e.g, x.direct ? In : ws, ker_moves ? Kp : Ker, Out, stream);
    const int freed = workspace_release(w, stream);
    return st == CONV_OK ? freed : st;
  }
  // bf16: stream-ordered workspace with the phase images of In, then
  // (strided only) the rearranged Ker; at stride 1 the padded In meets the
  // original Ker
  const size_t in_bytes = ((size_t)N * Cp * p.Hp * p.Wp * e + 255) / 256 * 256;
  const size_t ker_bytes = ker_moves ? (size_t)K * Cp * p.Rp * p.Sp * e : 0;
  Workspace w;
  st = workspace_acquire(0, in_bytes + ker_bytes, stream, &w);
  if (st != CONV_OK) return st;
  char* ws = static_cast<char*>(w.ptr);
  void* Kp = ker_moves ? ws + in_bytes : nullptr;
  st = launch_phase_split(p, dtype, In, Ker, ws, Kp, stream);
  if (st == CONV_OK)
    st = run_planned(inner, dtype, ws, ker_moves ? Kp : Ker, Out, stream);
  const int freed = workspace_release(w, stream);
  return st == CONV_OK ? freed : st;
}

// Installs an arena on the calling thread for the lifetime of the guard.
struct ArenaGuard {
  explicit ArenaGuard(ScratchArena* a) { set_thread_arena(a); }
  ~ArenaGuard() { set_thread_arena(nullptr); }
};

}  // namespace

extern "C" {

int conv_fwd_ex(int N, int C, int K, int H, int W, int R, int S, int stride_h, int stride_w, int pad_h,
                int pad_w, int dtype, const void* In, const void* Ker, float* Out, void* stream) {
  PhaseGeom p;
  const int st = phase_geom(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, &p);
  if (st != CONV_OK) return st;
  if (!In || !Ker || !Out) return CONV_ENULL;
  if (dtype != CONV_DTYPE_F32 && dtype != CONV_DTYPE_BF16) return CONV_EINVAL;
  if (!rewrites(p)) return run_selected(Shape{N, C, K, H, W, R, S}, dtype, In, Ker, Out, stream);
  bool split = false;
  ExEntry x;
  const int rt = ex_route(p, dtype, In, Ker, stream, false, &split, &x);
  if (rt != CONV_OK) return rt;
  if (split) {
    SplitEntry se = split_entry(split_shape(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, dtype));
    const int align = alignment_of(In, Ker);
    if (align != ALIGN_ALL) (void)ex_need(p, dtype, align, &(se.need = Need()));
    reserve_planned(se.need, stream);
    return run_split(se, false, In, Ker, Out, stream);
  }
  return run_ex(p, dtype, In, Ker, Out, stream, x);
}

int conv_fwd_ex_noalloc(int N, int C, int K, int H, int W, int R, int S, int stride_h, int stride_w, int pad_h,
                        int pad_w, int dtype, const void* In, const void* Ker, float* Out, void* stream) {
  PhaseGeom p;
  int st = phase_geom(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, &p);
  if (st != CONV_OK) return st;
  if (!In || !Ker || !Out) return CONV_ENULL;
  if (dtype != CONV_DTYPE_F32 && dtype != CONV_DTYPE_BF16) return CONV_EINVAL;
  Need planned;
  st = ex_need(p, dtype, alignment_of(In, Ker), &planned);
  if (st != CONV_OK) return st;
  size_t need = planned.total;
  if (need > (size_t)CONV_NOALLOC_SCRATCH_BYTES) return CONV_ESCRATCH;
  bool split = false;
  ExEntry x;
  st = ex_route(p, dtype, In, Ker, stream, true, &split, &x);
  if (st != CONV_OK) return st;
  SplitEntry e;
  if (split) {
    e = split_entry(split_shape(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, dtype));
    need = e.p.pk_bytes;
  }
  void* base = nullptr;
  if (need > 0) {
    st = noalloc_scratch(&base);
    if (st != CONV_OK) return st;
  }
  ScratchArena arena{static_cast<char*>(base), need > 0 ? (size_t)CONV_NOALLOC_SCRATCH_BYTES : 0, 0};
  ArenaGuard guard(&arena);
  if (split) return run_split(e, false, In, Ker, Out, stream);
  return run_ex(p, dtype, In, Ker, Out, stream, x);
}

int conv_fwd_ex_plan(int N, int C, int K, int H, int W, int R, int S, int stride_h, int stride_w, int pad_h,
                     int pad_w, int dtype, conv_plan_t* plan_out, int32_t* direct) {
  PhaseGeom p;
  int st = phase_geom(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, &p);
  if (st != CONV_OK) return st;
  if (!plan_out) return CONV_ENULL;
  if (dtype != CONV_DTYPE_F32 && dtype != CONV_DTYPE_BF16) return CONV_EINVAL;
  const bool rewrite = stride_h > 1 || stride_w > 1 || pad_h > 0 || pad_w > 0;
  if (dtype == CONV_DTYPE_F32 && rewrite) {
    ExEntry x;
    st = cached_ex_entry(p, ALIGN_ALL, ALIGN_ALL, &x);
    if (st != CONV_OK) return st;
    *plan_out = x.e.plan;
    if (direct) *direct = x.direct ? 1 : 0;
    return CONV_OK;
  }
  if (direct) *direct = 0;
  return cached_plan(Shape{N, C * p.na * p.nb, K, p.Hp, p.Wp, p.Rp, p.Sp}, dtype, plan_out);
}

int conv_fwd_ex_inner_shape(int N, int C, int K, int H, int W, int R, int S, int stride_h, int stride_w,
                            int pad_h, int pad_w, int32_t inner[9]) {
  if (!inner) return CONV_ENULL;
  PhaseGeom p;
  const int st = phase_geom(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, &p);
  if (st != CONV_OK) return st;
  const int32_t v[9] = {N, C * p.na * p.nb, K, p.Hp, p.Wp, p.Rp, p.Sp, p.P, p.Q};
  for (int i = 0; i < 9; ++i) inner[i] = v[i];
  return CONV_OK;
}

int conv_fwd_plan(int N, int C, int K, int H, int W, int R, int S, int dtype,
                  conv_plan_t* plan_out) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!plan_out) return CONV_ENULL;
  if (dtype != CONV_DTYPE_F32 && dtype != CONV_DTYPE_BF16) return CONV_EINVAL;
  return cached_plan(Shape{N, C, K, H, W, R, S}, dtype, plan_out);
}

int conv_fwd_bf16_out_plan(int N, int C, int K, int H, int W, int R, int S, conv_plan_t* plan_out) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!plan_out) return CONV_ENULL;
  Entry e;
  st = cached_entry_bf16_out(Shape{N, C, K, H, W, R, S}, ALIGN_ALL, (W - S + 1) % 8 == 0, &e);
  if (st == CONV_OK) *plan_out = e.plan;
  return st;
}

int conv_fwd_with_plan(int N, int C, int K, int H, int W, int R, int S, const void* In,
                       const void* Ker, float* Out, const conv_plan_t* plan, void* stream) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!In || !Ker || !Out || !plan) return CONV_ENULL;
  const Shape s{N, C, K, H, W, R, S};
  conv_plan_t p = *plan;
  st = score_plan(s, &p);
  if (st != CONV_OK) return st;
  return run(s, In, Ker, Out, p, stream);
}

int conv_fwd_score_plan(int N, int C, int K, int H, int W, int R, int S, conv_plan_t* plan) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!plan) return CONV_ENULL;
  conv_plan_t p = *plan;
  st = score_plan(Shape{N, C, K, H, W, R, S}, &p);
  if (st != CONV_OK) return st;
  *plan = p;
  return CONV_OK;
}

int conv_fwd_candidates(int N, int C, int K, int H, int W, int R, int S, int dtype,
                        conv_plan_t* plans, int cap) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (cap < 0 || (cap > 0 && !plans)) return CONV_EINVAL;
  if (dtype != CONV_DTYPE_F32 && dtype != CONV_DTYPE_BF16) return CONV_EINVAL;
  const int n = enumerate_plans(Shape{N, C, K, H, W, R, S}, dtype, plans, cap);
  return n > 0 ? n : CONV_ENOPLAN;
}

int conv_fwd_tune(int N, int C, int K, int H, int W, int R, int S, int dtype, const void* In,
                  const void* Ker, float* Out, int top_n, int reps, void* stream,
                  conv_plan_t* plan_out, float* times_us) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!In || !Ker || !Out || !plan_out) return CONV_ENULL;
  if (dtype != CONV_DTYPE_F32 && dtype != CONV_DTYPE_BF16) return CONV_EINVAL;
  if (top_n < 1 || top_n > CONV_TUNE_MAX || reps < 1 || reps > 1000) return CONV_EINVAL;
  const Shape s{N, C, K, H, W, R, S};
  const int align = alignment_of(In, Ker);
  // the model's best plans (best first) that run with these tensors
  std::vector<conv_plan_t> buf(4096);
  const int n = enumerate_plans(s, dtype, buf.data(), (int)buf.size());
  std::vector<Entry> cand;
  for (int i = 0; i < n && i < (int)buf.size() && (int)cand.size() < top_n; ++i) {
    Entry e;
    e.plan = buf[i];
    e.v = find_variant(buf[i].variant);
    if (!e.v || !variant_fits(*e.v, dtype, align) || !resolve_geom(s, *e.v, e.plan, &e.g, nullptr)) continue;
    cand.push_back(e);
  }
  if (cand.empty()) return CONV_ENOPLAN;
  size_t best = 0;
  float best_us = 0.f;
  for (size_t i = 0; i < cand.size(); ++i) {
    float us = 0.f;
    const Entry& c = cand[i];
    st = time_launches([&] { return launch(*c.v, c.g, In, Ker, Out, stream); }, stream, reps, &us);
    if (st != CONV_OK) return st;
    if (times_us) times_us[i] = us;
    if (i == 0 || us < best_us) {
      best = i;
      best_us = us;
    }
  }
  // the split-operand kernels stay this layer's route only if they beat the plan
  const SplitShape q = split_shape(N, C, K, H, W, R, S, 1, 1, 0, 0, dtype);
  cand[best].split = split_route(q, align);
  if (cand[best].split) {
    const SplitEntry se = split_entry(q);
    float us = 0.f;
    st = time_launches([&] { return run_split(se, false, In, Ker, Out, stream); }, stream, reps, &us);
    if (st != CONV_OK) return st;
    cand[best].split = us < best_us ? 1 : 0;
  }
  {
    std::lock_guard<std::mutex> lk(g_mu);
    g_cache[Key{N, C, K, H, W, R, S, dtype, align}] = cand[best];
  }
  *plan_out = cand[best].plan;
  return (int)cand.size();
}

int conv_model_volume(const int perm[7], const int64_t N[7], const int64_t T[7], int out_factor,
                      double dv[3]) {
  if (!perm || !N || !T || !dv) return CONV_ENULL;
  int seen = 0;
  for (int i = 0; i < 7; ++i) {
    if (perm[i] < 0 || perm[i] > 6 || (seen >> perm[i]) & 1) return CONV_EINVAL;
    seen |= 1 << perm[i];
    if (T[i] < 1 || T[i] > N[i]) return CONV_EINVAL;
  }
  if (out_factor < 0) return CONV_EINVAL;
  model_volume(perm, N, T, out_factor, dv);
  return CONV_OK;
}

int conv_fwd_geometry(int N, int C, int K, int H, int W, int R, int S, const conv_plan_t* plan,
                      int32_t* out, int cap) {
  int st = validate_shape(N, C, K, H, W, R, S);
  if (st != CONV_OK) return st;
  if (!plan || (cap > 0 && !out)) return CONV_ENULL;
  const Variant* v = find_variant(plan->variant);
  if (!v || v->phase_skip) return CONV_EINVAL;  // phase skip: conv_fwd_ex_geometry only
  Geom g;
  int lds = 0;
  if (!resolve_geom(Shape{N, C, K, H, W, R, S}, *v, *plan, &g, &lds)) return CONV_EINVAL;
  return export_geometry(*v, g, lds, out, cap);
}

int conv_fwd_ex_geometry(int N, int C, int K, int H, int W, int R, int S, int stride_h, int stride_w, int pad_h,
                         int pad_w, const conv_plan_t* plan, int32_t* out, int cap) {
  PhaseGeom p;
  int st = phase_geom(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, &p);
  if (st != CONV_OK) return st;
  if (!plan || (cap > 0 && !out)) return CONV_ENULL;
  const Variant* v = find_variant(plan->variant);
  if (!v) return CONV_EINVAL;
  Geom g;
  int lds = 0;
  const Shape inner{N, C * p.na * p.nb, K, p.Hp, p.Wp, p.Rp, p.Sp};
  if (!resolve_geom(inner, *v, *plan, &g, &lds)) return CONV_EINVAL;
  const bool rewrite = stride_h > 1 || stride_w > 1 || pad_h > 0 || pad_w > 0;
  const bool direct = rewrite && phase_direct(*v, p, plan->dtype, &g);  // nph stays 0 where it does not apply
  if (v->phase_skip && !direct) return CONV_EINVAL;  // phase skip runs only reading In directly
  return export_geometry(*v, g, lds, out, cap);
}

int conv_fwd_split_plan(int N, int C, int K, int H, int W, int R, int S, int stride_h, int stride_w, int pad_h,
                        int pad_w, int dtype, int32_t* out, int cap) {
  PhaseGeom p;
  const int st = phase_geom(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, &p);
  if (st != CONV_OK) return st;
  if (cap > 0 && !out) return CONV_ENULL;
  if (dtype != CONV_DTYPE_F32 && dtype != CONV_DTYPE_BF16) return CONV_EINVAL;
  const SplitShape q = split_shape(N, C, K, H, W, R, S, stride_h, stride_w, pad_h, pad_w, dtype);
  SplitEntry e = split_entry(q);
  if (stride_h == 1 && stride_w == 1 && pad_h == 0 && pad_w == 0) {
    // conv_fwd_tune may have found the plan faster
    std::lock_guard<std::mutex> lk(g_mu);
    const auto it = g_cache.find(Key{N, C, K, H, W, R, S, dtype, ALIGN_ALL});
    if (it != g_cache.end() && it->second.split == 0) e.use = false;
  }
  int32_t f[CONV_SPLIT_FIELDS] = {0};
  if (e.use) {
    const SplitConfig& c = *e.p.cfg;
    const SplitGeom& g = e.p.g;
    const int32_t v[CONV_SPLIT_FIELDS] = {
        1, c.id, c.mode, c.vec, c.wk, c.wp, c.nwk, c.nwp, c.nwc, c.npl, c.ni, c.ns, c.one,
        g.tr, g.tw, g.tiles_rows, g.tiles_cols, g.tiles_k, g.order, g.num_tiles, g.na, g.nb, g.Hi, g.rm, g.cm,
        g.in_rows, g.in_wp, g.E, g.Epad, g.co, g.nchunks, g.steps, g.blocks, g.items, g.ng, g.buf_bytes, g.tab_off,
        e.p.lds_bytes, (int32_t)e.p.pk_bytes, (int32_t)e.p.us};
    std::memcpy(f, v, sizeof(f));
  }
  for (int i = 0; i < cap && i < CONV_SPLIT_FIELDS; ++i) out[i] = f[i];
  return CONV_SPLIT_FIELDS;
}

int conv_fwd_release_workspaces(void* stream) { return workspace_release_stream(stream); }

const char* conv_fwd_strerror(int status) {
  switch (status) {
    case CONV_OK: return "ok";
    case CONV_EINVAL: return "invalid argument (extent <= 0, R > H, S > W, or a bad plan)";
    case CONV_ENULL: return "null pointer";
    case CONV_ERANGE: return "tensor too large (2^31 elements or more)";
    case CONV_ENOPLAN: return "no kernel configuration fits this shape";
    case CONV_EHIP: return "HIP runtime error at launch";
    case CONV_ESCRATCH: return "the call needs more scratch than the allocation-free entry point holds";
    default: return "unknown status";
  }
}

}  // extern "C"
