// Chooser of the split-operand kernels (host only): launch geometry of a
// configuration and tile, and the configuration and tile with the least
// estimated time.
#include <algorithm>
#include <cmath>
#include <cstring>

#include "split_internal.h"

namespace convfwd {
namespace {
constexpr int kLds = 163840, kCus = 256;
int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
}  // namespace

bool split_geometry(const SplitShape& s, const SplitConfig& c, int tr, int tw, int order, int co, SplitPlan* p) {
  const bool bf16 = s.dtype == CONV_DTYPE_BF16;
  if ((c.npl == 1) != bf16) return false;
  const int64_t e = bf16 ? 2 : 4;
  const int64_t in_b = (int64_t)s.N * s.C * s.H * s.W * e, ker_b = (int64_t)s.K * s.C * s.R * s.S * e;
  const int64_t lim = int64_t(1) << 31;  // 32-bit byte offsets below the out-of-range marker
  if (in_b >= lim || ker_b >= lim) return false;
  const int BK = 16 * c.wk * c.nwk, BP = 16 * c.wp * c.nwp, NT = c.threads();
  const int64_t steps = c.mode == SPLIT_POINT   ? cdiv(co, 4)
                        : c.mode == SPLIT_IMAGE ? cdiv((int64_t)s.R * ((s.S + 1) / 2), 4)
                                                : cdiv((int64_t)co * s.R * s.S, 4);
  if (steps > 64 || cdiv(steps, c.nwc) != c.ns) return false;
  SplitGeom g;
  std::memset(&g, 0, sizeof(g));
  g.N = s.N; g.C = s.C; g.K = s.K; g.H = s.H; g.W = s.W; g.R = s.R; g.S = s.S;
  g.sh = s.sh; g.sw = s.sw; g.ph = s.ph; g.pw = s.pw; g.P = s.P; g.Q = s.Q;
  g.order = order;
  g.co = co;
  int64_t rows, cols, kt, chunks, blocks;
  if (c.mode == SPLIT_POINT) {
    if (s.R != 1 || s.S != 1 || s.sh != 1 || s.sw != 1 || s.ph || s.pw || s.C % 8) return false;
    g.na = g.nb = 1; g.rm = g.cm = 1; g.Hi = s.P;
    g.tr = 1; g.tw = BK;
    rows = cdiv((int64_t)s.N * s.P * s.Q, BK);
    cols = 1;
    kt = cdiv(s.K, BP);
    g.in_rows = 1; g.in_wp = BP; g.E = BP;
    g.Epad = BP + (co > 4 ? 8 : 0);
    chunks = cdiv(s.C, 8 * co);
    blocks = rows * (BK / 16);
    g.st_bytes = (unsigned)ker_b;
  } else {
    if (tr < 1 || tw < 1 || tw > s.Q || (int64_t)tr * tw > BP) return false;
    int extra, xcols;
    if (c.mode == SPLIT_IMAGE) {
      if (s.C > 4 || co != 1) return false;
      const int Sp = (s.S + 1) / 2;
      g.na = g.nb = 1; g.rm = s.sh; g.cm = s.sw;
      g.Hi = (s.P - 1) * s.sh + s.R;
      extra = s.R;
      xcols = ((tw - 1) * s.sw + 2 * Sp + 1) / 2;  // pixel pairs
      chunks = 1;
    } else {
      g.na = std::min(s.sh, s.R); g.nb = std::min(s.sw, s.S); g.rm = g.cm = 1;
      const int Rp = (s.R + s.sh - 1) / s.sh, Sp = (s.S + s.sw - 1) / s.sw;
      g.Hi = s.P + Rp - 1;
      extra = Rp;
      xcols = tw + Sp - 1;
      chunks = cdiv(s.C, 8 * co);
    }
    g.tr = tr; g.tw = tw;
    const int64_t NP = (int64_t)s.N * s.P;
    rows = cdiv(NP, tr);
    cols = cdiv(s.Q, tw);
    kt = cdiv(s.K, BK);
    int in_rows = 0;
    // staged rows of the worst tile: tiles repeat with the period of P / gcd(P, tr) tiles
    const int64_t lim_rt = std::min<int64_t>(rows, s.P);
    for (int64_t rt = 0; rt < lim_rt; ++rt) {
      const int64_t r0 = rt * tr, r1 = std::min<int64_t>(r0 + tr, NP) - 1;
      const int64_t a = (r0 / s.P) * g.Hi + (r0 % s.P) * g.rm, b = (r1 / s.P) * g.Hi + (r1 % s.P) * g.rm + extra - 1;
      in_rows = std::max<int>(in_rows, (int)(b - a + 1));
    }
    g.in_rows = in_rows; g.in_wp = xcols;
    const int64_t E = (int64_t)g.na * g.nb * in_rows * xcols;
    if (E > 16384) return false;
    g.E = (int)E;
    g.Epad = (int)cdiv(E + (c.vec > 1 ? 1 : 0), 16) * 16;  // (vector staging: a slot for pixels outside the tile)
    if (c.vec > 1) {
      // (bf16) groups of four pixels inside the image row, dword-aligned; both
      // column phases of a stride of 2
      if (s.W < 4 || s.sw > 2 || g.nb != s.sw || s.W % 2) return false;
      g.ng = (int)cdiv(std::min<int64_t>(s.W, (int64_t)(tw - 1) * s.sw + s.S + 1), 4);
      g.E4 = g.na * in_rows * g.ng;
    }
    blocks = kt * (BK / 16);
    g.st_bytes = (unsigned)in_b;
  }
  if (chunks > 1 && c.one) return false;
  g.items = co * (c.vec > 1 ? g.E4 : g.E);
  if (g.items > c.ni * NT) return false;
  // a grid dimension takes fewer than 2^32 threads
  if (rows * cols * kt >= (int64_t(1) << 24) || rows * cols * kt * NT >= (int64_t(1) << 32)) return false;
  g.tiles_rows = (int)rows; g.tiles_cols = (int)cols; g.tiles_k = (int)kt;
  g.num_tiles = (int)(rows * cols * kt);
  g.nchunks = (int)chunks; g.steps = (int)steps;
  const int64_t pk = blocks * chunks * steps * c.npl * 1024;
  if (pk >= lim || blocks >= (1 << 24)) return false;
  g.blocks = (int)blocks;
  g.pk_bytes = (unsigned)pk;
  // (bf16: units past the last tap read an octet of zeros)
  g.buf_bytes = (c.npl * co + (bf16 && 4 * steps > (int64_t)co * s.R * s.S ? 1 : 0)) * g.Epad * 16;
  const int stage = (c.one ? 1 : 2) * g.buf_bytes;
  const int red = c.nwc > 1 ? NT / 64 * c.wk * c.wp * 1024 : 0;
  g.tab_off = std::max(stage, red);
  const int lds = g.tab_off + 16 * g.steps + 16;  // (a word for the non-finite flag)
  if (lds > kLds) return false;
  if (c.mode == SPLIT_CONV && 4 * 16 * (8 * s.R * s.S + 1) * e > 65536) return false;  // packing kernel's LDS
  g.dv_E = make_fastdiv(c.vec > 1 ? g.E4 : g.E);
  g.dv_wp = make_fastdiv(c.vec > 1 ? g.ng : g.in_wp);
  g.dv_Ez = make_fastdiv(g.E);
  g.dv_wpz = make_fastdiv(g.in_wp);
  g.dv_rows = make_fastdiv(g.in_rows);
  g.dv_Hi = make_fastdiv(g.Hi);
  g.dv_P = make_fastdiv(g.P);
  g.dv_tw = make_fastdiv(g.tw);
  g.dv_tiles_k = make_fastdiv(g.tiles_k);
  g.dv_tiles_cols = make_fastdiv(g.tiles_cols);
  g.dv_tiles_rows = make_fastdiv(g.tiles_rows);
  g.dv_nb = make_fastdiv(c.mode == SPLIT_POINT ? co : g.nb);
  g.dv_PQ = make_fastdiv(g.P * g.Q);
  p->cfg = &c;
  p->g = g;
  p->lds_bytes = lds;
  p->pk_bytes = (size_t)pk;
  return true;
}

namespace {
// Estimated time in us.  Per-workgroup timestamps on MI355X (3x3 layers of
// 128 and 512 channels, 512 -> 1024 at batch 1): a chunk takes the MFMA time
// of its SIMD plus the time of the CU's vector-memory instructions, 17 cycles
// each (within one workgroup they hardly overlap; counters give 11 to 17);
// set-up, first loads and the last stores take 4-5 us per workgroup; the
// packing and the second launch 5 us plus the packing's traffic.  Workgroups
// per CU come from the waves per SIMD that an instance is declared for; the
// bf16 instances of eight waves are declared for one workgroup and have the
// registers for two (110 to 126), so their estimates are high where the tiles
// exceed the CUs (1x1 C16 K752 43x31 at batch 19: 40 us, measured 31).
double split_estimate(const SplitShape& s, const SplitPlan& p) {
  const SplitConfig& c = *p.cfg;
  const SplitGeom& g = p.g;
  const int waves = c.threads() / 64;
  const double prod = c.npl == 3 ? 6 : 1;
  const double mfma = (double)g.steps * c.wk * c.wp * prod * c.nwk * c.nwp / 4 * (waves > 4 ? 16.0 : 18.5);
  const double vmem = waves * (c.ni * (c.mode == SPLIT_POINT ? 2.0 : 8.0) + c.ns * c.wk * c.npl) * 17.0;
  const int res = std::max(1, std::min(c.occ * 4 / waves, kLds / p.lds_bytes));  // workgroups per CU
  const double per_cu = std::ceil((double)g.num_tiles / kCus);
  // a tile writes runs of tw outputs, and 128-byte lines cut between
  // workgroups cost twice (bf16 226x226 layer: 28-column tiles 111 us,
  // 112-column ones 62 us); whole rows follow each other
  const double run = g.tw * 4.0;
  const double out_us = (double)s.N * s.K * s.P * s.Q * 4.0 / 4.5e6 *
                        (c.mode == SPLIT_POINT || g.tw == s.Q ? 1.0 : (run + 124.0) / run);
  double main;
  if (res > 1 && per_cu > 1) {
    // workgroups on a CU overlap each other's loads, MFMAs and stores
    const double loop = g.nchunks * (std::max(mfma, vmem) + 0.35 * std::min(mfma, vmem)) / 1900.0;
    main = std::max(per_cu * loop, out_us) + std::ceil(per_cu / res) * 2.5 + out_us / per_cu;
  } else {
    const double loop = g.nchunks * (mfma + vmem) * 0.95 / 1900.0;
    main = per_cu * (loop + 3.5) + out_us;
  }
  // the staged halos, from the L2
  main += (double)g.num_tiles * g.nchunks * g.items * 8.0 * (c.vec > 1 ? c.vec : 1) * (c.npl == 3 ? 4.0 : 2.0) / 12e6;
  const double pack = 5.0 + (double)p.pk_bytes * (c.npl == 3 ? 5.0 / 3 : 2.0) / 5.0e6;
  return pack + 0.88 * main;
}
}  // namespace

bool split_choose(const SplitShape& s, SplitPlan* best) {
  int n = 0;
  const SplitConfig* cs = split_configs(&n);
  bool found = false;
  for (int ci = 0; ci < n; ++ci) {
    const SplitConfig& c = cs[ci];
    const int BP = 16 * c.wp * c.nwp;
    for (int co : {1, 2, 4, 8, 16}) {
      const int order = s.K > s.N * s.P * s.Q ? 1 : 0;
      if (c.mode == SPLIT_POINT) {
        SplitPlan p;
        if (co < 4 || !split_geometry(s, c, 1, 1, order, co, &p)) continue;
        p.us = split_estimate(s, p);
        if (!found || p.us < best->us) *best = p, found = true;
        continue;
      }
      for (int m = 1; m <= 16; ++m) {
        const int tw = (int)cdiv(s.Q, m);
        if (tw > BP) continue;
        const int tmax = (int)std::min<int64_t>(BP / tw, (int64_t)s.N * s.P);
        int prev = 0;
        for (int tr : {tmax, tmax - 1, tmax / s.P * s.P, (int)cdiv(s.P, cdiv(s.P, tmax))}) {
          if (tr < 1 || tr > tmax || tr == prev) continue;
          prev = tr;
          SplitPlan p;
          if (!split_geometry(s, c, tr, tw, order, co, &p)) continue;
          p.us = split_estimate(s, p);
          if (!found || p.us < best->us) *best = p, found = true;
        }
        if (tw == 1) break;
      }
    }
  }
  return found;
}

}  // namespace convfwd
