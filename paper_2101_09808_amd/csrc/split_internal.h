// Split-operand convolution: launch plan and geometry shared by the chooser
// (split_route.cpp) and the kernels (split_kernels.hip).
#pragma once

#include "conv_internal.h"

namespace convfwd {

// The layer as the caller states it (stride, padding; stride 1 without
// padding for the plain entry points).
struct SplitShape {
  int N, C, K, H, W, R, S;
  int sh, sw, ph, pw;
  int P, Q;
  int dtype;  // CONV_DTYPE_* of In and Ker
};

// How the operands of an MFMA step are staged (the kernels' MODE).
enum {
  // In staged and split in LDS [octet of 8 channels][pixel], read through its
  // na x nb phase images (na = min(sh, R), nb = min(sw, S)): tap (r, s) of
  // output (h, w) is pixel (h + r / sh, w + s / sw) of phase (r % sh, s % sw),
  // whose images have Hi = P + Rp - 1 rows.  Ker packed.
  SPLIT_CONV = 0,
  // at most 4 channels: LDS [pixel][4 channels], an MFMA operand's 8 values
  // are two neighbouring pixels; Hi = (P - 1) sh + R rows.  Ker packed.
  SPLIT_IMAGE = 1,
  // 1x1 layers with many output channels: Ker rows staged and split, In packed.
  SPLIT_POINT = 2,
};

// Launch geometry, passed by value to the kernels.
struct SplitGeom {
  int N, C, K, H, W, R, S, sh, sw, ph, pw, P, Q;
  int na, nb, Hi, rm, cm;   // phases; staged rows per image; staged rows / columns per output row / column
  int tr, tw;               // tile: output rows (flattened n P + h) x columns; POINT: 1 x pixels (flattened n P Q + p)
  int tiles_rows, tiles_cols, tiles_k, order, num_tiles;
  int in_rows, in_wp;       // staged rows, items per staged row
  int E, Epad;              // items per octet; LDS slots (16 bytes) per octet
  int co;                   // channel octets per chunk (IMAGE: 1)
  int nchunks, steps;       // chunks of 8 co channels; MFMA steps per chunk
  int blocks;               // 16-row blocks of the packed operand
  int items;                // staging items per chunk
  int ng, E4;               // vector staging: groups of pixels per staged row, per octet
  unsigned st_bytes, pk_bytes;  // staged tensor, packed operand
  int buf_bytes, tab_off;   // LDS: bytes of one staging buffer, offset of the step table
  FastDiv dv_E, dv_wp, dv_rows, dv_Hi, dv_P, dv_tw, dv_tiles_k, dv_tiles_cols, dv_tiles_rows, dv_nb, dv_PQ, dv_Ez, dv_wpz;
};

// One compiled instance of the split kernel.
struct SplitConfig {
  int id, mode;
  int vec;      // pixels per staging load (4: bf16 CONV layers of one chunk)
  int wk, wp, nwk, nwp, nwc, npl;
  int ni;       // staging items per thread, at most
  int ns;       // MFMA steps per chunk and wave group
  int one;      // one chunk only
  int occ;      // waves per SIMD it is declared for (its registers may allow more)
  int threads() const { return nwk * nwp * nwc * 64; }
};
const SplitConfig* split_configs(int* count);

// A launch: instance, geometry, dynamic LDS, bytes of the packed operand.
struct SplitPlan {
  const SplitConfig* cfg;
  SplitGeom g;
  int lds_bytes;
  size_t pk_bytes;
  double us;  // estimated time
};

// Geometry of a configuration and tile; false if it does not fit.
// tr x tw: the tile (POINT: ignored); co: channel octets per chunk.
bool split_geometry(const SplitShape& s, const SplitConfig& c, int tr, int tw, int order, int co, SplitPlan* p);
// The best plan by estimated time; false if no configuration takes the layer.
bool split_choose(const SplitShape& s, SplitPlan* p);
// Enqueues the packing and the convolution; Pk has p.pk_bytes bytes.
int split_launch(const SplitPlan& p, bool out_bf16, const void* In, const void* Ker, void* Pk, void* Out, void* stream);

}  // namespace convfwd
