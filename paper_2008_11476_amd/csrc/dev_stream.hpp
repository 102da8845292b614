// Building blocks of the generated streaming kernels (codegen_stream.cpp).
//
// One wave owns a strip of image columns, LP (4 or 8) consecutive pixels per
// lane, and streams a band of rows top to bottom.  A row of a value is held
// as pairs of 16-bit elements (PR: pixel k and pixel k + LP/2 share a
// register, so one packed instruction handles two pixels) or, for F32, S32
// and wide intermediate results, as one register per pixel (WR).  With the
// pair layout the horizontal neighbour of both halves of pair k is pair
// k +- 1; only the pairs at the lane's ends need pixels of the adjacent lane,
// which arrive through DPP wave shifts.  The outermost lanes of a strip hold
// halo pixels and store nothing.
#pragma once
#include "dev_generic.hpp"

namespace hvx {

typedef short v2s __attribute__((ext_vector_type(2)));
typedef unsigned short v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v2w __attribute__((ext_vector_type(2)));
typedef uint32_t v4w __attribute__((ext_vector_type(4)));

// ---- packed 16-bit arithmetic (two pixels per instruction) -------------------
#define HVX_PK2(name, T, expr)                                          \
  __device__ __forceinline__ uint32_t name(uint32_t a_, uint32_t b_) {  \
    const T a = __builtin_bit_cast(T, a_), b = __builtin_bit_cast(T, b_); \
    return __builtin_bit_cast(uint32_t, (T)(expr));                     \
  }
HVX_PK2(pk_add, v2u, a + b)
HVX_PK2(pk_sub, v2u, a - b)
HVX_PK2(pk_mul, v2u, a* b)
HVX_PK2(pk_max, v2s, __builtin_elementwise_max(a, b))
HVX_PK2(pk_min, v2s, __builtin_elementwise_min(a, b))
HVX_PK2(pk_minu, v2u, __builtin_elementwise_min(a, b))
HVX_PK2(pk_adds, v2s, __builtin_elementwise_add_sat(a, b))
HVX_PK2(pk_subs, v2s, __builtin_elementwise_sub_sat(a, b))
#undef HVX_PK2
__device__ __forceinline__ uint32_t pk_shr(uint32_t a, int s) {
  return __builtin_bit_cast(uint32_t, (v2u)(__builtin_bit_cast(v2u, a) >> (unsigned short)s));
}
__device__ __forceinline__ uint32_t pk_sar(uint32_t a, int s) {
  return __builtin_bit_cast(uint32_t, (v2s)(__builtin_bit_cast(v2s, a) >> (short)s));
}
__device__ __forceinline__ constexpr uint32_t pk_c(int c) { return ((uint32_t)c & 0xFFFFu) * 0x10001u; }
// acc + c e, one instruction (the compiler does not form it from a product and a sum)
template <int C>
__device__ __forceinline__ uint32_t pk_mad(uint32_t e, uint32_t acc) {
  uint32_t r;
  if constexpr (C >= 1 && C <= 64)  // an inline constant, taken from the low half for both halves
    asm("v_pk_mad_u16 %0, %1, %3, %2 op_sel_hi:[1,0,1]" : "=v"(r) : "v"(e), "v"(acc), "n"(C));
  else
    asm("v_pk_mad_u16 %0, %1, %3, %2" : "=v"(r) : "v"(e), "v"(acc), "s"(pk_c(C)));
  return r;
}
__device__ __forceinline__ uint32_t bit_sel(uint32_t m, uint32_t a, uint32_t b) {
  return __builtin_amdgcn_bitop3_b32(m, a, b, 0xCA);
}
// all ones in the halves whose element is negative
__device__ __forceinline__ uint32_t pk_neg_mask(uint32_t a) { return pk_sar(a, 15); }
// a / 2^s toward zero (signed)
__device__ __forceinline__ uint32_t pk_div2(uint32_t a, int s) {
  return s == 0 ? a : pk_sar(pk_add(a, pk_shr(pk_sar(a, 15), 16 - s)), s);
}
// user kernels' comparison and selection on pairs (gt: 1 or 0)
__device__ __forceinline__ uint32_t pk_gt(uint32_t a, uint32_t b) { return pk_shr(pk_subs(b, a), 15); }
__device__ __forceinline__ uint32_t pk_selnz(uint32_t p, uint32_t x, uint32_t y) {
  return bit_sel(pk_neg_mask(p | pk_sub(0u, p)), x, y);
}

// ---- neighbouring lanes ---------------------------------------------------------
// Lane i receives lane i - 1's (i + 1's) register.  The empty asm keeps the
// move a separate instruction: folded into a consuming add or subtract, a
// whole-wave shift gave wrong results on gfx950.
__device__ __forceinline__ uint32_t lane_left(uint32_t v) {
  uint32_t r = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xF, 0xF, true);
  asm("" : "+v"(r));
  return r;
}
__device__ __forceinline__ uint32_t lane_right(uint32_t v) {
  uint32_t r = (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xF, 0xF, true);
  asm("" : "+v"(r));
  return r;
}

template <int LP>
struct PR {  // a row's pixels of one lane as 16-bit pairs
  uint32_t v[LP / 2];
};
template <int LP>
struct WR {  // one register per pixel
  int v[LP];
};
// rows extended by R pixels on each side: entry R + k is pair (pixel) k
template <int LP, int R>
struct PX {
  uint32_t v[LP / 2 + 2 * R];
};
template <int LP, int R>
struct WX {
  int v[LP + 2 * R];
};

template <int R, int LP>
__device__ __forceinline__ PX<LP, R> ext(const PR<LP>& p) {
  PX<LP, R> e;
#pragma unroll
  for (int k = 0; k < LP / 2; ++k) e.v[R + k] = p.v[k];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const uint32_t l = p.v[LP / 2 - 1 - i], r = p.v[i];
    e.v[R - 1 - i] = __builtin_amdgcn_alignbit(l, lane_left(l), 16);
    e.v[R + LP / 2 + i] = __builtin_amdgcn_alignbit(lane_right(r), r, 16);
  }
  return e;
}
template <int R, int LP>
__device__ __forceinline__ WX<LP, R> ext(const WR<LP>& p) {
  WX<LP, R> e;
#pragma unroll
  for (int k = 0; k < LP; ++k) e.v[R + k] = p.v[k];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    e.v[R - 1 - i] = (int)lane_left((uint32_t)p.v[LP - 1 - i]);
    e.v[R + LP + i] = (int)lane_right((uint32_t)p.v[i]);
  }
  return e;
}

template <int LP>
__device__ __forceinline__ void fill(PR<LP>& r, int c) {
#pragma unroll
  for (int k = 0; k < LP / 2; ++k) r.v[k] = pk_c(c);
}
template <int LP>
__device__ __forceinline__ void fill(WR<LP>& r, int c) {
#pragma unroll
  for (int k = 0; k < LP; ++k) r.v[k] = c;
}
template <int LP>
__device__ __forceinline__ WR<LP> wide(const PR<LP>& p) {  // signed 16-bit elements
  WR<LP> w;
#pragma unroll
  for (int k = 0; k < LP / 2; ++k) {
    w.v[k] = (int)(int16_t)(uint16_t)p.v[k];
    w.v[k + LP / 2] = (int)p.v[k] >> 16;
  }
  return w;
}
template <int LP>
__device__ __forceinline__ const WR<LP>& wide(const WR<LP>& w) {
  return w;
}
template <int LP>
__device__ __forceinline__ PR<LP> packed(const WR<LP>& w) {
  PR<LP> p;
#pragma unroll
  for (int k = 0; k < LP / 2; ++k)
    p.v[k] = __builtin_amdgcn_perm((uint32_t)w.v[k + LP / 2], (uint32_t)w.v[k], 0x05040100u);
  return p;
}

// ---- rows in memory ----------------------------------------------------------------
// Rows are read and written through buffer descriptors of one row each, made
// from its (wave-uniform) address: the lane's byte offset is the only vector
// operand, a lane that must not store has an offset outside the descriptor
// (the hardware drops it) and a row that must not be touched has an empty
// one.  So a row's code has no branch around its loads and stores, and the
// compiler counts the outstanding ones exactly.
constexpr uint32_t kNoLane = 0x80000000u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* base, int64_t pitch, int row, uint32_t bytes) {
  const uint64_t a = (uint64_t)base + (uint64_t)((int64_t)row * pitch);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
  const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)bytes);
  return __builtin_amdgcn_make_buffer_rsrc((void*)((uint64_t)hi << 32 | lo), 0, (int)n, 0x00027000);
}

template <int NB>  // bytes per lane: 4, 8, 16 or 32
struct Raw {
  uint32_t d[NB / 4];
};
template <int NB>
__device__ __forceinline__ Raw<NB> row_load(const void* base, int64_t pitch, int row, uint32_t bytes, uint32_t off) {
  const __amdgpu_buffer_rsrc_t r = row_rsrc(base, pitch, row, bytes);
  Raw<NB> x;
  if constexpr (NB == 4) {
    x.d[0] = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
  } else if constexpr (NB == 8) {
    const v2w q = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0);
    x.d[0] = q.x;
    x.d[1] = q.y;
  } else {
#pragma unroll
    for (int i = 0; i < NB / 16; ++i) {
      const v4w q = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16 * i, 0, 0);
      x.d[4 * i] = q.x;
      x.d[4 * i + 1] = q.y;
      x.d[4 * i + 2] = q.z;
      x.d[4 * i + 3] = q.w;
    }
  }
  return x;
}
// AUX 2: non-temporal
template <int NB, int AUX>
__device__ __forceinline__ void row_store(const Raw<NB>& x, __amdgpu_buffer_rsrc_t r, uint32_t off) {
  if constexpr (NB == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(x.d[0], r, off, 0, AUX);
  } else if constexpr (NB == 8) {
    __builtin_amdgcn_raw_buffer_store_b64(v2w{x.d[0], x.d[1]}, r, off, 0, AUX);
  } else {
#pragma unroll
    for (int i = 0; i < NB / 16; ++i)
      __builtin_amdgcn_raw_buffer_store_b128(v4w{x.d[4 * i], x.d[4 * i + 1], x.d[4 * i + 2], x.d[4 * i + 3]}, r,
                                             off + 16 * i, 0, AUX);
  }
}

// loaded bytes -> a row (U8, S16 and UYVY elements packed; S32 and F32 wide)
template <int DF, int LP>
__device__ __forceinline__ PR<LP> unpack_pk(const Raw<LP*(DF == DF_U8 ? 1 : 2)>& x) {
  PR<LP> p;
  if constexpr (DF == DF_U8 && LP == 4) {
    p.v[0] = __builtin_amdgcn_perm(0u, x.d[0], 0x0c020c00u);
    p.v[1] = __builtin_amdgcn_perm(0u, x.d[0], 0x0c030c01u);
  } else if constexpr (DF == DF_U8) {
#pragma unroll
    for (int k = 0; k < 4; ++k) p.v[k] = __builtin_amdgcn_perm(x.d[1], x.d[0], 0x0c040c00u + 0x00010001u * k);
  } else {
#pragma unroll
    for (int k = 0; k < LP / 2; ++k)
      p.v[k] = __builtin_amdgcn_perm(x.d[LP / 4 + k / 2], x.d[k / 2], (k & 1) ? 0x07060302u : 0x05040100u);
  }
  return p;
}
template <int LP>
__device__ __forceinline__ WR<LP> unpack_wd(const Raw<LP * 4>& x) {
  WR<LP> w;
#pragma unroll
  for (int k = 0; k < LP; ++k) w.v[k] = (int)x.d[k];
  return w;
}
// a row -> bytes to store
template <int DF, int LP>
__device__ __forceinline__ Raw<LP*(DF == DF_U8 ? 1 : 2)> pack_row(const PR<LP>& p) {
  Raw<LP*(DF == DF_U8 ? 1 : 2)> x;
  if constexpr (DF == DF_U8) {
    const uint32_t t0 = p.v[0] | p.v[1] << 8;  // elements lie in 0..255
    if constexpr (LP == 4) {
      x.d[0] = t0;
    } else {
      const uint32_t t1 = p.v[2] | p.v[3] << 8;
      x.d[0] = __builtin_amdgcn_perm(t1, t0, 0x05040100u);
      x.d[1] = __builtin_amdgcn_perm(t1, t0, 0x07060302u);
    }
  } else {
#pragma unroll
    for (int k = 0; k < LP / 4; ++k) {
      x.d[k] = __builtin_amdgcn_perm(p.v[2 * k + 1], p.v[2 * k], 0x05040100u);
      x.d[LP / 4 + k] = __builtin_amdgcn_perm(p.v[2 * k + 1], p.v[2 * k], 0x07060302u);
    }
  }
  return x;
}
template <int DF, int LP>
__device__ __forceinline__ Raw<LP * 4> pack_row(const WR<LP>& w) {
  Raw<LP * 4> x;
#pragma unroll
  for (int k = 0; k < LP; ++k) x.d[k] = (uint32_t)w.v[k];
  return x;
}

// ---- the strip, and positions outside the image --------------------------------------
template <int LP>
struct Strip {
  int x0;        // first pixel of the lane
  int W, H;
  int zl;        // lane holding x = 0, or -1
  int rl, rq;    // lane and pixel within it holding x = W - 1 (the lane may lie outside the wave)
  bool left;     // the lane lies left of the image
  bool whole;    // x = W - 1 ends a lane (uniform)
  uint32_t ml;   // the high half in the lane just left of x = 0
  uint32_t mr[2][LP / 2];  // pairs' pixels from W, and from W + 1 on
  bool keep;     // the lane stores all its pixels
  bool ragged;   // the lane stores the first W - x0 of its pixels
};
template <int LP>
__device__ __forceinline__ Strip<LP> make_strip(int strip, int halo, int out_lanes, int W, int H) {
  Strip<LP> s;
  const int lane = (int)(threadIdx.x & 63);
  const int base = (strip * out_lanes - halo) * LP;  // the first lane's first pixel (may be negative)
  s.x0 = base + lane * LP;
  s.W = W;
  s.H = H;
  s.zl = strip == 0 ? halo : -1;
  // (unsigned: rq is then known to lie in 0 .. LP - 1, which saves an edge
  // strip's row of F32 pixels 6 of 164 vector instructions)
  s.rl = (int)((unsigned)(W - 1 - base) / LP);
  s.rq = (int)((unsigned)(W - 1) % LP);
  s.left = s.x0 < 0;
  s.ml = s.x0 == -LP ? 0xFFFF0000u : 0u;
#pragma unroll
  for (int k = 0; k < LP / 2; ++k)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      s.mr[j][k] = (s.x0 + k >= W + j ? 0xFFFFu : 0u) | (s.x0 + k + LP / 2 >= W + j ? 0xFFFF0000u : 0u);
  s.whole = W % LP == 0;
  const bool own = lane >= halo && lane < halo + out_lanes && s.x0 < W;
  s.keep = own && s.x0 + LP <= W;
  s.ragged = own && s.x0 + LP > W;
  return s;
}

// pixel q (uniform) of lane `lane` (uniform), in every lane; picked with
// uniform masks (a chain of selects would become an indexed access to scratch
// memory)
template <int LP>
__device__ __forceinline__ int strip_px(const PR<LP>& p, int lane, int q) {
  uint32_t v = 0;
#pragma unroll
  for (int k = 0; k < LP / 2; ++k) v |= p.v[k] & (q % (LP / 2) == k ? ~0u : 0u);
  const uint32_t s = (uint32_t)__builtin_amdgcn_readlane((int)v, lane & 63);
  return (int)(q >= LP / 2 ? s >> 16 : s & 0xFFFFu);
}
template <int LP>
__device__ __forceinline__ int strip_px(const WR<LP>& p, int lane, int q) {
  int v = 0;
#pragma unroll
  for (int k = 0; k < LP; ++k) v |= p.v[k] & (q == k ? ~0 : 0);
  return __builtin_amdgcn_readlane(v, lane & 63);
}
// the element c where `m` holds for the pixel
template <int LP, class M>
__device__ __forceinline__ void put_where(PR<LP>& p, int c, const M& m) {
#pragma unroll
  for (int k = 0; k < LP / 2; ++k)
    p.v[k] = bit_sel((m(k) ? 0xFFFFu : 0u) | (m(k + LP / 2) ? 0xFFFF0000u : 0u), pk_c(c), p.v[k]);
}
template <int LP, class M>
__device__ __forceinline__ void put_where(WR<LP>& p, int c, const M& m) {
#pragma unroll
  for (int k = 0; k < LP; ++k) p.v[k] = m(k) ? c : p.v[k];
}

// Position read for x in [-2, n + 1] under the MIRROR border (reflect-101,
// repeated: a two-pixel axis has period two).
__device__ __forceinline__ int mirror_near(int x, int n) {
  if (n <= 2) return n == 1 ? 0 : x & 1;
  return x < 0 ? -x : (x < n ? x : 2 * (n - 1) - x);
}

// Columns outside the image take the border rule MODE of the operators that
// read the value (R: their largest horizontal radius; R = 0: none).  Only
// the strips at the image's left and right edge hold such columns.  On the
// left the R pixels beside the image lie in one lane and come from the next
// by a lane shift; on the right the pixel they repeat may lie anywhere in
// its lane and is read into a scalar.  No branches: they would cost more than
// the few instructions, in registers moved where they join.
template <int R, int LP>
__device__ __forceinline__ void put_right(PR<LP>& p, const Strip<LP>& s, const int (&v)[R]) {
#pragma unroll
  for (int j = 0; j < R; ++j)
#pragma unroll
    for (int k = 0; k < LP / 2; ++k) p.v[k] = bit_sel(s.mr[j][k], pk_c(v[j]), p.v[k]);
}
template <int R, int LP>
__device__ __forceinline__ void put_right(WR<LP>& p, const Strip<LP>& s, const int (&v)[R]) {
#pragma unroll
  for (int j = 0; j < R; ++j)
#pragma unroll
    for (int k = 0; k < LP; ++k) p.v[k] = s.x0 + k >= s.W + j ? v[j] : p.v[k];
}
template <int MODE, int R, template <int> class ROW, int LP>
__device__ __forceinline__ void fix_right(ROW<LP>& p, const Strip<LP>& s, int c) {
  if constexpr (MODE == B_MIRROR) {
    int v[R];
#pragma unroll
    for (int j = 1; j <= R; ++j) {
      const int r = s.rl * LP + s.rq - (s.W - 1 - mirror_near(s.W - 1 + j, s.W));
      v[j - 1] = strip_px(p, r / LP, r % LP);
    }
    put_right(p, s, v);
  } else {
    const int v[1] = {MODE == B_CONSTANT ? c : strip_px(p, s.rl, s.rq)};
    put_right(p, s, v);
  }
}
// any width
template <int MODE, int R, template <int> class ROW, int LP>
__device__ __forceinline__ void fix_cols_any(ROW<LP>& p, const Strip<LP>& s, int c) {
  if constexpr (R > 0) {
    const int x0 = s.x0;
    int lv[R];
#pragma unroll
    for (int j = 1; j <= R; ++j) {
      const int l = MODE == B_MIRROR ? mirror_near(-j, s.W) : 0;
      lv[j - 1] = MODE == B_CONSTANT ? c : strip_px(p, max(s.zl, 0) + l / LP, l % LP);
    }
    fix_right<MODE, R>(p, s, c);
#pragma unroll
    for (int j = 1; j <= R; ++j) put_where(p, lv[j - 1], [&](int q) { return x0 + q == -j; });
  }
}
// images of at least eight columns
template <int MODE, int R, int LP>
__device__ __forceinline__ void fix_cols(PR<LP>& p, const Strip<LP>& s, int c) {
  if constexpr (R > 0) {
    constexpr int H = LP / 2;
    uint32_t v[R];
#pragma unroll
    for (int j = 1; j <= R; ++j) {  // pixel -j: the high half of pair H - j
      v[j - 1] = pk_c(c);
      if constexpr (MODE == B_MIRROR) {
        v[j - 1] = lane_right(p.v[j % H]);
        if (j < H) v[j - 1] <<= 16;
      } else if constexpr (MODE != B_CONSTANT) {
        v[j - 1] = lane_right(p.v[0]) << 16;
      }
    }
    fix_right<MODE, R>(p, s, c);
#pragma unroll
    for (int j = 1; j <= R; ++j) p.v[H - j] = bit_sel(s.ml, v[j - 1], p.v[H - j]);
  }
}
template <int MODE, int R, int LP>
__device__ __forceinline__ void fix_cols(WR<LP>& p, const Strip<LP>& s, int c) {
  if constexpr (R > 0) {
    int v[R];
#pragma unroll
    for (int j = 1; j <= R; ++j)
      v[j - 1] = MODE == B_CONSTANT ? c : (int)lane_right((uint32_t)p.v[MODE == B_MIRROR ? j : 0]);
    fix_right<MODE, R>(p, s, c);
#pragma unroll
    for (int j = 1; j <= R; ++j) p.v[LP - j] = s.ml ? v[j - 1] : p.v[LP - j];
  }
}

// Row of memory that row r of a group input reads (MODE as above).
template <int MODE>
__device__ __forceinline__ int src_row(int r, int H) {
  if constexpr (MODE == B_MIRROR) r = mirror_pos(r, H);
  return min(max(r, 0), H - 1);
}

// Stores row `row` of a value.  COL: the strip lies at the image's left or
// right edge; of the lane that holds W - 1 amid its pixels the bytes up to it
// are stored, in pieces of 16, 8, 4, 2 and 1 by the bits of their (uniform)
// number.
template <int DF, int LP, bool COL, bool NT, class ROW>
__device__ __forceinline__ void emit_row(const ROW& p, void* base, int64_t pitch, int row, const Strip<LP>& s, uint32_t off) {
  constexpr int BPP = DF == DF_U8 ? 1 : (DF == DF_S16 ? 2 : 4), NB = LP * BPP, AUX = NT ? 2 : 0;
  Raw<NB> x = pack_row<DF, LP>(p);
  const __amdgpu_buffer_rsrc_t r = row_rsrc(base, pitch, row, (uint32_t)(s.W * BPP));
  row_store<NB, AUX>(x, r, off);
  if constexpr (COL) {
    if (!s.whole) {
      const int n = (s.rq + 1) * BPP;
      uint32_t o = s.ragged ? (uint32_t)(s.x0 * BPP) : kNoLane;
      if constexpr (NB > 16) {
        if (n & 16) {
          __builtin_amdgcn_raw_buffer_store_b128(v4w{x.d[0], x.d[1], x.d[2], x.d[3]}, r, o, 0, AUX);
          o += 16;
#pragma unroll
          for (int i = 0; i + 4 < NB / 4; ++i) x.d[i] = x.d[i + 4];
        }
      }
      if constexpr (NB > 8) {
        if (n & 8) {
          __builtin_amdgcn_raw_buffer_store_b64(v2w{x.d[0], x.d[1]}, r, o, 0, AUX);
          o += 8;
#pragma unroll
          for (int i = 0; i + 2 < NB / 4; ++i) x.d[i] = x.d[i + 2];
        }
      }
      if constexpr (NB > 4) {
        if (n & 4) {
          __builtin_amdgcn_raw_buffer_store_b32(x.d[0], r, o, 0, AUX);
          o += 4;
          x.d[0] = x.d[1];
        }
      }
      if constexpr (BPP <= 2) {
        if (n & 2) {
          __builtin_amdgcn_raw_buffer_store_b16((uint16_t)x.d[0], r, o, 0, AUX);
          o += 2;
          x.d[0] >>= 16;
        }
      }
      if constexpr (BPP == 1)
        if (n & 1) __builtin_amdgcn_raw_buffer_store_b8((uint8_t)x.d[0], r, o, 0, AUX);
    }
  }
}

// ---- operators on rows ------------------------------------------------------------------
// Each computes what local_eval / point_eval define, pixel for pixel.
#define HVX_ROW for (int k = 0; k < LP / 2; ++k)

template <int LP>
__device__ __forceinline__ PR<LP> row_channel_y(const PR<LP>& a) {
  PR<LP> r;
#pragma unroll
  HVX_ROW r.v[k] = pk_shr(a.v[k], 8);
  return r;
}
template <int LP>
__device__ __forceinline__ PR<LP> row_gauss3(const PR<LP>& a, const PR<LP>& b, const PR<LP>& c) {
  PR<LP> t, r;
#pragma unroll
  HVX_ROW t.v[k] = pk_mad<2>(b.v[k], pk_add(a.v[k], c.v[k]));
  const PX<LP, 1> e = ext<1>(t);
#pragma unroll
  HVX_ROW r.v[k] = pk_shr(pk_mad<2>(e.v[k + 1], pk_add(e.v[k], e.v[k + 2])), 4);
  return r;
}
__device__ __forceinline__ uint32_t pk_14641(uint32_t a, uint32_t b, uint32_t c, uint32_t d, uint32_t e) {
  return pk_mad<6>(c, pk_mad<4>(pk_add(b, d), pk_add(a, e)));
}
template <int LP>  // sums up to 65280, in unsigned 16-bit halves
__device__ __forceinline__ PR<LP> row_gauss5(const PR<LP>& a, const PR<LP>& b, const PR<LP>& c, const PR<LP>& d,
                                             const PR<LP>& e) {
  PR<LP> t, r;
#pragma unroll
  HVX_ROW t.v[k] = pk_14641(a.v[k], b.v[k], c.v[k], d.v[k], e.v[k]);
  const PX<LP, 2> x = ext<2>(t);
#pragma unroll
  HVX_ROW r.v[k] = pk_shr(pk_14641(x.v[k], x.v[k + 1], x.v[k + 2], x.v[k + 3], x.v[k + 4]), 8);
  return r;
}
template <int LP>  // floor(s / 9) = (7282 s) >> 16 for s <= 2295
__device__ __forceinline__ PR<LP> row_box3(const PR<LP>& a, const PR<LP>& b, const PR<LP>& c) {
  PR<LP> t, r;
#pragma unroll
  HVX_ROW t.v[k] = pk_add(pk_add(a.v[k], b.v[k]), c.v[k]);
  const PX<LP, 1> e = ext<1>(t);
#pragma unroll
  HVX_ROW {
    const uint32_t s = pk_add(pk_add(e.v[k], e.v[k + 1]), e.v[k + 2]);
    r.v[k] = __builtin_amdgcn_perm((s >> 16) * 7282u, (s & 0xFFFFu) * 7282u, 0x07060302u);
  }
  return r;
}
template <bool MAX, int LP>
__device__ __forceinline__ PR<LP> row_rank3(const PR<LP>& a, const PR<LP>& b, const PR<LP>& c) {
  auto f = [](uint32_t x, uint32_t y) { return MAX ? pk_max(x, y) : pk_min(x, y); };
  PR<LP> t, r;
#pragma unroll
  HVX_ROW t.v[k] = f(f(a.v[k], b.v[k]), c.v[k]);
  const PX<LP, 1> e = ext<1>(t);
#pragma unroll
  HVX_ROW r.v[k] = f(f(e.v[k], e.v[k + 1]), e.v[k + 2]);
  return r;
}
__device__ __forceinline__ uint32_t pk_med3(uint32_t a, uint32_t b, uint32_t c) {
  return pk_max(pk_min(a, b), pk_min(pk_max(a, b), c));
}
template <int LP>  // columns sorted, then the largest minimum, the median of medians, the smallest maximum
__device__ __forceinline__ PR<LP> row_median3(const PR<LP>& a, const PR<LP>& b, const PR<LP>& c) {
  PR<LP> lo, md, hi, r;
#pragma unroll
  HVX_ROW {
    const uint32_t mn = pk_min(b.v[k], c.v[k]), mx = pk_max(b.v[k], c.v[k]);
    lo.v[k] = pk_min(a.v[k], mn);
    md.v[k] = pk_min(pk_max(a.v[k], mn), mx);
    hi.v[k] = pk_max(a.v[k], mx);
  }
  const PX<LP, 1> l = ext<1>(lo), m = ext<1>(md), h = ext<1>(hi);
#pragma unroll
  HVX_ROW r.v[k] = pk_med3(pk_max(pk_max(l.v[k], l.v[k + 1]), l.v[k + 2]), pk_med3(m.v[k], m.v[k + 1], m.v[k + 2]),
                           pk_min(pk_min(h.v[k], h.v[k + 1]), h.v[k + 2]));
  return r;
}
template <int LP>
__device__ __forceinline__ PR<LP> row_sobel_x(const PR<LP>& a, const PR<LP>& b, const PR<LP>& c) {
  PR<LP> t, r;
#pragma unroll
  HVX_ROW t.v[k] = pk_mad<2>(b.v[k], pk_add(a.v[k], c.v[k]));
  const PX<LP, 1> e = ext<1>(t);
#pragma unroll
  HVX_ROW r.v[k] = pk_sub(e.v[k + 2], e.v[k]);
  return r;
}
template <int LP>
__device__ __forceinline__ PR<LP> row_sobel_y(const PR<LP>& a, const PR<LP>& c) {
  PR<LP> t, r;
#pragma unroll
  HVX_ROW t.v[k] = pk_sub(c.v[k], a.v[k]);
  const PX<LP, 1> e = ext<1>(t);
#pragma unroll
  HVX_ROW r.v[k] = pk_mad<2>(e.v[k + 1], pk_add(e.v[k], e.v[k + 2]));
  return r;
}
// NonMaxSuppression over a (2 R + 1)^2 window (w: its rows, top to bottom)
template <int R, int DF, int LP>
__device__ __forceinline__ PR<LP> row_nonmax(const PR<LP>* const (&w)[2 * R + 1]) {
  PX<LP, R> m[2];  // the largest of each column above and below the row
  {
    PR<LP> u = *w[0], d = *w[R + 1];
#pragma unroll
    for (int j = 1; j < R; ++j)
#pragma unroll
      HVX_ROW {
        u.v[k] = pk_max(u.v[k], w[j]->v[k]);
        d.v[k] = pk_max(d.v[k], w[R + 1 + j]->v[k]);
      }
    m[0] = ext<R>(u);
    m[1] = ext<R>(d);
  }
  const PX<LP, R> e = ext<R>(*w[R]);
  PR<LP> r;
#pragma unroll
  HVX_ROW {
    uint32_t before = m[0].v[k], after = m[1].v[k];
#pragma unroll
    for (int i = 1; i <= 2 * R; ++i) {
      before = pk_max(before, m[0].v[k + i]);
      after = pk_max(after, m[1].v[k + i]);
    }
#pragma unroll
    for (int i = 1; i <= R; ++i) {
      before = pk_max(before, e.v[R + k - i]);
      after = pk_max(after, e.v[R + k + i]);
    }
    const uint32_t p = e.v[R + k];
    r.v[k] = bit_sel(pk_neg_mask(pk_subs(before, p) & ~pk_subs(p, after)), p, DF == DF_U8 ? 0u : 0x80008000u);
  }
  return r;
}
// Magnitude of gradients up to 32768: the integer root from the hardware's
// square root (its error is far below one half), rounded by the exact
// remainder: with q within one of the root and d = s - q^2, the rounded root
// is q where d <= q and q + 1 where d > q.
__device__ __forceinline__ int magnitude_of(uint32_t s) {
  const uint32_t q = (uint32_t)__builtin_amdgcn_sqrtf((float)s);
  const uint32_t m = q + ((int)(s - __umul24(q, q)) > (int)q ? 1u : 0u);
  return (int)min(m, 32767u);
}
// SMALL: gradients up to 1020 (Sobel of U8): the hardware's root, rounded to
// the nearest integer, is the rounded root of the sum (test_gpu_roots.py
// compares all pairs of gradients).  Adding 2^23 rounds it and leaves the
// integer in the low half, which is all that packing takes: 5 instructions a
// pixel instead of 10.
template <bool SMALL, int LP>
__device__ __forceinline__ PR<LP> row_magnitude(const PR<LP>& a, const PR<LP>& b) {
  const WR<LP> x = wide(a), y = wide(b);
  WR<LP> r;
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    const uint32_t s = (uint32_t)(x.v[q] * x.v[q]) + (uint32_t)(y.v[q] * y.v[q]);
    if constexpr (SMALL) r.v[q] = __float_as_int(__builtin_amdgcn_sqrtf((float)s) + 8388608.f);
    else r.v[q] = magnitude_of(s);
  }
  return packed(r);
}
template <int LP>  // |gradients| <= 1023
__device__ __forceinline__ PR<LP> row_phase(const PR<LP>& a, const PR<LP>& b) {
  PR<LP> r;
#pragma unroll
  HVX_ROW r.v[k] = phase_pair(a.v[k], b.v[k]) & 0x00FF00FFu;
  return r;
}
// exact products of 16-bit gradients.  NZ: a product of zero and a negative
// number is +0 rather than -0 (the sums that read it do not tell them apart)
template <bool NZ, int LP>
__device__ __forceinline__ WR<LP> row_mulf(const PR<LP>& a, const PR<LP>& b) {
#pragma clang fp contract(off)
  const WR<LP> x = wide(a), y = wide(b);
  WR<LP> r;
#pragma unroll
  for (int q = 0; q < LP; ++q)
    r.v[q] = __float_as_int(NZ ? __builtin_fmaf((float)x.v[q], (float)y.v[q], 0.f) : (float)x.v[q] * (float)y.v[q]);
  return r;
}
// Sums of five columns left to right, each addition rounded.  TRI: sums of
// three are exact, so neighbouring pixels share the first two additions.
template <bool NZ, bool TRI, int LP>
__device__ __forceinline__ WR<LP> row_columns5f(const WR<LP>& t) {
#pragma clang fp contract(off)
  const WX<LP, 2> x = ext<2>(t);
  WR<LP> r;
  float p = 0.f;
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    auto at = [&](int i) { return __int_as_float(x.v[q + i]); };
    float s;
    if constexpr (TRI) {
      if (q % 2 == 0) p = at(1) + at(2);  // of pixels q and q + 1
      s = q % 2 == 0 ? at(0) + p : p + at(2);
    } else {
      s = NZ ? at(0) : 0.f + at(0);
      s = s + at(1);
      s = s + at(2);
    }
    s = s + at(3);
    r.v[q] = __float_as_int(s + at(4));
  }
  return r;
}
// F32 Box5x5 in the fixed order of local_eval: each column top to bottom,
// then the columns left to right.  NZ: no element is -0, so the leading
// additions of zero change nothing.
template <bool NZ, int LP>
__device__ __forceinline__ WR<LP> row_box5f(const WR<LP>& a, const WR<LP>& b, const WR<LP>& c, const WR<LP>& d,
                                            const WR<LP>& e) {
#pragma clang fp contract(off)
  WR<LP> t;
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    float s = NZ ? __int_as_float(a.v[q]) : 0.f + __int_as_float(a.v[q]);
    s = s + __int_as_float(b.v[q]);
    s = s + __int_as_float(c.v[q]);
    s = s + __int_as_float(d.v[q]);
    t.v[q] = __float_as_int(s + __int_as_float(e.v[q]));
  }
  return row_columns5f<NZ, false>(t);
}
// Whole numbers as floats, and products of such rows added to or taken from
// sums that stay below 2^24 (exact, so in any order).
template <int LP>
__device__ __forceinline__ WR<LP> floats(const PR<LP>& p) {
  WR<LP> w = wide(p);
#pragma unroll
  for (int q = 0; q < LP; ++q) w.v[q] = __float_as_int((float)w.v[q]);
  return w;
}
template <bool ADD, int LP>
__device__ __forceinline__ void row_fma(WR<LP>& s, const WR<LP>& a, const WR<LP>& b) {
#pragma unroll
  for (int q = 0; q < LP; ++q) {
    const float x = __int_as_float(a.v[q]);
    s.v[q] = __float_as_int(__builtin_fmaf(ADD ? x : -x, __int_as_float(b.v[q]), __int_as_float(s.v[q])));
  }
}
#undef HVX_ROW

// ---- global operators reduced over the strips ---------------------------------------------
// A group of waves keeps one LDS histogram in 16 interleaved copies (at
// most four lanes of a wave share a counter) and each lane its partial sums or
// extremes over its items; the group writes them to its slot at the end.
constexpr int kStreamHistCopies = 16;

// Calls f(element, counted) for the pixels of a row that the lane owns.
template <bool COL, int LP, class F>
__device__ __forceinline__ void own_pixels(const PR<LP>& p, const Strip<LP>& s, F&& f) {
  if (!(s.keep || (COL && s.ragged))) return;
#pragma unroll
  for (int k = 0; k < LP / 2; ++k) {
    f((int)(int16_t)(uint16_t)p.v[k], !COL || s.x0 + k < s.W);
    f((int)p.v[k] >> 16, !COL || s.x0 + k + LP / 2 < s.W);
  }
}
// (value - OFF) * BINS / RANGE for values of [OFF, OFF + RANGE)
template <int BINS, int OFF, int RANGE>
__device__ __forceinline__ void hist_add(uint32_t* mine, int v, bool in) {
  uint32_t b = (uint32_t)v;
  if constexpr (BINS != 256 || OFF != 0 || RANGE != 256) {
    const uint32_t x = (uint32_t)(v - OFF);
    in = in && x < (uint32_t)RANGE;
    b = in ? x * (uint32_t)BINS / (uint32_t)RANGE : 0u;
  }
  atomicAdd(&mine[b * kStreamHistCopies], in ? 1u : 0u);
}
__device__ __forceinline__ void sums_add(RedSlot& q, int v, bool in) {
  const uint32_t x = in ? (uint32_t)v : 0u;
  q.cmn += x;  // 32-bit sums of one band (at most 64 rows of 8 pixels), widened at its end (sums_wrap)
  q.cmx += __umul24(x, x);
}
__device__ __forceinline__ void sums_wrap(RedSlot& q) {
  q.s1 += q.cmn;
  q.s2 += q.cmx;
  q.cmn = q.cmx = 0;
}
__device__ __forceinline__ void minmax_add(RedSlot& q, int v, bool in) {
  q.mn = min(q.mn, in ? v : 2147483647);
  q.mx = max(q.mx, in ? v : -2147483647 - 1);
}
__device__ __forceinline__ void mmcount_add(RedSlot& q, int v, bool in) {
  if (!in) return;
  q.cmn = v < q.mn ? 1u : q.cmn + (v == q.mn ? 1u : 0u);
  q.cmx = v > q.mx ? 1u : q.cmx + (v == q.mx ? 1u : 0u);
  q.mn = min(q.mn, v);
  q.mx = max(q.mx, v);
}
__device__ __forceinline__ RedSlot red_slot() {
  RedSlot q;
  q.mn = 2147483647;
  q.mx = -2147483647 - 1;
  q.cmn = q.cmx = 0;
  q.s1 = q.s2 = 0;
  return q;
}
// Window of wide rows around pixel q, for operators evaluated pixel by pixel.
template <int LP, int RX, int RY>
struct RowsRd {
  const WX<LP, RX> (&w)[2 * RY + 1];
  int q;
  __device__ __forceinline__ int operator()(int dx, int dy) const { return w[RY + dy].v[RX + q + dx]; }
};

}  // namespace hvx
