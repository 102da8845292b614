// Kernels generated for fused groups: source emission, hipRTC compilation,
// a process-wide cache of code objects and their launch.
//
// A group with a local operator is streamed in strips where it can be
// (codegen_stream.cpp); groups of point operators take four pixels of a row
// per thread; the rest, and tuned tiles, are the tile form written here.
//
// A generated tile kernel evaluates the group's operators in stages.  A
// stage is a run of operators that need no barrier between them: each
// thread sweeps the positions of the stage's extent and, at each position,
// evaluates every operator of the stage whose own extent holds it, keeping
// the results in registers.  A value crosses into LDS only when a local
// operator of a later stage reads it at window offsets (or a later stage
// reads it at all); a local operator that reads a value of the current
// stage starts a new stage.  Group inputs that local operators read are
// loaded into LDS with their halo; inputs read only by point operators are
// read from global memory at the pixel itself.  Every window offset, tile
// pitch and LDS offset is a literal, so a read is one LDS access with a
// constant offset.  Tiles whose halo lies inside the image take a body
// without border tests; the others apply each operator's border rule.
#include "codegen_emit.h"

#include <hip/hiprtc.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <numeric>
#include <string>
#include <vector>

#ifndef HVX_ARCH
#define HVX_ARCH "gfx950"
#endif

namespace hvx {

// the device headers the generated source includes, embedded at build time
extern const int kRtcHeaderCount;
extern const char* const kRtcHeaderNames[];
extern const char* const kRtcHeaderTexts[];

bool conv_rank_one(const GOp& o, int a[5], int b[5]) {
  const int cols = o.p0, rows = o.p1;
  int j0 = -1;
  for (int j = 0; j < rows && j0 < 0; ++j)
    for (int i = 0; i < cols; ++i)
      if (o.mask[j * cols + i]) j0 = j;
  if (j0 < 0) return false;
  int g = 0;
  for (int i = 0; i < cols; ++i) g = std::gcd(g, std::abs(o.mask[j0 * cols + i]));
  int i0 = -1;
  for (int i = 0; i < cols; ++i) {
    b[i] = o.mask[j0 * cols + i] / g;
    if (b[i] && i0 < 0) i0 = i;
  }
  for (int j = 0; j < rows; ++j) {
    const int m0 = o.mask[j * cols + i0];
    if (m0 % b[i0]) return false;
    a[j] = m0 / b[i0];
    for (int i = 0; i < cols; ++i)
      if (o.mask[j * cols + i] != a[j] * b[i]) return false;
  }
  return true;
}

namespace {

constexpr int kGenThreads = 256;
constexpr int kGenLdsBytes = 48 * 1024;
constexpr int kMaxDevices = 64;

std::string float_lit(float f) {
  uint32_t u;
  memcpy(&u, &f, 4);
  return fmt("__builtin_bit_cast(float, 0x%08xu)", u);
}

// column-first costs (4 + 2 rx) column sums of the non-zero weights of a
// plus four sums of those of b, against four sums over the mask's non-zeros
bool separable_pays(const GOp& o, const int a[5], const int b[5]) {
  int na = 0, nb = 0, nm = 0;
  for (int j = 0; j < o.p1; ++j) na += a[j] != 0;
  for (int i = 0; i < o.p0; ++i) nb += b[i] != 0;
  for (int k = 0; k < o.p0 * o.p1; ++k) nm += o.mask[k] != 0;
  return na * (4 + 2 * o.rx) + 4 * nb < 4 * nm;
}

// "0u + c * (unsigned)(e) ..." over the non-zero weights: 32-bit wrapping.
// With `i24` every e lies in [-2^23, 2^23): a weight that is not a power of
// two then multiplies through the 24-bit multiplier (exact, full rate) in
// place of the 32-bit one.
std::string weighted_sum(const int* c, const std::vector<std::string>& e, bool i24) {
  std::string s = "0u";
  for (size_t k = 0; k < e.size(); ++k) {
    if (!c[k]) continue;
    const unsigned m = (unsigned)std::abs(c[k]);
    s += c[k] > 0 ? " + " : " - ";
    if (m == 1) s += "(unsigned)(" + e[k] + ")";
    else if (i24 && (m & (m - 1))) s += "(unsigned)__mul24((int)(" + e[k] + fmt("), %u)", m);
    else s += fmt("%uu * (unsigned)(", m) + e[k] + ")";
  }
  return s;
}

// The operator as a constant the device helpers fold over.
void emit_gop(Text& t, int k, const GOp& o) {
  std::string m, c, kc;
  for (int i = 0; i < kMaxMask; ++i) m += fmt("%s%d", i ? ", " : "", o.mask[i]);
  for (int i = 0; i < kMaxExpr; ++i) c += fmt("%s%d", i ? ", " : "", o.code[i]);
  for (int i = 0; i < kMaxExprConst; ++i) kc += fmt("%s%d", i ? ", " : "", o.kc[i]);
  t("__device__ constexpr GOp gop%d = {%d, %d, {%d, %d, %d}, %d, %d, %s, %d, %d, %d, %d, %d, %d, %s, {%s}, {%s}, {%s}};",
    k, o.kind, o.out, o.in[0], o.in[1], o.in[2], o.border, o.cint, float_lit(o.cf).c_str(), o.rx, o.ry, o.p0, o.p1,
    o.p2, o.p3, float_lit(o.pf).c_str(), m.c_str(), c.c_str(), kc.c_str());
}

// What is known of an F32 value when the kernel is written.  Grid: every
// value is a multiple of 2^grid; top: none exceeds 2^top in magnitude.
// Integers lie on grid 0, and rounding a sum or product of numbers on a grid
// leaves it on that grid, so long as nothing falls below the normal range.
constexpr int kNoGrid = -1000, kNoTop = 1000;
struct Known {
  int grid = kNoGrid, top = kNoTop;
  bool nonneg = false;
};

Known known_float(uint32_t bits) {
  Known r;
  float f;
  memcpy(&f, &bits, 4);
  if (!std::isfinite(f)) return r;
  r.nonneg = f >= 0.f;
  r.grid = r.top = 0;
  if (f == 0.f) return r;
  int e;
  const double m = ldexp(fabs(frexp((double)f, &e)), 24);  // an integer of 24 bits
  r.grid = e - 24 + __builtin_ctzll((unsigned long long)m);
  r.top = e;
  return r;
}
// either of two values
Known known_either(const Known& a, const Known& b) {
  return {std::min(a.grid, b.grid), std::max(a.top, b.top), a.nonneg && b.nonneg};
}
Known known_product(const Known& a, const Known& b) {
  Known r;
  if (a.grid != kNoGrid && b.grid != kNoGrid && a.grid + b.grid >= -120) r.grid = a.grid + b.grid;
  if (a.top + b.top <= 126) r.top = a.top + b.top;
  r.nonneg = a.nonneg && b.nonneg;
  return r;
}
Known known_sum(const Known& a, const Known& b) {
  Known r = known_either(a, b);
  r.top = r.top + 1 <= 126 ? r.top + 1 : kNoTop;
  return r;
}

// A user kernel's postfix program as one expression (Section 5.1).  The
// arithmetic follows the interpreter's rules: 32-bit wrapping integer
// arithmetic with the result saturated to the output format, or F32 with
// every operation rounded (no contraction, but for a scaling by 2^-n that is
// exact and so rounds nothing).  `in`: what is known of its inputs; returns
// what is known of its result.
bool emit_expr(Text& t, int k, const GOp& o, bool local, int out_df, const Known in[3], Known* out, std::string* why) {
  const bool fl = o.p1 != 0;
  struct Part {
    std::string s;
    Known is;
    std::string base;  // F32: s is base * scale, exactly
    float scale = 0.f;
  };
  std::vector<Part> st;
  if (o.p0 < 1 || o.p0 > kMaxExpr) {
    *why = "malformed user kernel";
    return false;
  }
  for (int i = 0; i < o.p0; ++i) {
    const int op = o.code[i] & 0xFF, arg = o.code[i] >> 8;
    const size_t need = (op == X_IN || op == X_INW || op == X_CONST) ? 0
                        : (op == X_NEG || op == X_ABS || op == X_SQRT) ? 1
                        : (op == X_CLAMP || op == X_SEL)               ? 3
                                                                       : 2;
    if (st.size() < need || (op == X_CONST && (arg < 0 || arg >= kMaxExprConst)) || (op == X_SQRT && !fl)) {
      *why = "malformed user kernel";
      return false;
    }
    Part q[3];
    for (size_t n = need; n-- > 0; st.pop_back()) q[n] = st.back();
    const std::string &a = q[0].s, &b = q[1].s, &c = q[2].s;
    Part r;
    switch (op) {
      case X_IN:
      case X_INW: {
        std::string v = local ? (op == X_IN ? std::string("rd(0, 0)") : fmt("rd(%d, %d)", arg % 5 - 2, arg / 5 - 2))
                              : fmt("a%d", arg);
        if (fl) v = ((o.p2 >> (op == X_IN ? arg : 0)) & 1) ? "__int_as_float(" + v + ")" : "(float)(" + v + ")";
        r.s = v;
        if (local) r.is = in[0];
        else if (arg >= 0 && arg < 3) r.is = in[arg];
        break;
      }
      case X_CONST:
        r.s = fmt(fl ? "__int_as_float((int)0x%08xu)" : "(int)0x%08xu", (uint32_t)o.kc[arg]);
        if (fl) r.is = known_float((uint32_t)o.kc[arg]);
        break;
      case X_ADD:
      case X_SUB: {
        if (fl) {
          const bool sub = op == X_SUB;
          r.s = "(" + a + (sub ? " - " : " + ") + b + ")";
          if (!q[0].base.empty())
            r.s = fmt("__builtin_fmaf(%af, ", q[0].scale) + q[0].base + (sub ? ", -(" : ", (") + b + "))";
          else if (!q[1].base.empty())
            r.s = fmt("__builtin_fmaf(%af, ", sub ? -q[1].scale : q[1].scale) + q[1].base + ", " + a + ")";
          r.is = known_sum(q[0].is, q[1].is);
          r.is.nonneg &= !sub;
        } else {
          r.s = std::string(op == X_ADD ? "gx_add(" : "gx_sub(") + a + ", " + b + ")";
        }
        break;
      }
      case X_MUL:
      case X_DIV: {
        if (!fl) {
          r.s = std::string(op == X_MUL ? "gx_mul(" : "gx_div(") + a + ", " + b + ")";
          break;
        }
        r.s = "(" + a + (op == X_MUL ? " * " : " / ") + b + ")";
        // a literal power of two on the right
        const int16_t w = o.code[i - 1];
        float d = 0.f;
        int e;
        if ((w & 0xFF) == X_CONST) memcpy(&d, &o.kc[w >> 8], 4);
        const bool pow2 = d > 0.f && std::isfinite(d) && frexp((double)d, &e) == 0.5 && e > -60 && e < 60;
        if (op == X_MUL) {
          r.is = known_product(q[0].is, q[1].is);
          r.is.nonneg |= a == b;
        } else if (pow2) {
          d = 1.f / d;
          uint32_t u;
          memcpy(&u, &d, 4);
          r.is = known_product(q[0].is, known_float(u));
        }
        if (pow2 && d <= 1.f && r.is.grid != kNoGrid) {
          r.base = a;
          r.scale = d;
        }
        break;
      }
      case X_MIN:
      case X_MAX:
        r.s = (op == X_MIN ? (fl ? "fminf(" : "min(") : (fl ? "fmaxf(" : "max(")) + a + ", " + b + ")";
        r.is = known_either(q[0].is, q[1].is);
        if (op == X_MAX) r.is.nonneg = q[0].is.nonneg || q[1].is.nonneg;
        break;
      case X_GT:
        r.s = "((" + a + ") > (" + b + ")" + (fl ? " ? 1.f : 0.f)" : " ? 1 : 0)");
        r.is = {0, 0, true};
        break;
      case X_NEG:
        r.s = fl ? "(-(" + a + "))" : "gx_neg(" + a + ")";
        r.is = q[0].is;
        r.is.nonneg = false;
        break;
      case X_ABS:
        r.s = fl ? "fabsf(" + a + ")" : "gx_abs(" + a + ")";
        r.is = q[0].is;
        r.is.nonneg = true;
        break;
      case X_SQRT: {
        const Known& x = q[0].is;
        const bool bounded = x.nonneg && x.grid >= -96 && x.top <= 126;
        r.s = (bounded ? "sqrt_bounded(" : "__builtin_sqrtf(") + a + ")";
        if (bounded) r.is = {kNoGrid, std::max(x.top, 1), true};
        break;
      }
      case X_CLAMP:
        r.s = fl ? "fminf(fmaxf(" + a + ", " + b + "), " + c + ")" : "min(max(" + a + ", " + b + "), " + c + ")";
        r.is = known_either(q[0].is, known_either(q[1].is, q[2].is));
        break;
      case X_SEL:
        r.s = "((" + a + ") != " + (fl ? "0.f" : "0") + " ? (" + b + ") : (" + c + "))";
        r.is = known_either(q[1].is, q[2].is);
        break;
      default: *why = "malformed user kernel"; return false;
    }
    st.push_back(r);
  }
  if (st.size() != 1) {
    *why = "malformed user kernel";
    return false;
  }
  if (fl) *out = st[0].is;
  if (local) t("template <class RD> __device__ __forceinline__ int gx_expr%d(const RD& rd) {", k);
  else t("__device__ __forceinline__ int gx_expr%d(int a0, int a1, int a2) {", k);
  t("#pragma clang fp contract(off)");
  if (fl) {
    t("  const float r = %s;", st[0].s.c_str());
    t("  return __float_as_int(r);");
  } else {
    t("  const int r = %s;", st[0].s.c_str());
    t(out_df == DF_U8 ? "  return min(max(r, 0), 255);" : "  return min(max(r, -32768), 32767);");
  }
  t("}");
  return true;
}

}  // namespace

void emit_prelude(Text& t, const GProg& P, const char* header, std::string* why, bool* ok) {
  t("namespace __hip_internal {}");
  t("using namespace __hip_internal;");
  t("#include \"%s\"", header);
  t("#include \"gen_abi.h\"");
  t("namespace hvx {");
  t("__device__ __forceinline__ int gx_add(int a, int b) { return (int)((uint32_t)a + (uint32_t)b); }");
  t("__device__ __forceinline__ int gx_sub(int a, int b) { return (int)((uint32_t)a - (uint32_t)b); }");
  t("__device__ __forceinline__ int gx_mul(int a, int b) { return (int)((uint32_t)a * (uint32_t)b); }");
  t("__device__ __forceinline__ int gx_neg(int a) { return (int)(0u - (uint32_t)a); }");
  t("__device__ __forceinline__ int gx_abs(int a) { return a < 0 ? gx_neg(a) : a; }");
  t("__device__ __forceinline__ int gx_div(int x, int y) { return y == 0 ? 0 : (y == -1 ? gx_neg(x) : x / y); }");
  // a value's LDS tile read under an operator's border rule (edge tiles)
  t("template <int BORDER>");
  t("__device__ __forceinline__ int gx_rd(const int32_t* L, int rw, int ey, int ex, int tx0, int ty0, int W, int H,");
  t("                                    int x, int y, int cval) {");
  t("  if (BORDER != B_REPEAT && (x < 0 || y < 0 || x >= W || y >= H)) {");
  t("    if (BORDER == B_CONSTANT) return cval;");
  t("    if (BORDER == B_MIRROR) {");
  t("      x = mirror_pos(x, W);");
  t("      y = mirror_pos(y, H);");
  t("    }");
  t("    x = min(max(x, 0), W - 1);");
  t("    y = min(max(y, 0), H - 1);");
  t("  }");
  t("  return L[(y - ty0 + ey) * rw + (x - tx0 + ex)];");
  t("}");
  // the image of a batch that work-group `blk` belongs to: the last whose
  // first work-group is at or before it (a uniform binary search)
  t("__device__ __forceinline__ int gx_batch_image(const GenBatchImage* imgs, int n, int blk) {");
  t("  int lo = 0, hi = n - 1;");
  t("  while (lo < hi) {");
  t("    const int mid = (lo + hi + 1) >> 1;");
  t("    if (imgs[mid].block0 <= blk) lo = mid;");
  t("    else hi = mid - 1;");
  t("  }");
  t("  return lo;");
  t("}");
  // four elements of a row from x on; zero outside the image (edge tiles)
  t("__device__ __forceinline__ void gx_load4_edge(int df, const void* base, int64_t pitch, int x, int y, int W, int H,");
  t("                                              int v[4]) {");
  t("#pragma unroll");
  t("  for (int q = 0; q < 4; ++q)");
  t("    v[q] = (y >= 0 && y < H && x + q >= 0 && x + q < W) ? gload(df, base, pitch, x + q, y) : 0;");
  t("}");
  // element j of a 16-byte chunk of a row in format DF (int bits)
  t("template <int DF>");
  t("__device__ __forceinline__ int gx_elem(const uint4& d, int j) {");
  t("  const int bpp = DF == DF_U8 ? 1 : ((DF == DF_S16 || DF == DF_UYVY) ? 2 : 4);");
  t("  const int k = j * bpp / 4, sh = (j * bpp % 4) * 8;");
  t("  const uint32_t w = k == 0 ? d.x : (k == 1 ? d.y : (k == 2 ? d.z : d.w));");
  t("  if (DF == DF_U8) return (int)((w >> sh) & 0xFFu);");
  t("  if (DF == DF_S16) return (int)(int16_t)(uint16_t)(w >> sh);");
  t("  if (DF == DF_UYVY) return (int)((w >> sh) & 0xFFFFu);");
  t("  return (int)w;");
  t("}");
  Known known[kMaxGVals];
  for (int i = 0; i < P.nvals; ++i) {
    const int df = P.vals[i].df;
    if (df != DF_F32) known[i] = {0, df == DF_U8 ? 8 : df == DF_S16 ? 15 : 31, df == DF_U8 || df == DF_UYVY};
  }
  for (int k = 0; k < P.nops; ++k) {
    emit_gop(t, k, P.ops[k]);
    const GOp& o = P.ops[k];
    Known in[3], out;
    for (int i = 0; i < 3; ++i)
      if (o.in[i] >= 0) in[i] = known[o.in[i]];
    if (is_local(o.kind) && o.border == B_CONSTANT) {
      uint32_t c;
      const float v = P.vals[o.in[0]].df == DF_F32 ? o.cf : (float)o.cint;
      memcpy(&c, &v, 4);
      in[0] = known_either(in[0], known_float(c));
    }
    if (o.kind == OP_MULF) {
      out = known_product(in[0], in[1]);
      out.nonneg |= o.in[0] == o.in[1];
    }
    if (o.kind == OP_BOX5F) {
      out = in[0];  // the sum of 25
      out.top = in[0].top <= 120 ? in[0].top + 5 : kNoTop;
    }
    if (o.kind == OP_EXPR || o.kind == OP_EXPR_LOCAL)
      if (!emit_expr(t, k, o, o.kind == OP_EXPR_LOCAL, P.vals[o.out].df, in, &out, why)) *ok = false;
    if (o.out >= 0 && P.vals[o.out].df == DF_F32) known[o.out] = out;
  }
  t("}  // namespace hvx");
  t("using namespace hvx;");
}

namespace {

// ---- the point form ----------------------------------------------------------

bool emit_points(const GProg& P, uint32_t stream, GenSource* out, std::string* why) {
  Text t;
  bool ok = true;
  emit_prelude(t, P, "dev_generic.hpp", why, &ok);
  if (!ok) return false;
  t("extern \"C\" __global__ __launch_bounds__(%d) void hvx_gen(const IOTable io0, int W0, int H0,",
    kGenThreads);
  t("                                                           const GenBatchImage* __restrict__ imgs, int nimg,");
  t("                                                           uint32_t* __restrict__ ws) {");
  // one image (the program's size), or one image of a batch of images
  t("  IOTable io;");
  t("  int W, H, blk = (int)blockIdx.x;");
  t("  if (nimg == 0) {");
  t("    io = io0;");
  t("    W = W0;");
  t("    H = H0;");
  t("  } else {");
  t("    const int i = gx_batch_image(imgs, nimg, blk);");
  t("    io = imgs[i].io;");
  t("    W = imgs[i].w;");
  t("    H = imgs[i].h;");
  t("    blk -= imgs[i].block0;");
  t("  }");
  t("  const int bx = (W + 1023) >> 10;");
  t("  const int y = blk / bx;");
  t("  const int x = ((blk - y * bx) * %d + (int)threadIdx.x) * 4;", kGenThreads);
  t("  if (y >= H || x >= W) return;");
  std::vector<int> read(P.nvals, 0);
  for (int k = 0; k < P.nops; ++k)
    for (int i = 0; i < 3; ++i)
      if (P.ops[k].in[i] >= 0) read[P.ops[k].in[i]] = 1;
  for (int v = 0; v < P.nvals; ++v) {
    const GVal& gv = P.vals[v];
    if (!gv.input || !read[v] || gv.df == DF_BUF) continue;
    t("  int v%d[4];", v);
    t("  load4(%d, (const uint8_t*)io.ptr[%d] + (size_t)y * io.pitch[%d], x, W, v%d);", gv.df, gv.io, gv.io, v);
  }
  for (int k = 0; k < P.nops; ++k) {
    const GOp& o = P.ops[k];
    const GVal& ov = P.vals[o.out];
    t("  int v%d[4];", o.out);
    t("#pragma unroll");
    t("  for (int q = 0; q < 4; ++q) {");
    auto in = [&](int i) { return o.in[i] >= 0 && P.vals[o.in[i]].df != DF_BUF ? fmt("v%d[q]", o.in[i]) : std::string("0"); };
    if (o.kind == OP_LUT)
      t("    v%d[q] = ((const uint8_t*)io.ptr[%d])[%d + (v%d[q] & 0xFF)];", o.out, P.vals[o.in[1]].io, 256 * 4, o.in[0]);
    else if (o.kind == OP_EXPR)
      t("    v%d[q] = gx_expr%d(%s, %s, %s);", o.out, k, in(0).c_str(), in(1).c_str(), in(2).c_str());
    else
      t("    v%d[q] = point_eval(gop%d, %d, %s, %s, %s, %s);", o.out, k, ov.df,
        P.vals[o.in[0]].df == DF_F32 ? "true" : "false", in(0).c_str(), in(1).c_str(), in(2).c_str());
    t("  }");
    if (ov.store)
      t("  store4<%s>(%d, (uint8_t*)io.ptr[%d] + (size_t)y * io.pitch[%d], x, W, v%d);",
        (stream >> o.out) & 1 ? "true" : "false", ov.df, ov.io, ov.io, o.out);
  }
  t("}");
  out->text = t.s;
  out->form = GEN_POINTS;
  out->tw = out->th = 0;
  out->red = false;
  out->lds_words = 0;
  return true;
}

// ---- the tile form -----------------------------------------------------------

enum Src { S_REG = 1, S_LDS, S_GLB };

struct Layout {
  int nstages = 0;
  std::vector<int> op_stage;
  std::vector<int> stage_ev, stage_eh;  // vertical / horizontal extent of each stage's sweep
  std::vector<int> def_stage, last_lds, needs_lds, producer, lds_off;
  std::vector<int> eh;  // horizontal extent of each value: a multiple of 4
  std::vector<std::array<int, 3>> src;
  int lds_words = 0;
  // The border rule the local operators reading a value apply to it, as
  // (mode, constant bits).  When every such value has one rule, edge tiles
  // hold each value's positions outside the image resolved by that rule and
  // run the interior code; otherwise they read through each operator's rule.
  std::vector<int> bmode, bconst;
  bool resolved = true;
};

int round4(int x) { return (x + 3) / 4 * 4; }

void plan_stages(const GProg& P, Layout& L) {
  const int nv = P.nvals, no = P.nops;
  L.op_stage.assign(no, 0);
  L.def_stage.assign(nv, -1);
  L.producer.assign(nv, -1);
  L.needs_lds.assign(nv, 0);
  L.last_lds.assign(nv, -2);
  L.src.assign(no, {0, 0, 0});
  int cur = 0;
  for (int k = 0; k < no; ++k) {
    const GOp& o = P.ops[k];
    bool reads_cur = false;
    if (is_local(o.kind))
      for (int i = 0; i < 3; ++i)
        if (o.in[i] >= 0 && L.producer[o.in[i]] >= 0 && L.def_stage[o.in[i]] == cur) reads_cur = true;
    if (reads_cur) ++cur;
    L.op_stage[k] = cur;
    L.producer[o.out] = k;
    L.def_stage[o.out] = cur;
  }
  L.nstages = cur + 1;
  // reads: local operators read LDS; point operators and reductions read
  // registers within a stage, LDS across stages, group inputs where they are
  for (int k = 0; k < no; ++k) {
    const GOp& o = P.ops[k];
    for (int i = 0; i < 3; ++i) {
      const int v = o.in[i];
      if (v < 0 || P.vals[v].df == DF_BUF) continue;
      if (is_local(o.kind)) {
        L.src[k][i] = S_LDS;
        L.needs_lds[v] = 1;
      } else if (L.producer[v] >= 0) {
        L.src[k][i] = L.def_stage[v] == L.op_stage[k] ? S_REG : S_LDS;
        if (L.src[k][i] == S_LDS) L.needs_lds[v] = 1;
      }
    }
  }
  for (int k = 0; k < no; ++k) {
    const GOp& o = P.ops[k];
    for (int i = 0; i < 3; ++i) {
      const int v = o.in[i];
      if (v < 0 || P.vals[v].df == DF_BUF) continue;
      if (L.producer[v] < 0 && !is_local(o.kind)) L.src[k][i] = L.needs_lds[v] ? S_LDS : S_GLB;
      if (L.src[k][i] == S_LDS) L.last_lds[v] = std::max(L.last_lds[v], L.op_stage[k]);
    }
  }
  // Horizontal extents, consumers first: interior tiles evaluate four
  // horizontally adjacent pixels per thread, so every operator runs over a
  // horizontal extent that is a multiple of 4 (the extra columns are
  // computed like any other), and its input must then hold that extent plus
  // the operator's radius, again rounded up to a multiple of 4.
  L.eh.assign(nv, 0);
  for (int k = no - 1; k >= 0; --k) {
    const GOp& o = P.ops[k];
    const int need = (is_global_op(o.kind) ? 0 : L.eh[o.out]) + (is_local(o.kind) ? o.rx : 0);
    for (int i = 0; i < 3; ++i)
      if (o.in[i] >= 0) L.eh[o.in[i]] = std::max(L.eh[o.in[i]], round4(need));
  }
  L.bmode.assign(nv, -1);
  L.bconst.assign(nv, 0);
  for (int k = 0; k < no; ++k) {
    const GOp& o = P.ops[k];
    if (!is_local(o.kind)) continue;
    const int v = o.in[0];
    uint32_t c = (uint32_t)o.cint;  // the border constant as the input's element bits
    if (P.vals[v].df == DF_F32) memcpy(&c, &o.cf, 4);
    const int mode = o.border == B_UNDEFINED ? B_REPLICATE : o.border;
    const int cb = mode == B_CONSTANT ? (int)c : 0;
    if (L.bmode[v] >= 0 && (L.bmode[v] != mode || L.bconst[v] != cb)) L.resolved = false;
    // REPEAT reads periodic copies: only a group input's load provides them
    if (mode == B_REPEAT && L.producer[v] >= 0) L.resolved = false;
    L.bmode[v] = mode;
    L.bconst[v] = cb;
  }
  L.stage_ev.assign(L.nstages, 0);
  L.stage_eh.assign(L.nstages, 0);
  for (int k = 0; k < no; ++k) {
    const GOp& o = P.ops[k];
    if (is_global_op(o.kind)) continue;
    L.stage_ev[L.op_stage[k]] = std::max(L.stage_ev[L.op_stage[k]], P.vals[o.out].ext);
    L.stage_eh[L.op_stage[k]] = std::max(L.stage_eh[L.op_stage[k]], L.eh[o.out]);
  }
}

// LDS geometry of a value kept on chip: rows of `rw` words, image column x
// of the tile at column x - tx0 + co, image row y at row y - ty0 + e (its
// vertical extent).  A group input is loaded in whole 16-byte chunks of its
// rows, so its rows start at a 16-byte boundary of the image row before the
// halo.  Every row width and column offset is a multiple of 4 words.
int input_cols(const GVal& v, int eh) {
  const int bpp = df_bytes(v.df);
  return ((eh * bpp + 15) / 16 * 16) / bpp;
}

void value_geometry(const GProg& P, const Layout& L, int v, int tw, int* rw, int* co) {
  const GVal& gv = P.vals[v];
  *co = gv.input ? input_cols(gv, L.eh[v]) : L.eh[v];
  *rw = tw + 2 * *co;
}

// First-fit LDS blocks; two values share words only if one is last read in
// a stage before the other is written.  Blocks start at 16-byte boundaries.
int place_lds(const GProg& P, Layout& L, int tw, int th) {
  const int nv = P.nvals;
  L.lds_off.assign(nv, -1);
  std::vector<int> order;
  for (int v = 0; v < nv; ++v)
    if (L.needs_lds[v]) order.push_back(v);
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return L.def_stage[a] < L.def_stage[b]; });
  std::vector<std::array<int, 4>> blocks;  // offset, size, first stage, last stage
  int top = 0;
  for (int v : order) {
    int rw, co;
    value_geometry(P, L, v, tw, &rw, &co);
    const int sz = round4(rw * (th + 2 * P.vals[v].ext));
    const int d = L.def_stage[v], l = std::max(L.last_lds[v], d);
    std::vector<std::array<int, 2>> busy;
    for (auto& b : blocks)
      if (!(b[3] < d || l < b[2])) busy.push_back({b[0], b[1]});
    std::sort(busy.begin(), busy.end());
    int pos = 0;
    for (auto& b : busy) {
      if (pos + sz <= b[0]) break;
      pos = std::max(pos, b[0] + b[1]);
    }
    L.lds_off[v] = pos;
    top = std::max(top, pos + sz);
    blocks.push_back({pos, sz, d, l});
  }
  L.lds_words = top;
  return top;
}

// Load group input v into LDS.  Interior tiles read whole 16-byte chunks
// (every chunk holds a byte of the extent, so it lies inside the row's
// pitch, a multiple of 64 bytes): one vector load per chunk, all of a
// thread's loads issued before the first LDS write.  (Loading four elements
// per lane instead, so that the 16-byte LDS writes of consecutive lanes are
// consecutive, measured slower overall.)  Edge tiles read element by element
// inside the image (or the periodic copies under REPEAT).
void emit_load(Text& t, const GProg& P, const Layout& L, int v, int TW, int TH) {
  const GVal& gv = P.vals[v];
  const int e = gv.ext, eh = L.eh[v], bpp = df_bytes(gv.df);
  int rw, co;
  value_geometry(P, L, v, TW, &rw, &co);
  const int rows = TH + 2 * e, epc = 16 / bpp, cpr = rw / epc, nch = cpr * rows;
  const int kc = (nch + kGenThreads - 1) / kGenThreads;
  const int off = L.lds_off[v];
  t("  {  // load value %d: %d rows of %d columns (halo %d rows, %d columns)", v, rows, rw, e, eh);
  t("    const uint8_t* base = (const uint8_t*)io.ptr[%d];", gv.io);
  t("    const int64_t pitch = io.pitch[%d];", gv.io);
  t("    if constexpr (IN) {");
  t("      uint4 d[%d];", kc);
  t("#pragma unroll");
  t("      for (int k = 0; k < %d; ++k) {", kc);
  t("        const int c = (int)threadIdx.x + k * %d;", kGenThreads);
  t("        if (c < %d) {", nch);
  t("          const int row = c / %d, q = c - row * %d;", cpr, cpr);
  t("          d[k] = *(const uint4*)(base + (size_t)(ty0 - %d + row) * pitch + (size_t)(tx0 - %d) * %d + q * 16);", e,
    co, bpp);
  t("        }");
  t("      }");
  t("#pragma unroll");
  t("      for (int k = 0; k < %d; ++k) {", kc);
  t("        const int c = (int)threadIdx.x + k * %d;", kGenThreads);
  t("        if (c < %d) {", nch);
  t("          const int row = c / %d, q = c - row * %d;", cpr, cpr);
  t("          gx_i4* dst = (gx_i4*)(L + %d + row * %d + q * %d);", off, rw, epc);
  t("#pragma unroll");
  t("          for (int j = 0; j < %d; j += 4)", epc);
  t("            dst[j / 4] = gx_i4{gx_elem<%d>(d[k], j), gx_elem<%d>(d[k], j + 1), gx_elem<%d>(d[k], j + 2),", gv.df,
    gv.df, gv.df);
  t("                                   gx_elem<%d>(d[k], j + 3)};", gv.df);
  t("        }");
  t("      }");
  t("    } else {");
  t("      for (int i = (int)threadIdx.x; i < %d; i += %d) {", rw * rows, kGenThreads);
  t("        const int ly = i / %d, lx = i - ly * %d;", rw, rw);
  t("        int x = tx0 - %d + lx, y = ty0 - %d + ly;", co, e);
  t("        if (lx < %d || lx >= %d) continue;  // outside the extent", co - eh, co + TW + eh);
  if (gv.wrap) {
    t("        L[%d + i] = gload(%d, base, pitch, repeat_pos(x, W), repeat_pos(y, H));", off, gv.df);
  } else if (L.resolved) {
    // positions outside the image take the border rule of the operators reading the value
    t("        if (x < 0 || y < 0 || x >= W || y >= H) {");
    if (L.bmode[v] == B_CONSTANT) {
      t("          L[%d + i] = (int)0x%08xu;", off, (uint32_t)L.bconst[v]);
      t("          continue;");
    } else if (L.bmode[v] == B_MIRROR) {
      t("          x = mirror_pos(x, W);");
      t("          y = mirror_pos(y, H);");
    }
    t("          x = min(max(x, 0), W - 1);");
    t("          y = min(max(y, 0), H - 1);");
    t("        }");
    t("        L[%d + i] = gload(%d, base, pitch, x, y);", off, gv.df);
  } else {
    t("        if (x >= 0 && y >= 0 && x < W && y < H) L[%d + i] = gload(%d, base, pitch, x, y);", off, gv.df);
  }
  t("      }");
  t("    }");
  t("  }");
}

// Edge tiles: the positions of value v outside the image, resolved by the
// border rule of the operators reading it from the positions inside (which
// lie in the value's tile: a border rule maps a position to one within the
// value's extent of the image's edge).
void emit_fill(Text& t, const GProg& P, const Layout& L, int v, int TW, int TH) {
  const int e = P.vals[v].ext, eh = L.eh[v];
  int rw, co;
  value_geometry(P, L, v, TW, &rw, &co);
  const int rows = TH + 2 * e, off = L.lds_off[v];
  t("    for (int i = (int)threadIdx.x; i < %d; i += %d) {  // border of value %d", rw * rows, kGenThreads, v);
  t("      const int ly = i / %d, lx = i - ly * %d;", rw, rw);
  t("      int x = tx0 - %d + lx, y = ty0 - %d + ly;", co, e);
  t("      if (lx < %d || lx >= %d || (x >= 0 && y >= 0 && x < W && y < H)) continue;", co - eh, co + TW + eh);
  if (L.bmode[v] == B_CONSTANT) {
    t("      L[%d + i] = (int)0x%08xu;", off, (uint32_t)L.bconst[v]);
  } else {
    if (L.bmode[v] == B_MIRROR) {
      t("      x = mirror_pos(x, W);");
      t("      y = mirror_pos(y, H);");
    }
    t("      x = min(max(x, 0), W - 1);");
    t("      y = min(max(y, 0), H - 1);");
    t("      L[%d + i] = L[%d + (y - ty0 + %d) * %d + (x - tx0 + %d)];", off, off, e, rw, co);
  }
  t("    }");
}

// The sweeps of one stage.  Edge tiles (1 px per thread) skip positions
// outside the image and read windows through each operator's border rule.
// Interior tiles take groups of four horizontally adjacent pixels per
// thread: a local operator's window comes from LDS as 16-byte reads (three
// per window row), LDS values move four words at a time, and outputs are
// stored four pixels at a time.
struct StageEmitter {
  Text& t;
  const GProg& P;
  const Layout& L;
  int TW, TH;
  int* slot;
  uint32_t stream;  // values no later kernel reads: non-temporal stores

  void geometry(int v, int* rw, int* co) const { value_geometry(P, L, v, TW, rw, co); }

  // LDS index of value v at the sweep position (+ constant offsets)
  std::string lds_index(int v, int ES_V, int ES_H, const char* dx, const char* dy) const {
    int rw, co;
    geometry(v, &rw, &co);
    return fmt("%d + (ly + %d + %s) * %d + (lx + %d + %s)", L.lds_off[v], P.vals[v].ext - ES_V, dy, rw, co - ES_H, dx);
  }

  void one_pixel(int s) {
    const int ESV = L.stage_ev[s], ESH = L.stage_eh[s];
    const int RW = TW + 2 * ESH, RH = TH + 2 * ESV;
    bool need_own = false;
    for (int k = 0; k < P.nops; ++k)
      if (L.op_stage[k] == s && (is_reduce_op(P.ops[k].kind) || P.vals[P.ops[k].out].store)) need_own = true;
    t("    for (int i = (int)threadIdx.x; i < %d; i += %d) {", RW * RH, kGenThreads);
    t("      const int ly = i / %d, lx = i - ly * %d;", RW, RW);
    t("      const int x = tx0 - %d + lx, y = ty0 - %d + ly;", ESH, ESV);
    t("      if (x < 0 || y < 0 || x >= W || y >= H) continue;");
    if (need_own) t("      const bool own = lx >= %d && lx < %d && ly >= %d && ly < %d;", ESH, ESH + TW, ESV, ESV + TH);
    for (int k = 0; k < P.nops; ++k) {
      if (L.op_stage[k] != s) continue;
      const GOp& o = P.ops[k];
      auto at = [&](int i) -> std::string {
        const int v = o.in[i];
        if (v < 0 || P.vals[v].df == DF_BUF) return "0";
        switch (L.src[k][i]) {
          case S_REG: return fmt("v%d", v);
          case S_GLB: return fmt("gload(%d, io.ptr[%d], io.pitch[%d], x, y)", P.vals[v].df, P.vals[v].io, P.vals[v].io);
          default: return "L[" + lds_index(v, ESV, ESH, "0", "0") + "]";
        }
      };
      if (is_reduce_op(o.kind)) {
        t("      if (own) red_add(rs, %d, gop%d, %s);", (*slot)++, k, at(0).c_str());
        continue;
      }
      const GVal& ov = P.vals[o.out];
      const int EV = ov.ext, EH = L.eh[o.out];
      t("      int v%d = 0;", o.out);
      t("      if (lx >= %d && lx < %d && ly >= %d && ly < %d) {", ESH - EH, ESH + EH + TW, ESV - EV, ESV + EV + TH);
      if (is_local(o.kind)) {
        const int v = o.in[0];
        int rw, co;
        geometry(v, &rw, &co);
        uint32_t cval = (uint32_t)o.cint;  // the border constant as the input's element bits
        if (P.vals[v].df == DF_F32) memcpy(&cval, &o.cf, 4);
        t("        auto rd = [&](int dx, int dy) -> int {");
        t("          return gx_rd<%d>(L + %d, %d, %d, %d, tx0, ty0, W, H, x + dx, y + dy, (int)0x%08xu);", o.border,
          L.lds_off[v], rw, P.vals[v].ext, co, cval);
        t("        };");
        if (o.kind == OP_EXPR_LOCAL) t("        v%d = gx_expr%d(rd);", o.out, k);
        else t("        v%d = local_eval<%s>(gop%d, %d, rd);", o.out, o.kind == OP_NONLINEAR ? "true" : "false", k, ov.df);
      } else if (o.kind == OP_LUT) {
        t("        v%d = ((const uint8_t*)io.ptr[%d])[%d + (%s & 0xFF)];", o.out, P.vals[o.in[1]].io, 256 * 4,
          at(0).c_str());
      } else if (o.kind == OP_EXPR) {
        t("        v%d = gx_expr%d(%s, %s, %s);", o.out, k, at(0).c_str(), at(1).c_str(), at(2).c_str());
      } else {
        t("        v%d = point_eval(gop%d, %d, %s, %s, %s, %s);", o.out, k, ov.df,
          P.vals[o.in[0]].df == DF_F32 ? "true" : "false", at(0).c_str(), at(1).c_str(), at(2).c_str());
      }
      if (L.needs_lds[o.out]) t("        L[%s] = v%d;", lds_index(o.out, ESV, ESH, "0", "0").c_str(), o.out);
      if (ov.store) t("        if (own) gstore(%d, io.ptr[%d], io.pitch[%d], x, y, v%d);", ov.df, ov.io, ov.io, o.out);
      t("      }");
    }
    t("    }");
  }

  void four_pixels(int s, bool edge) {
    const int ESV = L.stage_ev[s], ESH = L.stage_eh[s];
    const int GR = (TW + 2 * ESH) / 4, RH = TH + 2 * ESV;
    bool need_own = false;
    for (int k = 0; k < P.nops; ++k)
      if (L.op_stage[k] == s && (is_reduce_op(P.ops[k].kind) || P.vals[P.ops[k].out].store)) need_own = true;
    t("    for (int i = (int)threadIdx.x; i < %d; i += %d) {", GR * RH, kGenThreads);
    t("      const int ly = i / %d, lx = (i - ly * %d) * 4;", GR, GR);
    t("      const int x = tx0 - %d + lx, y = ty0 - %d + ly;", ESH, ESV);
    if (need_own) t("      const bool own = lx >= %d && lx < %d && ly >= %d && ly < %d;", ESH, ESH + TW, ESV, ESV + TH);
    for (int k = 0; k < P.nops; ++k) {
      if (L.op_stage[k] != s) continue;
      const GOp& o = P.ops[k];
      // four elements of input i at the position: an array name
      auto at4 = [&](int i) -> std::string {
        const int v = o.in[i];
        if (v < 0 || P.vals[v].df == DF_BUF) return "gx_zero4";
        const std::string n = fmt("a%d_%d", k, i);
        switch (L.src[k][i]) {
          case S_REG: return fmt("v%d", v);
          case S_GLB:
            t("        int %s[4];", n.c_str());
            if (edge)
              t("        gx_load4_edge(%d, io.ptr[%d], io.pitch[%d], x, y, W, H, %s);", P.vals[v].df, P.vals[v].io,
                P.vals[v].io, n.c_str());
            else
              t("        load4(%d, (const uint8_t*)io.ptr[%d] + (size_t)y * io.pitch[%d], x, W, %s);", P.vals[v].df,
                P.vals[v].io, P.vals[v].io, n.c_str());
            return n;
          default: {
            t("        int %s[4];", n.c_str());
            t("        { const gx_i4 q = gx_ld4(L + %s); %s[0] = q.x; %s[1] = q.y; %s[2] = q.z; %s[3] = q.w; }",
              lds_index(v, ESV, ESH, "0", "0").c_str(), n.c_str(), n.c_str(), n.c_str(), n.c_str());
            return n;
          }
        }
      };
      if (is_reduce_op(o.kind)) {
        t(edge ? "      if (own && y < H) {" : "      if (own) {");
        const std::string a = at4(0);
        t("#pragma unroll");
        if (edge)
          t("        for (int q = 0; q < 4; ++q) if (x + q < W) red_add(rs, %d, gop%d, %s[q]);", (*slot)++, k, a.c_str());
        else
          t("        for (int q = 0; q < 4; ++q) red_add(rs, %d, gop%d, %s[q]);", (*slot)++, k, a.c_str());
        t("      }");
        continue;
      }
      const GVal& ov = P.vals[o.out];
      const int EV = ov.ext, EH = L.eh[o.out];
      t("      int v%d[4] = {0, 0, 0, 0};", o.out);
      t("      if (lx >= %d && lx < %d && ly >= %d && ly < %d) {", ESH - EH, ESH + EH + TW, ESV - EV, ESV + EV + TH);
      if (is_local(o.kind)) {
        const int v = o.in[0], R = o.ry;
        int rw, co;
        geometry(v, &rw, &co);
        // window row j: input row y - R + j, columns x - 4 .. x + 7
        t("        int w[%d][12];", 2 * R + 1);
        t("#pragma unroll");
        t("        for (int j = 0; j < %d; ++j) {", 2 * R + 1);
        const std::string dy = fmt("(j - %d)", R);
        t("          const int32_t* r = L + %s;", lds_index(v, ESV, ESH, "-4", dy.c_str()).c_str());
        t("#pragma unroll");
        t("          for (int c = 0; c < 3; ++c) {");
        t("            const gx_i4 q = gx_ld4(r + 4 * c);");
        t("            w[j][4 * c] = q.x; w[j][4 * c + 1] = q.y; w[j][4 * c + 2] = q.z; w[j][4 * c + 3] = q.w;");
        t("          }");
        t("        }");
        int ca[5], cb[5];
        const int vdf = P.vals[v].df;
        if (o.kind == OP_CONVOLVE && (vdf == DF_U8 || vdf == DF_S16) && conv_rank_one(o, ca, cb) &&
            separable_pays(o, ca, cb)) {
          // column sums first (columns x - rx .. x + 3 + rx), shared by the
          // four outputs; the mask is flipped as in the operator's definition
          // (inputs are U8 or S16; a column sum stays within 24 bits when
          // the sum of |a| times the input's largest magnitude does)
          const int rx = o.rx, ry = o.ry;
          long long bound = 0;
          for (int j = 0; j < o.p1; ++j) bound += std::abs(ca[j]);
          bound *= vdf == DF_U8 ? 255 : 32768;
          for (int c = 4 - rx; c <= 7 + rx; ++c) {
            std::vector<std::string> e;
            for (int j = -ry; j <= ry; ++j) e.push_back(fmt("w[%d][%d]", R - j, c));
            t("        const unsigned cs%d = %s;", c, weighted_sum(ca, e, true).c_str());
          }
          for (int q = 0; q < 4; ++q) {
            std::vector<std::string> e;
            for (int i = -rx; i <= rx; ++i) e.push_back(fmt("cs%d", 4 + q - i));
            t("        {");
            t("          const int s = (int)(%s);", weighted_sum(cb, e, bound < (1 << 23)).c_str());
            t("          const int d = s >= 0 ? (s >> %d) : -((-s) >> %d);", o.p2, o.p2);
            t("          v%d[%d] = %s(d);", o.out, q, ov.df == DF_U8 ? "sat_u8" : "sat_s16");
            t("        }");
          }
        } else {
        t("        const int (*wp)[12] = w;");
        t("#pragma unroll");
        t("        for (int q = 0; q < 4; ++q) {");
        if (o.kind == OP_EXPR_LOCAL) {
          t("          v%d[q] = gx_expr%d([&](int dx, int dy) { return wp[%d + dy][4 + q + dx]; });", o.out, k, R);
        } else {
          t("          switch (q) {");
          for (int q = 0; q < 4; ++q)
            t("            case %d: v%d[%d] = local_eval<%s>(gop%d, %d, WinRd<%d, %d>{wp}); break;", q, o.out, q,
              o.kind == OP_NONLINEAR ? "true" : "false", k, ov.df, R, q);
          t("          }");
        }
        t("        }");
        }
      } else if (o.kind == OP_LUT) {
        const std::string a = at4(0);
        t("#pragma unroll");
        t("        for (int q = 0; q < 4; ++q) v%d[q] = ((const uint8_t*)io.ptr[%d])[%d + (%s[q] & 0xFF)];", o.out,
          P.vals[o.in[1]].io, 256 * 4, a.c_str());
      } else {
        const std::string a = at4(0), b = at4(1), c = at4(2);
        t("#pragma unroll");
        if (o.kind == OP_EXPR)
          t("        for (int q = 0; q < 4; ++q) v%d[q] = gx_expr%d(%s[q], %s[q], %s[q]);", o.out, k, a.c_str(), b.c_str(),
            c.c_str());
        else
          t("        for (int q = 0; q < 4; ++q) v%d[q] = point_eval(gop%d, %d, %s, %s[q], %s[q], %s[q]);", o.out, k,
            ov.df, P.vals[o.in[0]].df == DF_F32 ? "true" : "false", a.c_str(), b.c_str(), c.c_str());
      }
      if (L.needs_lds[o.out])
        t("        *(gx_i4*)(L + %s) = gx_i4{v%d[0], v%d[1], v%d[2], v%d[3]};",
          lds_index(o.out, ESV, ESH, "0", "0").c_str(), o.out, o.out, o.out, o.out);
      if (ov.store)
        t("        if (own%s) store4<%s>(%d, (uint8_t*)io.ptr[%d] + (size_t)y * io.pitch[%d], x, W, v%d);",
          edge ? " && y < H" : "", (stream >> o.out) & 1 ? "true" : "false", ov.df, ov.io, ov.io, o.out);
      t("      }");
    }
    t("    }");
  }
};

// the tile form without the prelude
bool emit_tiles(const GProg& P, int tw_req, int th_req, uint32_t stream, GenSource* out, std::string* why) {
  Layout L;
  plan_stages(P, L);
  int nred = 0;
  for (int k = 0; k < P.nops; ++k) nred += is_reduce_op(P.ops[k].kind) ? 1 : 0;
  const bool red = nred > 0;
  const int hist_words = red ? kGenThreads / 64 * kHistWords : 0;  // a histogram per wave
  static const int shapes[][2] = {{128, 16}, {64, 16}, {64, 8}, {32, 8}, {32, 4}, {16, 4}};
  int TW = 0, TH = 0;
  if (tw_req > 0) {
    if (tw_req % 16 == 0 && th_req > 0 && place_lds(P, L, tw_req, th_req) + hist_words <= kGenLdsBytes / 4) {
      TW = tw_req;
      TH = th_req;
    }
  } else {
    for (auto& s : shapes)
      if (place_lds(P, L, s[0], s[1]) + hist_words <= kGenLdsBytes / 4) {
        TW = s[0];
        TH = s[1];
        break;
      }
  }
  if (!TW) {
    *why = "values kept on chip exceed the LDS budget";
    return false;
  }
  // a tile is interior when every position any stage sweeps, and every
  // input column a window reads, lies inside the image
  int ev_max = 0, eh_max = 0;
  for (int v = 0; v < P.nvals; ++v) {
    ev_max = std::max(ev_max, P.vals[v].ext);
    eh_max = std::max(eh_max, L.eh[v]);
  }
  const int LW = std::max(4, L.lds_words + hist_words);

  Text t;
  t("__device__ constexpr int gx_zero4[4] = {0, 0, 0, 0};");
  // LDS is read and written in whole 16-byte units: consecutive lanes then
  // touch consecutive banks.  A read whose components are not all used would
  // be narrowed to single dwords at a 16-byte lane stride, which hit a
  // quarter of the banks; the empty asm keeps the whole vector.
  t("typedef int gx_i4 __attribute__((ext_vector_type(4)));");
  t("__device__ __forceinline__ gx_i4 gx_ld4(const int32_t* p) {");
  t("  const gx_i4 q = *(const gx_i4*)p;");
  t("  asm volatile(\"\" :: \"v\"(q));");
  t("  return q;");
  t("}");
  // one tile: IN = its halo lies inside the image
  t("template <bool IN>");
  t("__device__ __forceinline__ void gen_tile(const IOTable& io, int W, int H, int tx0, int ty0, int32_t* L%s) {",
    red ? ", RedState& rs" : "");
  bool loads = false;
  for (int v = 0; v < P.nvals; ++v)
    if (P.vals[v].input && L.needs_lds[v]) {
      emit_load(t, P, L, v, TW, TH);
      loads = true;
    }
  if (loads) t("  __syncthreads();");
  int slot_in = 0, slot_edge = 0;
  for (int s = 0; s < L.nstages; ++s) {
    t("  // stage %d: extent %d rows, %d columns", s, L.stage_ev[s], L.stage_eh[s]);
    t("  if constexpr (IN) {");
    StageEmitter{t, P, L, TW, TH, &slot_in, stream}.four_pixels(s, false);
    t("  } else {");
    if (L.resolved) {
      StageEmitter{t, P, L, TW, TH, &slot_edge, stream}.four_pixels(s, true);
      // values of this stage that later windows read: their border
      bool fills = false;
      for (int k = 0; k < P.nops; ++k) {
        const int v = P.ops[k].out;
        if (L.op_stage[k] != s || is_global_op(P.ops[k].kind) || L.bmode[v] < 0) continue;
        if (!fills) t("    __syncthreads();");
        fills = true;
        emit_fill(t, P, L, v, TW, TH);
      }
    } else {
      StageEmitter{t, P, L, TW, TH, &slot_edge, stream}.one_pixel(s);
    }
    t("  }");
    if (s + 1 < L.nstages) t("  __syncthreads();");
  }
  t("}");
  t("extern \"C\" __global__ __launch_bounds__(%d) void hvx_gen(const IOTable io0, int W0, int H0,",
    kGenThreads);
  t("                                                           const GenBatchImage* __restrict__ imgs, int nimg,");
  t("                                                           uint32_t* __restrict__ ws) {");
  t("  __shared__ __attribute__((aligned(16))) int32_t L[%d];", LW);
  if (red) {
    t("  RedState rs;");
    t("  red_begin<%d, %d>(rs, (uint32_t*)(L + %d));", kGenThreads, kGenThreads / 64, L.lds_words);
  }
  // Work-groups go to the 8 XCDs in turn (block b to XCD b mod 8), each with
  // its own L2: give every XCD a contiguous run of tiles, so that tiles
  // side by side, whose rows share cache lines, meet in one L2.  A group that
  // reduces takes a contiguous run of tiles of its own.
  t("  const int nb = (int)gridDim.x, b = (int)blockIdx.x;");
  t("  const int per = nb / 8, rem = nb %% 8, xcd = b %% 8;");
  t("  int vb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + b / 8;");
  // one image (the program's size), or one tile of one image of a batch
  t("  IOTable io;");
  t("  int W, H, stride = nb, limit = 1 << 30;");
  t("  if (nimg == 0) {");
  t("    io = io0;");
  t("    W = W0;");
  t("    H = H0;");
  t("  } else {");
  t("    const int i = gx_batch_image(imgs, nimg, vb);");
  t("    io = imgs[i].io;");
  t("    W = imgs[i].w;");
  t("    H = imgs[i].h;");
  t("    vb -= imgs[i].block0;");
  t("    limit = vb + 1;  // one tile per work-group");
  t("  }");
  t("  const int tiles_x = (W + %d) / %d;", TW - 1, TW);
  t("  const int ntiles = min(tiles_x * ((H + %d) / %d), limit);", TH - 1, TH);
  t("  const int slot = vb;  // the group's tile, and its slot of partial results when it reduces");
  t("  for (int tile = vb; tile < ntiles; tile += stride) {");
  t("    const int tx0 = (tile %% tiles_x) * %d, ty0 = (tile / tiles_x) * %d;", TW, TH);
  t("    const bool in = tx0 >= %d && ty0 >= %d && tx0 + %d <= W && ty0 + %d <= H;", eh_max, ev_max, TW + eh_max,
    TH + ev_max);
  t("    if (in) gen_tile<true>(io, W, H, tx0, ty0, L%s);", red ? ", rs" : "");
  t("    else gen_tile<false>(io, W, H, tx0, ty0, L%s);", red ? ", rs" : "");
  t("    __syncthreads();  // the tile's LDS is free for the next tile");
  t("  }");
  if (red) {
    // the operators' partial results (the loop's last barrier has completed
    // the histogram)
    t("  __shared__ unsigned long long part[2][%d];", kGenThreads / 64);
    t("  uint32_t* const res = ws + (size_t)slot * %d;", red_slot_words(P));
    int n = 0, off = 0;
    for (int k = 0; k < P.nops; ++k) {
      const GOp& o = P.ops[k];
      if (!is_reduce_op(o.kind)) continue;
      if (o.kind == OP_HISTOGRAM || o.kind == OP_EQHIST) {
        t("  for (int i = (int)threadIdx.x; i < %d; i += %d) {", o.p0, kGenThreads);
        t("    uint32_t c = 0;");
        t("    for (int h = 0; h < rs.copies; ++h) c += rs.hist0[h * kHistWords + i];");
        t("    res[%d + i] = c;", off);
        t("  }");
      } else {
        t("  red_store<%d, %d>(rs.%s, part, res + %d);", o.kind, kGenThreads, n == 0 ? "a" : "b", off);
      }
      off += red_block_words(o.kind, o.p0);
      ++n;
    }
  }
  t("}");
  out->text = t.s;
  out->form = GEN_TILES;
  out->tw = TW;
  out->th = TH;
  out->red = red;
  out->lds_words = LW;
  return true;
}

}  // namespace

// ---- cache, compilation, launch --------------------------------------------------

struct GenKernel {
  int form = 0, tw = 0, th = 0;
  int ext = 0;
  bool red = false;
  int lds_words = 0;
  std::vector<char> code;
  std::mutex mu;
  hipModule_t mod[kMaxDevices] = {};
  hipFunction_t fn[kMaxDevices] = {};
};

namespace {
std::mutex g_cache_mu;
// never freed: code objects stay loaded until the process ends
std::map<std::string, GenKernel*>* g_cache = new std::map<std::string, GenKernel*>();  // by source text
std::map<std::string, GenKernel*>* g_by_program = new std::map<std::string, GenKernel*>();
// programs whose source the compiler rejected, with its log
std::map<std::string, std::string>* g_rejected = new std::map<std::string, std::string>();
}  // namespace

bool gen_wanted(const GProg& P) {
  if (P.nops != 1) return true;
  const GOp& o = P.ops[0];
  if (is_global_op(o.kind)) return true;
  if (is_point_op(o.kind)) return o.kind == OP_EXPR;
  // the one-operator local kernel reads a Convolve or NonLinearFilter mask
  // at run time; generated, the mask's zeros and products fold away
  const int in_df = P.vals[o.in[0]].df;
  return o.kind == OP_EXPR_LOCAL || o.kind == OP_CONVOLVE || o.kind == OP_NONLINEAR ||
         (in_df != DF_U8 && in_df != DF_F32);
}

// The source of a program's kernel (see gen_kernel).
static bool gen_source(const GProg& P, int tw, int th, uint32_t stream, GenSource* out, std::string* why) {
  bool any_local = false, any_red = false;
  for (int k = 0; k < P.nops; ++k) {
    const int kind = P.ops[k].kind;
    if (kind == OP_MMLOCS) {
      *why = "the location pass runs alone";
      return false;
    }
    any_local |= is_local(kind);
    any_red |= is_reduce_op(kind);
  }
  if (!any_local && !any_red) return emit_points(P, stream, out, why);
  // One source holds the forms the group can take; a kernel is compiled from it
  // with HVX_GEN_TILES or HVX_GEN_STREAM_ONLY defined, which leaves out the
  // other form.
  GenSource strip, tiles;
  std::string no_strip;
  const bool can_stream = emit_stream(P, stream, &strip, &no_strip);
  const bool can_tile = emit_tiles(P, tw, th, stream, &tiles, why);
  if (tw > 0 ? !can_tile : !can_tile && !can_stream) return false;
  Text t;
  bool ok = true;
  emit_prelude(t, P, can_stream ? "dev_stream.hpp" : "dev_generic.hpp", why, &ok);
  if (!ok) return false;
  // The streaming form is the faster one at every size measured, from
  // 320x240 (Tomasi 15.0 against 5.2 us a frame, Unsharp 5.5 against 3.3) to
  // 32 frames of 3840x2160 (1305 against 331 us).  A chosen tile asks for
  // tiles.
  const bool use_stream = can_stream && tw == 0;
  *out = use_stream ? strip : tiles;
  if (can_tile) t.s += can_stream ? "#ifndef HVX_GEN_STREAM_ONLY\n" + tiles.text + "#endif\n" : tiles.text;
  if (can_stream) t.s += can_tile ? "#ifndef HVX_GEN_TILES\n" + strip.text + "#endif\n" : strip.text;
  out->text = t.s;
  return true;
}

// Compile the kernel for `src`, or find it by its text (g_cache_mu is held).
// *rejected: null because the source does not compile.
static GenKernel* gen_compile(const GenSource& src, std::string* why, bool* rejected) {
  *rejected = false;
  const bool stream = src.form == GEN_STREAM;
  const std::string key = (stream ? "stream " : "") + src.text;
  auto it = g_cache->find(key);
  if (it != g_cache->end()) return it->second;
  const char* dir = getenv("HVX_GEN_DUMP");  // the sources, for reading
  if (dir && !g_cache->count(src.text) && !g_cache->count("stream " + src.text)) {
    const std::string path = std::string(dir) + "/hvx_gen_" + std::to_string(g_cache->size()) + ".hip";
    if (FILE* f = fopen(path.c_str(), "w")) {
      fputs(src.text.c_str(), f);
      fclose(f);
    }
  }
  hiprtcProgram prog;
  if (hiprtcCreateProgram(&prog, src.text.c_str(), "hvx_gen.hip", kRtcHeaderCount,
                          const_cast<const char**>(kRtcHeaderTexts),
                          const_cast<const char**>(kRtcHeaderNames)) != HIPRTC_SUCCESS) {
    *why = "hiprtcCreateProgram failed";
    return nullptr;
  }
  const char* opts[] = {"--offload-arch=" HVX_ARCH, "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                        "-packed-fp32-ops", "-w", stream ? "-DHVX_GEN_STREAM_ONLY" : "-DHVX_GEN_TILES"};
  const hiprtcResult r = hiprtcCompileProgram(prog, (int)(sizeof opts / sizeof opts[0]), opts);
  if (r != HIPRTC_SUCCESS) {
    *rejected = r == HIPRTC_ERROR_COMPILATION;
    size_t n = 0;
    hiprtcGetProgramLogSize(prog, &n);
    std::string log(n, '\0');
    if (n) hiprtcGetProgramLog(prog, &log[0]);
    *why = std::string("hipRTC: ") + hiprtcGetErrorString(r) + "\n" + log.substr(0, 4000);
    hiprtcDestroyProgram(&prog);
    return nullptr;
  }
  size_t n = 0;
  hiprtcGetCodeSize(prog, &n);
  GenKernel* k = new GenKernel();
  k->code.resize(n);
  hiprtcGetCode(prog, k->code.data());
  hiprtcDestroyProgram(&prog);
  k->form = src.form;
  k->tw = src.tw;
  k->th = src.th;
  k->ext = src.ext;
  k->red = src.red;
  k->lds_words = src.lds_words;
  (*g_cache)[key] = k;
  return k;
}

const GenKernel* gen_kernel(const GProg& P, int tw, int th, uint32_t stream, std::string* why) {
  // Writing the source takes longer than the rest of a verification, so a
  // kernel is found by the program itself first.
  GProg q;
  memcpy(&q, &P, sizeof q);
  q.w = q.h = q.tiles_x = q.tiles_y = 0;
  std::string key((const char*)&q, sizeof q);
  for (const uint32_t x : {(uint32_t)tw, (uint32_t)th, stream}) key.append((const char*)&x, sizeof x);
  std::lock_guard<std::mutex> l(g_cache_mu);
  auto it = g_by_program->find(key);
  if (it != g_by_program->end()) return it->second;
  auto no = g_rejected->find(key);
  if (no != g_rejected->end()) {
    *why = no->second;
    return nullptr;
  }
  GenSource src;
  if (!gen_source(P, tw, th, stream, &src, why)) return nullptr;
  bool rejected = false;
  GenKernel* k = gen_compile(src, why, &rejected);
  if (k) (*g_by_program)[key] = k;
  else if (rejected) (*g_rejected)[key] = *why;
  return k;
}

void gen_tile(const GenKernel* k, int* tw, int* th) {
  *tw = k->tw;
  *th = k->th;
}

hipError_t gen_load(const GenKernel* kc, int device) {
  GenKernel* k = const_cast<GenKernel*>(kc);
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> l(k->mu);
  if (k->fn[device]) return hipSuccess;
  hipModule_t m = nullptr;
  hipError_t e = hipModuleLoadData(&m, k->code.data());
  if (e != hipSuccess) return e;
  hipFunction_t f = nullptr;
  e = hipModuleGetFunction(&f, m, k->form == GEN_STREAM ? "hvx_gen_stream" : "hvx_gen");
  if (e != hipSuccess) {
    (void)hipModuleUnload(m);
    return e;
  }
  k->mod[device] = m;
  k->fn[device] = f;
  return hipSuccess;
}

// threads of a work-group: a streamed item is one wave's
static unsigned gen_threads(const GenKernel* k) {
  return k->form != GEN_STREAM ? kGenThreads : (k->red ? 64 * kStreamRedWaves : 64);
}

hipError_t gen_launch(const GenKernel* k, int device, const GProg& P, const IOTable& io,
                      int num_cus, hipStream_t s, uint32_t* ws) {
  if (device < 0 || device >= kMaxDevices || !k->fn[device]) return hipErrorInvalidDeviceFunction;
  // One work-group per tile (a persistent grid of as many groups as fit
  // the CUs measured slower: the hardware's own dispatch of short groups
  // overlaps one group's loads with another's arithmetic as well).  A
  // group that reduces writes its partial results to its slot of `ws`.
  int rows = gen_rows(k, P.w, P.h, (long long)gen_strips(k, P.w) * P.h, P.h % 4 == 0, num_cus);
  const long long grid = gen_slots(k, P.w, P.h, num_cus);
  if (grid <= 0) return hipSuccess;
  if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (k->red && !ws) return hipErrorInvalidValue;
  // the size travels in the arguments, not in the program's copy in device
  // memory: one dependent load less before a wave's first rows
  IOTable t = io;
  const GenBatchImage* none = nullptr;
  int w = P.w, h = P.h, zero = 0;
  void* args[] = {(void*)&t, (void*)&w, (void*)&h, (void*)&none, (void*)&zero, (void*)&ws, (void*)&rows};
  return hipModuleLaunchKernel(k->fn[device], (unsigned)grid, 1, 1, gen_threads(k), 1, 1, 0, s, args, nullptr);
}

// Rows of a band where one launch runs strips of the given total height: a
// multiple of `unit`, and at least `least`.
static int band_rows(const GenKernel* k, long long strip_rows, int unit, int least, int num_cus) {
  // Bands of r rows cost strip_rows / r items of r + ext + 3 steps each (the
  // steps before the first output row run part of the operators; 3 stand for
  // an item's start), shared by the SIMDs, plus about one item's latency at
  // the end, a step of a wave alone taking some 2.5 times its issue: the sum
  // is least at r^2 = 0.4 strip_rows (ext + 3) / SIMDs.  Measured: 1080p and
  // smaller frames are fastest at 4 to 8 rows (640x480 Tomasi 5.0 us against
  // 10.9 at 16), one 4K frame at 4 to 20, batches at 8 to 48 (eight 4K frames:
  // Tomasi 91.5 us at 20 rows, 117 at 4, 104 at 64); over five graphs and six
  // launches each the rule takes 15% longer than the best rows at most, 4% in
  // the median.
  const double simds = 4.0 * (num_cus > 0 ? num_cus : 256);
  if (k->red) {
    // the waves of a reducing kernel go on from item to item: whole rounds of
    // the waves that run at once, of short bands
    int best = least;
    double cost = 1e300;
    for (int r = best; r <= 64; r += unit) {
      const double c = ceil((double)strip_rows / r / (4 * simds)) * (r + k->ext + 3);
      if (c < cost) {
        cost = c;
        best = r;
      }
    }
    return best;
  }
  const double r = sqrt(0.4 * (double)strip_rows * (k->ext + 3) / simds);
  return std::min(std::max((int)(r / unit + 0.5) * unit, least), 32);
}

int gen_rows(const GenKernel* k, int w, int h, long long strip_rows, bool whole_heights, int num_cus) {
  if (k->form != GEN_STREAM) return 0;
  // a band of whole iterations holds the rows that its neighbours read and
  // share; one that goes row by row need not
  const int shift = whole_heights ? 0 : k->th - 1;
  const int least = std::max(1, (k->ext + shift + k->th - 1) / k->th) * k->th;
  const int rows = band_rows(k, strip_rows, k->th, least, num_cus);
  return stream_bands(w, h, rows, k->ext).whole ? rows : band_rows(k, strip_rows, 1, 1, num_cus);
}

int gen_strips(const GenKernel* k, int w) { return k->form == GEN_STREAM ? (w + k->tw - 1) / k->tw : 0; }

long long gen_blocks(const GenKernel* k, int w, int h, int rows) {
  if (k->form == GEN_POINTS) return (long long)((w + 1023) >> 10) * h;
  if (k->form == GEN_STREAM) return (long long)gen_strips(k, w) * stream_bands(w, h, rows, k->ext).n;
  return (long long)((w + k->tw - 1) / k->tw) * ((h + k->th - 1) / k->th);
}

long long gen_slots(const GenKernel* k, int w, int h, int num_cus) {
  const long long n = gen_blocks(k, w, h, gen_rows(k, w, h, (long long)gen_strips(k, w) * h, h % 4 == 0, num_cus));
  // a streamed kernel that reduces: groups of eight items' waves, at most two
  // a CU, each going on to further items
  if (k->form != GEN_STREAM || !k->red) return n;
  return std::min((n + kStreamRedWaves - 1) / kStreamRedWaves, 2LL * (num_cus > 0 ? num_cus : 256));
}

bool gen_batchable(const GenKernel* k) { return !k->red; }

hipError_t gen_launch_batch(const GenKernel* k, int device, const GenBatchImage* imgs, int n, long long blocks,
                            hipStream_t s) {
  if (device < 0 || device >= kMaxDevices || !k->fn[device]) return hipErrorInvalidDeviceFunction;
  if (k->red) return hipErrorInvalidValue;
  if (n <= 0 || blocks <= 0) return hipSuccess;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  IOTable t;
  memset(&t, 0, sizeof t);
  uint32_t* ws = nullptr;
  int none = 0, rows = 0;  // each image's own
  void* args[] = {(void*)&t, (void*)&none, (void*)&none, (void*)&imgs, (void*)&n, (void*)&ws, (void*)&rows};
  return hipModuleLaunchKernel(k->fn[device], (unsigned)blocks, 1, 1, gen_threads(k), 1, 1, 0, s, args, nullptr);
}

}  // namespace hvx
