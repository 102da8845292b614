// The streaming form of a generated kernel: a wave streams a strip of image
// columns down a band of rows, every value of the group in registers.
//
// At step t the newest row of value v is row t + ext(v) (ext: the rows of v
// its consumers still need beyond the outputs), so the outputs' row t is
// complete at the end of the step.  Each value keeps the rows its readers
// reach back to; the loop is unrolled, so advancing them is renaming.  A
// local operator combines its window rows vertically first and fetches the
// neighbouring lanes' pixels of the result only.  The steps before a band's
// first output row run only the operators whose rows are needed.
//
// Against the tile form, nothing passes through LDS and nothing waits for
// other waves, rows above and below are computed once per band instead of
// once per tile, and 16-bit values are held two to a register.  The 16-bit
// arithmetic is used only where every intermediate result provably fits (the
// ranges of all values are tracked below, from the formats and the
// operators); everything else runs in 32 bits, with the same definitions as
// the tile form.  Waves whose strip and band lie inside the image run a body
// without border code.
//
// What bounds it: over batches VALU issue (Tomasi: 176 instructions a row of
// 248 pixels, 32 3840x2160 frames 0.33 ms, all of it issue; in tiles 1.35 ms),
// on single frames the latency of one wave's steps and the launch.  Measured
// a process call, tiles -> streamed: Unsharp 4K 11.9 -> 7.1 us, FChain 4K
// 35.2 -> 15.2, the F32 corner response at 1021x1019 13.7 -> 6.5, Median ->
// Sobel -> Magnitude -> NonMaxSuppression at 1080p 19.4 -> 11.4.
#include <algorithm>
#include <array>
#include <cstdlib>
#include <cstring>

#include "codegen_emit.h"

namespace hvx {
namespace {

constexpr int kUnroll = kStreamUnroll;

struct Val {
  bool wide = false;       // S32 / F32: one register per pixel
  long long lo = 0, hi = 0;  // integer values (border constants of its readers included)
  bool nz = false;         // F32: never -0
  int depth = 1;           // rows held
  int rx = 0, ry = 0;      // largest radius of the local operators reading it
  int mode = -1, c = 0;    // their border rule (-1: no local reader)
  bool flt = false;        // held as floats: read by sliding sums of products only
  bool gone = false;       // a product formed inside its sliding sum
};

struct Term {  // a user kernel's subexpression on pairs
  std::string s;
  long long lo, hi;
  bool lit;
};

bool fits16(long long lo, long long hi) { return lo >= -32768 && hi <= 32767; }

struct Planner {
  const GProg& P;
  uint32_t nt;
  std::string* why;
  Val v[kMaxGVals];
  int E = 0, LP = 8, halo = 0, nred = 0;
  int T = 0;  // rows at the image's end whose steps know the rows below it: E, up to a multiple of kUnroll
  std::array<char, kMaxGOps> slide{};  // per operator: 1 a sliding sum, 2 whose sums of three columns are exact
  Text t;

  Planner(const GProg& p, uint32_t nt_, std::string* w) : P(p), nt(nt_), why(w) {}

  bool no(const char* m) {
    *why = m;
    return false;
  }

  // user kernel k on pairs: an expression of pair index k, or false where a
  // subexpression may leave 16 bits
  template <class LEAF>
  bool pair_expr(const GOp& o, const LEAF& leaf, Term* out) const {
    std::vector<Term> st;
    for (int i = 0; i < o.p0; ++i) {
      const int op = o.code[i] & 0xFF, arg = o.code[i] >> 8;
      Term r{"", 0, 0, false};
      auto pop = [&]() {
        Term x = st.back();
        st.pop_back();
        return x;
      };
      const size_t need = (op == X_IN || op == X_INW || op == X_CONST) ? 0
                          : (op == X_NEG || op == X_ABS || op == X_SQRT) ? 1
                          : (op == X_CLAMP || op == X_SEL)               ? 3
                                                                         : 2;
      if (st.size() < need) return false;
      switch (op) {
        case X_IN:
        case X_INW: r = leaf(op, arg); break;
        case X_CONST: r = {fmt("pk_c(%d)", o.kc[arg]), o.kc[arg], o.kc[arg], true}; break;
        case X_ADD: {
          const Term b = pop(), a = pop();
          r = {"pk_add(" + a.s + ", " + b.s + ")", a.lo + b.lo, a.hi + b.hi, false};
          break;
        }
        case X_SUB: {
          const Term b = pop(), a = pop();
          r = {"pk_sub(" + a.s + ", " + b.s + ")", a.lo - b.hi, a.hi - b.lo, false};
          break;
        }
        case X_MUL: {
          const Term b = pop(), a = pop();
          const long long p[4] = {a.lo * b.lo, a.lo * b.hi, a.hi * b.lo, a.hi * b.hi};
          r = {"pk_mul(" + a.s + ", " + b.s + ")", *std::min_element(p, p + 4), *std::max_element(p, p + 4), false};
          break;
        }
        case X_DIV: {
          const Term b = pop(), a = pop();
          if (!b.lit || b.lo < 1 || (b.lo & (b.lo - 1))) return false;
          int s = 0;
          while ((1LL << s) < b.lo) ++s;
          if (s > 14) return false;
          r = {a.lo >= 0 ? fmt("pk_shr(%s, %d)", a.s.c_str(), s) : fmt("pk_div2(%s, %d)", a.s.c_str(), s), a.lo / b.lo,
               a.hi / b.lo, false};
          break;
        }
        case X_NEG: {
          const Term a = pop();
          r = {"pk_sub(0u, " + a.s + ")", -a.hi, -a.lo, false};
          break;
        }
        case X_MIN:
        case X_MAX: {
          const Term b = pop(), a = pop();
          const bool mx = op == X_MAX;
          r = {(mx ? "pk_max(" : "pk_min(") + a.s + ", " + b.s + ")", mx ? std::max(a.lo, b.lo) : std::min(a.lo, b.lo),
               mx ? std::max(a.hi, b.hi) : std::min(a.hi, b.hi), false};
          break;
        }
        case X_ABS: {
          const Term a = pop();
          r = {"pk_max(" + a.s + ", pk_sub(0u, " + a.s + "))", a.lo >= 0 ? a.lo : (a.hi <= 0 ? -a.hi : 0),
               std::max(std::llabs(a.lo), std::llabs(a.hi)), false};
          break;
        }
        case X_CLAMP: {
          const Term c = pop(), b = pop(), a = pop();
          r = {"pk_min(pk_max(" + a.s + ", " + b.s + "), " + c.s + ")", std::min(std::max(a.lo, b.lo), c.lo),
               std::min(std::max(a.hi, b.hi), c.hi), false};
          break;
        }
        case X_GT: {
          const Term b = pop(), a = pop();
          r = {"pk_gt(" + a.s + ", " + b.s + ")", 0, 1, false};
          break;
        }
        case X_SEL: {
          const Term c = pop(), b = pop(), a = pop();
          r = {"pk_selnz(" + a.s + ", " + b.s + ", " + c.s + ")", std::min(b.lo, c.lo), std::max(b.hi, c.hi), false};
          break;
        }
        default: return false;
      }
      if (!fits16(r.lo, r.hi) || r.s.size() > 600) return false;
      st.push_back(r);
    }
    if (st.size() != 1) return false;
    *out = st[0];
    return true;
  }

  bool plan() {
    const int nv = P.nvals, no_ = P.nops;
    bool any_wide = false, any_local = false;
    std::vector<int> eh(nv, 0);
    for (int k = no_ - 1; k >= 0; --k) {
      const GOp& o = P.ops[k];
      if (o.kind == OP_MMLOCS || o.kind == OP_LUT || o.kind == OP_NONLINEAR)
        return no("holds an operator the streaming form does not cover");
      any_local |= is_local(o.kind);
      nred += is_reduce_op(o.kind) ? 1 : 0;
      for (int i = 0; i < 3; ++i) {
        if (o.in[i] < 0) continue;
        Val& x = v[o.in[i]];
        const int rx = is_local(o.kind) ? o.rx : 0, ry = is_local(o.kind) ? o.ry : 0;
        eh[o.in[i]] = std::max(eh[o.in[i]], eh[o.out] + rx);
        x.depth = std::max(x.depth, P.vals[o.in[i]].ext - P.vals[o.out].ext + ry + 1);
        x.rx = std::max(x.rx, rx);
        x.ry = std::max(x.ry, ry);
      }
      if (is_local(o.kind)) {
        if (o.border == B_REPEAT) return no("a periodic border");
        Val& x = v[o.in[0]];
        const int mode = o.border == B_UNDEFINED ? B_REPLICATE : o.border;
        uint32_t cb = (uint32_t)o.cint;
        if (P.vals[o.in[0]].df == DF_F32) memcpy(&cb, &o.cf, 4);
        const int c = mode == B_CONSTANT ? (int)cb : 0;
        if (x.mode >= 0 && (x.mode != mode || x.c != c)) return no("one value read under several border rules");
        x.mode = mode;
        x.c = c;
      }
    }
    if (!any_local && !nred) return no("no local operator");
    for (int i = 0; i < nv; ++i) {
      const GVal& g = P.vals[i];
      if (g.df == DF_BUF) continue;  // a global operator's result
      if ((g.df == DF_UYVY && !g.input)) return no("a format the streaming form does not cover");
      v[i].wide = g.df == DF_S32 || g.df == DF_F32;
      any_wide |= v[i].wide;
      if (g.store) v[i].depth = std::max(v[i].depth, g.ext + 1);
      E = std::max(E, g.ext);
      v[i].lo = g.df == DF_S16 ? -32768 : 0;
      v[i].hi = g.df == DF_U8 ? 255 : (g.df == DF_UYVY ? 65535 : 32767);
    }
    LP = any_wide ? 4 : 8;
    plan_slides();
    T = stream_tail(E);
    int emax = 0;
    for (int i = 0; i < nv; ++i) emax = std::max(emax, eh[i]);
    halo = (emax + LP - 1) / LP;
    for (int k = 0; k < no_; ++k)
      for (int i = 0; i < 3; ++i)
        if (P.ops[k].in[i] >= 0 && P.vals[P.ops[k].in[i]].df == DF_UYVY && P.ops[k].kind != OP_CHANNEL_Y)
          return no("a UYVY frame read other than for its luma");
    return true;
  }

  // Box sums of products of whole numbers (the structure tensor).  Where the
  // sums of five rows are whole numbers below 2^24, they are exact in any
  // order: each column keeps the sum of the four newest rows' products, adds
  // the new row's and takes the oldest's away, two fused multiply-adds per
  // pixel instead of a product and four additions, and the rings hold the
  // factors (two planes) instead of the products (three).  Tomasi, bound by
  // vector issue: 263 -> 196 instructions a row together with cheaper roots and
  // Threshold's constants as literals, 32 3840x2160 frames 0.47 -> 0.37 ms.
  // The product's border must be one of its factors' borders: their nearest
  // or mirrored pixels, or zero.
  void plan_slides() {
    std::vector<long long> amax(P.nvals, -1);  // |whole numbers| of Sobel gradients
    for (int k = 0; k < P.nops; ++k) {
      const GOp& o = P.ops[k];
      if ((o.kind != OP_SOBEL_X && o.kind != OP_SOBEL_Y) || v[o.in[0]].wide) continue;
      long long lo, hi;
      local_range(o.in[0], &lo, &hi);
      amax[o.out] = std::min(4 * (hi - lo), 32768LL);
    }
    auto readers = [&](int i, int kind) {  // how many, -1: others read it too
      int n = 0;
      for (int k = 0; k < P.nops; ++k)
        for (int j = 0; j < 3; ++j)
          if (P.ops[k].in[j] == i) {
            if (P.ops[k].kind != kind) return -1;
            ++n;
          }
      return P.vals[i].store ? -1 : n;
    };
    auto fits = [&](int k) {  // operator k is such a sum
      if (P.ops[k].kind != OP_BOX5F) return false;
      const int p = P.ops[k].in[0], m = producer(p);
      if (m < 0 || P.ops[m].kind != OP_MULF || readers(p, OP_BOX5F) != 1) return false;
      if (v[p].mode == B_CONSTANT && v[p].c != 0) return false;
      const long long a = amax[P.ops[m].in[0]], b = amax[P.ops[m].in[1]];
      return a > 0 && b > 0 && 5 * a * b <= 1 << 24;
    };
    // a factor is held as floats if all products that read it slide, under one
    // border rule; products are taken out until that holds for all factors
    std::vector<char> ok(P.nops);
    for (int k = 0; k < P.nops; ++k) ok[k] = fits(k);
    for (bool again = true; again;) {
      again = false;
      for (int k = 0; k < P.nops; ++k) {
        if (!ok[k]) continue;
        const int p = P.ops[k].in[0], m = producer(p);
        for (int j = 0; j < 2 && ok[k]; ++j) {
          const int a = P.ops[m].in[j];
          bool all = readers(a, OP_MULF) > 0;
          for (int i = 0; i < P.nops && all; ++i) {
            const GOp& q = P.ops[i];
            if (q.kind != OP_MULF || (q.in[0] != a && q.in[1] != a)) continue;
            const int b = box_of(q.out);
            all = b >= 0 && ok[b] && v[q.out].mode == v[p].mode;
          }
          if (!all) {
            ok[k] = 0;
            again = true;
          }
        }
      }
    }
    for (int k = 0; k < P.nops; ++k) {
      if (!ok[k]) continue;
      const int p = P.ops[k].in[0], m = producer(p);
      const long long big = amax[P.ops[m].in[0]] * amax[P.ops[m].in[1]];
      slide[k] = 15 * big <= 1 << 24 ? 2 : 1;
      v[p].gone = true;
      for (int j = 0; j < 2; ++j) {
        const int i = P.ops[m].in[j];
        Val& a = v[i];
        a.flt = true;
        a.mode = v[p].mode;
        a.c = 0;
        a.rx = a.ry = 2;
        a.depth = std::max(a.depth, P.vals[i].ext - P.vals[P.ops[k].out].ext + 3);
      }
    }
  }
  int producer(int i) const {
    for (int k = 0; k < P.nops; ++k)
      if (P.ops[k].out == i) return k;
    return -1;
  }
  int box_of(int i) const {  // the box filter that reads value i
    for (int k = 0; k < P.nops; ++k)
      if (P.ops[k].in[0] == i && P.ops[k].kind == OP_BOX5F) return k;
    return -1;
  }

  // row n of a sliding sum, operator k
  void emit_slide(int k) {
    const GOp& m = P.ops[producer(P.ops[k].in[0])];
    const int e = P.vals[P.ops[k].out].ext;
    auto add = [&](const char* s, bool plus, int dy) {
      t("        row_fma<%s>(%s, %s, %s);", plus ? "true" : "false", s, row(k, m.in[0], dy).c_str(),
        row(k, m.in[1], dy).c_str());
    };
    t("      WR<%d> cs = {};", LP);
    t("      if constexpr (V == kAny) {");
    for (int dy = -2; dy <= 2; ++dy) add("cs", true, dy);
    t("      } else {");
    // the four rows above the newest: for a band's first row, and where a row
    // above the image was known only now
    if (e > 0) t("        if constexpr (V == kTop ? from_top + %d == 0 : S == %d) {", e, 2 * E - 2 * e);
    else if (v[m.in[0]].mode == B_MIRROR) t("        if (COL && V == kMid && t == 0) {");
    else t("        if constexpr (false) {");
    t("        st.s%d = {};", k);
    const std::string s = fmt("st.s%d", k);
    for (int dy = -2; dy <= 1; ++dy) add(s.c_str(), true, dy);
    t("        }");
    t("        cs = st.s%d;", k);
    add("cs", true, 2);
    t("        st.s%d = cs;", k);
    add(s.c_str(), false, -2);
    t("      }");
    t("      n = row_columns5f<true, %s>(cs);", slide[k] == 2 ? "true" : "false");
  }
  // before the first step of a sliding sum without rows of its own to spare
  void emit_slide_start(int k) {
    const GOp& o = P.ops[k];
    if (P.vals[o.out].ext > 0) return;
    const GOp& m = P.ops[producer(o.in[0])];
    t("  if constexpr (V != kAny && S == %d) {", 2 * E - 1);
    t("    st.s%d = {};", k);
    for (int dy = -1; dy <= 2; ++dy)
      t("    row_fma<true>(st.s%d, %s, %s);", k, row(k, m.in[0], dy).c_str(), row(k, m.in[1], dy).c_str());
    t("  }");
  }

  // element range of a value as its local readers see it
  void local_range(int i, long long* lo, long long* hi) const {
    *lo = v[i].lo;
    *hi = v[i].hi;
    if (v[i].mode == B_CONSTANT && !v[i].wide) {
      *lo = std::min<long long>(*lo, v[i].c);
      *hi = std::max<long long>(*hi, v[i].c);
    }
  }

  // row t + ext(out) + dy of value i, as operator k reads it
  std::string row(int k, int i, int dy) const {
    return fmt("st.r%d[%d]", i, v[i].depth - 1 - (P.vals[i].ext - P.vals[P.ops[k].out].ext - dy));
  }

  // "c[0] e[0] + c[1] e[1] + ..." on pairs, modulo 2^16
  static std::string pair_sum(const std::vector<int>& c, const std::vector<std::string>& e) {
    std::string s;
    // start from a term of weight one, if there is one
    size_t first = 0;
    while (first < c.size() && c[first] != 1) ++first;
    if (first == c.size()) {
      first = 0;
      while (first < c.size() && !c[first]) ++first;
      if (first == c.size()) return "0u";
      s = c[first] == -1 ? "pk_sub(0u, " + e[first] + ")" : fmt("pk_mul(pk_c(%d), ", c[first]) + e[first] + ")";
    } else {
      s = e[first];
    }
    for (size_t i = 0; i < c.size(); ++i) {
      if (i == first || !c[i]) continue;
      if (c[i] == 1) s = "pk_add(" + s + ", " + e[i] + ")";
      else if (c[i] == -1) s = "pk_sub(" + s + ", " + e[i] + ")";
      else s = fmt("pk_mad<%d>(", c[i]) + e[i] + ", " + s + ")";
    }
    return s;
  }

  // Convolve on pairs, if every sum fits 16 bits
  bool emit_convolve_pairs(int k) {
    const GOp& o = P.ops[k];
    const int in = o.in[0], cols = o.p0, rows = o.p1, rx = o.rx, ry = o.ry;
    if (v[in].wide) return false;
    long long lo, hi, smin = 0, smax = 0;
    local_range(in, &lo, &hi);
    for (int i = 0; i < cols * rows; ++i) {
      const long long m = o.mask[i];
      if (m < -32768 || m > 32767) return false;
      smin += std::min(m * lo, m * hi);
      smax += std::max(m * lo, m * hi);
    }
    const bool uns = smin >= 0 && smax <= 65535;  // the sum as an unsigned half
    if (!uns && !fits16(smin, smax)) return false;
    int a[5], b[5];
    const char* PRn = LP == 8 ? "PR<8>" : "PR<4>";
    auto column = [&](const char* name, const std::vector<int>& c) {
      std::vector<std::string> e;
      for (int j = 0; j < rows; ++j) e.push_back(row(k, in, -(j - ry)) + ".v[k]");
      t("      %s %s;", PRn, name);
      t("#pragma unroll");
      t("      for (int k = 0; k < %d; ++k) %s.v[k] = %s;", LP / 2, name, pair_sum(c, e).c_str());
    };
    std::vector<int> hc;
    std::vector<std::string> he;
    if (conv_rank_one(o, a, b)) {
      column("cs", std::vector<int>(a, a + rows));
      t("      const PX<%d, %d> cx = ext<%d>(cs);", LP, rx, rx);
      for (int i = 0; i < cols; ++i) {
        hc.push_back(b[i]);
        he.push_back(fmt("cx.v[k + %d]", rx - (i - rx)));
      }
    } else {
      for (int i = 0; i < cols; ++i) {
        std::vector<int> c;
        bool any = false;
        for (int j = 0; j < rows; ++j) {
          c.push_back(o.mask[j * cols + i]);
          any |= c.back() != 0;
        }
        if (!any) continue;
        const int d = i - rx, r = std::abs(d);
        column(fmt("cs%d", i).c_str(), c);
        t("      const PX<%d, %d> cx%d = ext<%d>(cs%d);", LP, r, i, r, i);
        hc.push_back(1);
        he.push_back(fmt("cx%d.v[k + %d]", i, r - d));
      }
    }
    t("#pragma unroll");
    t("      for (int k = 0; k < %d; ++k) {", LP / 2);
    t("        uint32_t s = %s;", pair_sum(hc, he).c_str());
    long long dlo = smin >= 0 ? smin >> o.p2 : -((-smin) >> o.p2), dhi = smax >= 0 ? smax >> o.p2 : -((-smax) >> o.p2);
    if (o.p2) t(smin >= 0 ? "        s = pk_shr(s, %d);" : "        s = pk_div2(s, %d);", o.p2);
    const bool u8 = P.vals[o.out].df == DF_U8;
    const long long tlo = u8 ? 0 : -32768, thi = u8 ? 255 : 32767;
    if (dhi > thi) t(dhi > 32767 ? "        s = pk_minu(s, pk_c(%lld));" : "        s = pk_min(s, pk_c(%lld));", thi);
    if (dlo < tlo) t("        s = pk_max(s, pk_c(%lld));", tlo);
    t("        n.v[k] = s;");
    t("      }");
    v[o.out].lo = std::max(tlo, std::min(dlo, thi));
    v[o.out].hi = std::min(thi, std::max(dhi, tlo));
    return true;
  }

  // pixel by pixel, in 32 bits, with the tile form's definitions
  void emit_pixels(int k) {
    const GOp& o = P.ops[k];
    const bool pk = !v[o.out].wide;
    if (pk) t("      WR<%d> w;", LP);
    const char* dst = pk ? "w" : "n";
    if (is_local(o.kind)) {
      t("      const WX<%d, %d> win[%d] = {", LP, o.rx, 2 * o.ry + 1);
      for (int j = -o.ry; j <= o.ry; ++j) t("        ext<%d>(wide(%s)),", o.rx, row(k, o.in[0], j).c_str());
      t("      };");
      t("#pragma unroll");
      t("      for (int q = 0; q < %d; ++q) {", LP);
      t("        const RowsRd<%d, %d, %d> rd{win, q};", LP, o.rx, o.ry);
      if (o.kind == OP_EXPR_LOCAL) t("        %s.v[q] = gx_expr%d(rd);", dst, k);
      else t("        %s.v[q] = local_eval<false>(gop%d, %d, rd);", dst, k, P.vals[o.out].df);
      t("      }");
    } else {
      std::string a[3];
      for (int i = 0; i < 3; ++i) {
        a[i] = "0";
        if (o.in[i] < 0) continue;
        t("      const WR<%d> a%d = wide(%s);", LP, i, row(k, o.in[i], 0).c_str());
        a[i] = fmt("a%d.v[q]", i);
      }
      t("#pragma unroll");
      t("      for (int q = 0; q < %d; ++q)", LP);
      if (o.kind == OP_EXPR)
        t("        %s.v[q] = gx_expr%d(%s, %s, %s);", dst, k, a[0].c_str(), a[1].c_str(), a[2].c_str());
      else
        t("        %s.v[q] = point_eval(gop%d, %d, %s, %s, %s, %s);", dst, k, P.vals[o.out].df,
          P.vals[o.in[0]].df == DF_F32 ? "true" : "false", a[0].c_str(), a[1].c_str(), a[2].c_str());
    }
    if (pk) t("      n = packed(w);");
  }

  // the code that computes row n of operator k's output, and its range
  bool emit_op(int k) {
    const GOp& o = P.ops[k];
    const int in = o.in[0], out = o.out, odf = P.vals[out].df;
    const bool ipk = in >= 0 && !v[in].wide, opk = !v[out].wide;
    auto r = [&](int dy) { return row(k, in, dy); };
    auto call3 = [&](const char* f) { t("      n = %s(%s, %s, %s);", f, r(-1).c_str(), r(0).c_str(), r(1).c_str()); };
    long long lo = 0, hi = 0;
    if (ipk) local_range(in, &lo, &hi);
    switch (o.kind) {
      case OP_CHANNEL_Y: t("      n = row_channel_y(%s);", r(0).c_str()); return true;
      case OP_GAUSS3: call3("row_gauss3"); return true;
      case OP_BOX3: call3("row_box3"); return true;
      case OP_DILATE3: call3("row_rank3<true>"); return true;
      case OP_ERODE3: call3("row_rank3<false>"); return true;
      case OP_MEDIAN3: call3("row_median3"); return true;
      case OP_GAUSS5:
        t("      n = row_gauss5(%s, %s, %s, %s, %s);", r(-2).c_str(), r(-1).c_str(), r(0).c_str(), r(1).c_str(),
          r(2).c_str());
        return true;
      case OP_SOBEL_X:
      case OP_SOBEL_Y:
        if (o.kind == OP_SOBEL_X) call3("row_sobel_x");
        else t("      n = row_sobel_y(%s, %s);", r(-1).c_str(), r(1).c_str());
        v[out].lo = -4 * (hi - lo);
        v[out].hi = 4 * (hi - lo);
        return true;
      case OP_NONMAX: {
        const int R = o.p0;
        t("      const PR<%d>* const w[%d] = {", LP, 2 * R + 1);
        for (int j = -R; j <= R; ++j) t("        &%s,", r(j).c_str());
        t("      };");
        t("      n = row_nonmax<%d, %d>(w);", R, odf);
        return true;
      }
      case OP_MAGNITUDE: {
        bool small = true;
        for (int i = 0; i < 2; ++i) small &= v[o.in[i]].lo >= -1020 && v[o.in[i]].hi <= 1020;
        t("      n = row_magnitude<%s>(%s, %s);", small ? "true" : "false", r(0).c_str(), row(k, o.in[1], 0).c_str());
        v[out].lo = 0;
        if (small) v[out].hi = 1443;
        return true;
      }
      case OP_PHASE: {
        bool small = true;
        for (int i = 0; i < 2; ++i) small &= v[o.in[i]].lo >= -1023 && v[o.in[i]].hi <= 1023;
        if (small) t("      n = row_phase(%s, %s);", r(0).c_str(), row(k, o.in[1], 0).c_str());
        else emit_pixels(k);
        return true;
      }
      case OP_THRESHOLD:
        if (!ipk) {
          emit_pixels(k);
        } else {
          t("#pragma unroll");
          t("      for (int k = 0; k < %d; ++k)", LP / 2);
          if (o.p2 > 32767 || o.p2 < -32768)
            t("        n.v[k] = pk_c(%d);", o.p2 > 32767 ? o.p1 : o.p0);
          else
            t("        n.v[k] = bit_sel(pk_neg_mask(pk_subs(%s.v[k], pk_c(%d))), pk_c(%d), pk_c(%d));", r(0).c_str(), o.p2,
              o.p1, o.p0);
        }
        v[out].lo = std::min(o.p0, o.p1);
        v[out].hi = std::max(o.p0, o.p1);
        return true;
      case OP_ADD: {
        const std::string a = r(0) + ".v[k]", b = row(k, o.in[1], 0) + ".v[k]";
        t("#pragma unroll");
        t("      for (int k = 0; k < %d; ++k)", LP / 2);
        if (o.p0 == 0 && odf == DF_U8)
          t("        n.v[k] = pk_max(pk_min(pk_adds(%s, %s), pk_c(255)), 0u);", a.c_str(), b.c_str());
        else if (o.p0 == 0) t("        n.v[k] = pk_adds(%s, %s);", a.c_str(), b.c_str());
        else if (odf == DF_U8) t("        n.v[k] = pk_add(%s, %s) & 0x00FF00FFu;", a.c_str(), b.c_str());
        else t("        n.v[k] = pk_add(%s, %s);", a.c_str(), b.c_str());
        return true;
      }
      case OP_MULF: {
        bool only_box = !P.vals[out].store;
        for (int j = 0; j < P.nops; ++j)
          for (int i = 0; i < 3; ++i)
            if (P.ops[j].in[i] == out) only_box &= P.ops[j].kind == OP_BOX5F;
        v[out].nz = only_box;
        t("      n = row_mulf<%s>(%s, %s);", only_box ? "true" : "false", r(0).c_str(), row(k, o.in[1], 0).c_str());
        return true;
      }
      case OP_BOX5F:
        if (slide[k]) {
          emit_slide(k);
          return true;
        }
        t("      n = row_box5f<%s>(%s, %s, %s, %s, %s);", v[in].nz ? "true" : "false", r(-2).c_str(), r(-1).c_str(),
          r(0).c_str(), r(1).c_str(), r(2).c_str());
        return true;
      case OP_CONVOLVE:
        if (!emit_convolve_pairs(k)) emit_pixels(k);
        return true;
      case OP_EXPR: {
        Term e;
        bool pk = opk && o.p1 == 0;
        for (int i = 0; i < 3; ++i) pk &= o.in[i] < 0 || !v[o.in[i]].wide;
        if (pk && pair_expr(o,
                            [&](int, int arg) {
                              const int i = o.in[arg];
                              return Term{row(k, i, 0) + ".v[k]", v[i].lo, v[i].hi, false};
                            },
                            &e)) {
          store_expr(out, e);
        } else {
          emit_pixels(k);
        }
        return true;
      }
      case OP_EXPR_LOCAL: {
        Term e;
        if (ipk && opk && o.p1 == 0 &&
            pair_expr(o,
                      [&](int op, int arg) {
                        const int dx = op == X_IN ? 0 : arg % 5 - 2, dy = op == X_IN ? 0 : arg / 5 - 2;
                        return Term{fmt("xr%d.v[k + %d]", dy + 2, o.rx + dx), lo, hi, false};
                      },
                      &e)) {
          for (int j = -o.ry; j <= o.ry; ++j)
            t("      const PX<%d, %d> xr%d = ext<%d>(%s);", LP, o.rx, j + 2, o.rx, r(j).c_str());
          store_expr(out, e);
        } else {
          emit_pixels(k);
        }
        return true;
      }
      case OP_HARRIS: emit_pixels(k); return true;
    }
    return no("holds an operator the streaming form does not cover");
  }
  void store_expr(int out, const Term& e) {
    const bool u8 = P.vals[out].df == DF_U8;
    const long long tlo = u8 ? 0 : -32768, thi = u8 ? 255 : 32767;
    std::string s = e.s;
    if (e.hi > thi) s = fmt("pk_min(%s, pk_c(%lld))", s.c_str(), thi);
    if (e.lo < tlo) s = fmt("pk_max(%s, pk_c(%lld))", s.c_str(), tlo);
    t("#pragma unroll");
    t("      for (int k = 0; k < %d; ++k) n.v[k] = %s;", LP / 2, s.c_str());
    v[out].lo = std::max(tlo, std::min(e.lo, thi));
    v[out].hi = std::min(thi, std::max(e.hi, tlo));
  }

  std::string row_type(int i) const { return fmt(v[i].wide || v[i].flt ? "WR<%d>" : "PR<%d>", LP); }
  int raw_bytes(int i) const { return LP * df_bytes(P.vals[i].df); }

  // row n becomes value i's newest
  void emit_push(int i) {
    const int D = v[i].depth;
    if (D > 1) {
      t("#pragma unroll");
      t("      for (int j = 0; j < %d; ++j) st.r%d[j] = st.r%d[j + 1];", D - 1, i, i);
    }
    t("      st.r%d[%d] = n;", i, D - 1);
  }

  // columns of row n outside the image
  void emit_fix(int i) {
    const char* f = "      if constexpr (COL && V == kAny) fix_cols_any<%d, %d>(n, g, (int)0x%08xu);";
    t(f, v[i].mode, v[i].rx, (uint32_t)v[i].c);
    t("      else if constexpr (COL) fix_cols<%d, %d>(n, g, (int)0x%08xu);", v[i].mode, v[i].rx, (uint32_t)v[i].c);
  }

  // the arguments of a step: each input's loaded row, j its number in `name`
  static std::string raw_args(const std::vector<int>& ins, const char* name, int j) {
    std::string a;
    for (int i : ins) a += fmt(", %s%d[%d]", name, i, j);
    return a;
  }
  std::string prologue_args(const std::vector<int>& ins, int s) const {
    std::string a;
    for (int i : ins) {
      const int j = s - (2 * E - 2 * P.vals[i].ext);
      a += j >= 0 ? fmt(", a%d[%d]", i, j) : fmt(", c%d[0]", i);  // not read before step 2 E - 2 ext
    }
    return a;
  }
  void emit_strip_setup(const std::vector<int>& ins, bool col_always) {
    const int nv = P.nvals;
    t("  const Strip<SX_LP> g = make_strip<SX_LP>(strip, %d, %d, W, H);", halo, 64 - 2 * halo);
    t("  const int wr = (W + SX_LP - 1) / SX_LP * SX_LP, xl = min(max(g.x0, 0), wr - SX_LP);");
    t("  uint32_t off[%d];", kMaxIO);
    for (int i = 0; i < nv; ++i)
      if (P.vals[i].store && P.vals[i].df != DF_BUF)
        t("  off[%d] = g.keep ? (uint32_t)(g.x0 * %d) : kNoLane;", P.vals[i].io, df_bytes(P.vals[i].df));
    for (int i : ins) {
      const GVal& gv = P.vals[i];
      const int bpp = df_bytes(gv.df);
      // row r, from the row of memory its border rule gives; rows from `end`
      // on are not needed and not read (an empty descriptor)
      t("  auto ld%d = [&](int r, int end) {", i);
      t("    const uint32_t n = r < end ? (uint32_t)(wr * %d) : 0u;", bpp);
      t(col_always ? "    r = src_row<%d>(r, H);" : "    if constexpr (COL) r = src_row<%d>(r, H);",
        v[i].mode < 0 ? B_REPLICATE : v[i].mode);
      t("    return row_load<%d>(io.ptr[%d], io.pitch[%d], r, n, (uint32_t)(xl * %d));", raw_bytes(i), gv.io, gv.io, bpp);
      t("  };");
    }
    t("  SxState st = {};");
  }

  void emit_items(const std::vector<int>& ins) {
    // One strip of one band: rows [y0, y1), a multiple of kUnroll of them.  COL
    // false: strip and band lie inside the image.  COL true: any strip of an
    // image of at least eight columns; the band at the image's top starts with
    // steps that know the rows above the image, and the last one is the
    // image's last T rows, whose steps know the rows below it, all at compile
    // time.
    t("template <bool COL>");
    t("__device__ __forceinline__ void sx_item(SxRed& red, const IOTable& io, int W, int H, int strip, int y0, int y1,");
    t("                                        bool last, int own) {");
    emit_strip_setup(ins, false);
    t("  const int rows_end = COL && last ? H + %d : y1;", T);
    for (int i : ins) {
      const int e = P.vals[i].ext, nb = raw_bytes(i);
      if (e) {
        t("  Raw<%d> a%d[%d];", nb, i, 2 * e);
        t("#pragma unroll");
        t("  for (int j = 0; j < %d; ++j) a%d[j] = ld%d(y0 - %d + j, rows_end + %d);", 2 * e, i, i, e, e);
      }
      t("  Raw<%d> c%d[%d];", nb, i, kUnroll);
      t("#pragma unroll");
      t("  for (int j = 0; j < %d; ++j) c%d[j] = ld%d(y0 + %d + j, rows_end + %d);", kUnroll, i, i, e, e);
    }
    if (E > 0) {
      t("  if (COL && y0 == 0) {");
      for (int s = 0; s < 2 * E; ++s)
        t("    if constexpr (COL) sx_step<%d, kTop, COL>(st, red, g, io, off, %d, 0, own%s);", s, s - 2 * E,
          prologue_args(ins, s).c_str());
      t("  } else {");
      for (int s = 0; s < 2 * E; ++s)
        t("    sx_step<%d, kMid, COL>(st, red, g, io, off, y0 - %d, 0, own%s);", s, 2 * E - s, prologue_args(ins, s).c_str());
      t("  }");
    }
    t("  for (int t = y0; t < y1; t += %d) {", kUnroll);
    for (int i : ins) {
      t("    Raw<%d> n%d[%d];", raw_bytes(i), i, kUnroll);
      t("#pragma unroll");
      t("    for (int j = 0; j < %d; ++j) n%d[j] = ld%d(t + %d + j, y1 + %d);", kUnroll, i, i, kUnroll + P.vals[i].ext,
        P.vals[i].ext);
    }
    for (int j = 0; j < kUnroll; ++j)
      t("    sx_step<%d, kMid, COL>(st, red, g, io, off, t + %d, 0, own%s);", 2 * E, j, raw_args(ins, "c", j).c_str());
    for (int i : ins) {
      t("#pragma unroll");
      t("    for (int j = 0; j < %d; ++j) c%d[j] = n%d[j];", kUnroll, i, i);
    }
    t("  }");
    if (T > 0) {
      t("  if constexpr (COL) {");
      t("    if (last) {");
      for (int i : ins) {
        if (T <= kUnroll) continue;
        t("      Raw<%d> b%d[%d];", raw_bytes(i), i, T - kUnroll);
        t("#pragma unroll");
        t("      for (int j = 0; j < %d; ++j) b%d[j] = ld%d(H - %d + j, H + %d);", T - kUnroll, i, i,
          T - kUnroll - P.vals[i].ext, T);
      }
      for (int j = 0; j < T; ++j)
        t("      sx_step<%d, kTail, COL>(st, red, g, io, off, H - %d, 0, H%s);", 2 * E + 1 + j, T - j,
          raw_args(ins, j < kUnroll ? "c" : "b", j < kUnroll ? j : j - kUnroll).c_str());
      t("    }");
      t("  }");
    }
    t("}");
    // any size: row by row, every rule decided as it goes
    t("__device__ __forceinline__ void sx_small(SxRed& red, const IOTable& io, int W, int H, int strip, int y0, int y1) {");
    emit_strip_setup(ins, true);
    t("  for (int t = y0 - %d; t < y1; ++t) {", 2 * E);
    std::string a;
    for (int i : ins) {
      t("    const Raw<%d> x%d = ld%d(t + %d, H + %d);", raw_bytes(i), i, i, P.vals[i].ext, 2 * E + 1);
      a += fmt(", x%d", i);
    }
    t("    sx_step<%d, kAny, true>(st, red, g, io, off, t, y0, y1%s);", 2 * E, a.c_str());
    t("  }");
    t("}");
  }

  // the item `item` of the image: its strip and band
  void emit_item() {
    const int out_lanes = 64 - 2 * halo;
    t("  const int strip = item %% strips, band = item / strips;");
    t("  const StreamBand bn = stream_band(bd, band);");
    // inside the image: every pixel of every lane, every row the band reads
    t("  if (bd.whole && strip > 0 && (strip * %d + %d) * SX_LP <= W && band > 0 && !bn.last)", out_lanes,
      out_lanes + halo);
    t("    sx_item<false>(red, io, W, H, strip, bn.y0, bn.y1, false, bn.own);");
    t("  else if (bd.whole)");
    t("    sx_item<true>(red, io, W, H, strip, bn.y0, bn.y1, bn.last, bn.own);");
    t("  else sx_small(red, io, W, H, strip, bn.y0, bn.y1);");
  }

  void emit_geometry(int strip_px) {
    t("  const int strips = (W + %d) / %d;", strip_px - 1, strip_px);
    t("  const StreamBands bd = stream_bands(W, H, rows, %d);", E);
  }

  void emit_entry() {
    t("extern \"C\" __global__ __launch_bounds__(64) void hvx_gen_stream(const IOTable io0, int W0, int H0,");
    t("                                                           const GenBatchImage* __restrict__ imgs, int nimg,");
    t("                                                           uint32_t* __restrict__ ws, int rows) {");
    // every XCD takes a contiguous run of items (block b runs on XCD b mod 8),
    // so that neighbouring strips and bands share an L2
    t("  const int nb = (int)gridDim.x, b = (int)blockIdx.x;");
    t("  const int per = nb / 8, rem = nb %% 8, xcd = b %% 8;");
    t("  int item = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + b / 8;");
    t("  IOTable io;");
    t("  int W, H;");
    t("  if (nimg == 0) {");
    t("    io = io0;");
    t("    W = W0;");
    t("    H = H0;");
    t("  } else {");
    t("    const int i = gx_batch_image(imgs, nimg, item);");
    t("    io = imgs[i].io;");
    t("    W = imgs[i].w;");
    t("    H = imgs[i].h;");
    t("    rows = imgs[i].rows;");
    t("    item -= imgs[i].block0;");
    t("  }");
    const int strip_px = (64 - 2 * halo) * LP;
    emit_geometry(strip_px);
    t("  SxRed red;");
    emit_item();
    t("}");
  }

  // A reducing kernel: a group of eight waves, each going on from item to item
  // (items of one XCD's groups adjoin), then the group's partial results to
  // its slot of `ws`.  3840x2160 Gaussian3x3 -> Histogram + MeanStdDev: 11 us
  // (30 in tiles, whose 2025 groups each cleared, filled and stored a
  // histogram of their 2048 pixels), bound by one wave's latency over its
  // rows and the LDS additions.
  void emit_reducing_entry() {
    constexpr int NT = 64 * kStreamRedWaves;
    t("extern \"C\" __global__ __launch_bounds__(%d) void hvx_gen_stream(const IOTable io, int W, int H,", NT);
    t("                                                           const GenBatchImage* __restrict__ imgs, int nimg,");
    t("                                                           uint32_t* __restrict__ ws, int rows) {");
    t("  __shared__ unsigned long long part[2][%d];", NT / 64);
    t("  SxRed red;");
    int hist = -1, off = 0;
    for (int k = 0; k < P.nops; ++k) {
      if (!is_reduce_op(P.ops[k].kind)) continue;
      t("  red.q%d = red_slot();", k);
      if (P.ops[k].kind == OP_HISTOGRAM || P.ops[k].kind == OP_EQHIST) hist = k;
    }
    if (hist >= 0) {
      t("  __shared__ __attribute__((aligned(16))) uint32_t hist[%d * kStreamHistCopies];", P.ops[hist].p0);
      t("  for (int i = (int)threadIdx.x; i < %d * kStreamHistCopies; i += %d) hist[i] = 0;", P.ops[hist].p0, NT);
      t("  red.hist = hist + (threadIdx.x & (kStreamHistCopies - 1));");
      t("  __syncthreads();");
    }
    t("  const int nb = (int)gridDim.x, b = (int)blockIdx.x;");
    t("  const int per = nb / 8, rem = nb %% 8, xcd = b %% 8;");
    t("  const int vb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + b / 8;");
    const int strip_px = (64 - 2 * halo) * LP;
    emit_geometry(strip_px);
    t("  const int items = strips * bd.n;");
    t("  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));");
    t("  for (int item = vb * %d + wave; item < items; item += nb * %d) {", NT / 64, NT / 64);
    emit_item();
    for (int k = 0; k < P.nops; ++k)
      if (P.ops[k].kind == OP_SUMS) t("  sums_wrap(red.q%d);", k);
    t("  }");
    t("  uint32_t* slot = ws + (size_t)vb * %d;", red_slot_words(P));
    if (hist >= 0) t("  __syncthreads();");
    for (int k = 0; k < P.nops; ++k) {
      const GOp& o = P.ops[k];
      if (!is_reduce_op(o.kind)) continue;
      if (k == hist) {
        t("  for (int b = (int)threadIdx.x; b < %d; b += %d) {", o.p0, NT);
        t("    uint32_t c = 0;");
        t("#pragma unroll");
        t("    for (int j = 0; j < kStreamHistCopies; j += 4) {");
        t("      const uint4 q = *(const uint4*)(hist + b * kStreamHistCopies + ((j + 4 * b) & (kStreamHistCopies - 1)));");
        t("      c += q.x + q.y + q.z + q.w;");
        t("    }");
        t("    slot[%d + b] = c;", off);
        t("  }");
      } else {
        t("  red_store<%d, %d>(red.q%d, part, slot + %d);", o.kind, NT, k, off);
      }
      off += red_block_words(o.kind, o.p0);
    }
    t("}");
  }

  bool emit() {
    const int nv = P.nvals;
    t("namespace hvx {");
    t("constexpr int SX_LP = %d;", LP);
    // the rows each value holds, oldest first
    t("struct SxState {");
    for (int i = 0; i < nv; ++i)
      if (P.vals[i].df != DF_BUF && !v[i].gone) t("  %s r%d[%d];", row_type(i).c_str(), i, v[i].depth);
    for (int k = 0; k < P.nops; ++k)
      if (slide[k]) t("  WR<%d> s%d;  // the four newest rows' products", LP, k);
    t("};");
    // partial results of the global operators over a lane's items
    t("struct SxRed {");
    t("  uint32_t* hist;");
    for (int k = 0; k < P.nops; ++k)
      if (is_reduce_op(P.ops[k].kind)) t("  RedSlot q%d;", k);
    t("};");
    std::string args, in_list;
    std::vector<int> ins;
    for (int i = 0; i < nv; ++i)
      if (P.vals[i].input) {
        ins.push_back(i);
        args += fmt(", const Raw<%d>& x%d", raw_bytes(i), i);
      }
    // Step S of a band (0 .. 2 E - 1 before its first output row, then 2 E);
    // the outputs' row is t.  V says what is known of the rows: kMid, all lie
    // inside the image; kTop, the band starts at row 0 (t = S - 2 E); kTail,
    // step 2 E + 1 + j is the output row H - T + j; kAny, nothing.  COL: the
    // strip lies at the image's left or right edge.  Rows from `own` on are
    // another band's to count.
    t("enum { kMid, kTop, kTail, kAny };");
    t("template <int S, int V, bool COL>");
    t("__device__ __forceinline__ void sx_step(SxState& st, SxRed& red, const Strip<SX_LP>& g, const IOTable& io,");
    t("                                        const uint32_t (&off)[%d], int t, int first, int own%s) {", kMaxIO, args.c_str());
    t("  constexpr int from_top = S - %d, from_end = S - %d;  // t, t - H where they are known", 2 * E, 2 * E + 1 + T);
    for (int i : ins) {
      const GVal& gv = P.vals[i];
      t("  if constexpr (S >= %d) {  // input %d, row t + %d", 2 * E - 2 * gv.ext, i, gv.ext);
      if (v[i].wide) t("      %s n = unpack_wd<SX_LP>(x%d);", row_type(i).c_str(), i);
      else t("      %s n = unpack_pk<%d, SX_LP>(x%d);", row_type(i).c_str(), gv.df, i);
      if (v[i].mode >= 0) emit_fix(i);
      if (v[i].mode == B_CONSTANT) {
        t("      const int r = t + %d;", gv.ext);
        t("      if (V == kTop ? from_top + %d < 0 : V == kTail ? from_end + %d >= 0 : V == kAny && (r < 0 || r >= g.H))",
          gv.ext, gv.ext);
        t("        fill(n, (int)0x%08xu);", (uint32_t)v[i].c);
      }
      emit_push(i);
      t("  }");
    }
    for (int k = 0; k < P.nops; ++k) {
      const int i = P.ops[k].out;
      const GVal& gv = P.vals[i];
      if (is_reduce_op(P.ops[k].kind) || v[i].gone) continue;
      const int D = v[i].depth;
      // rows outside the image that no operator reads are left as they are
      t("  if constexpr (S >= %d) {  // value %d, row t + %d", 2 * E - 2 * gv.ext, i, gv.ext);
      t("    %s n;", row_type(i).c_str());
      t("    const int r = t + %d;", gv.ext);
      t("    constexpr bool above = V == kTop && from_top + %d < 0, below = V == kTail && from_end + %d >= 0;", gv.ext,
        gv.ext);
      t("    if constexpr (above || below) {");
      if (v[i].mode == B_CONSTANT) {
        t("      fill(n, (int)0x%08xu);", (uint32_t)v[i].c);
      } else if (v[i].mode == B_MIRROR) {
        // r - H = 0: two rows back; 1: four
        const int two = std::max(0, D - 2), four = std::max(0, D - 4);
        t("      n = st.r%d[from_end + %d <= 0 ? %d : %d];", i, gv.ext, two, four);
      } else {
        t("      n = st.r%d[%d];", i, D - 1);  // above the image: set when row 0 is known
      }
      t("    } else if (V != kAny || (r >= 0 && r < g.H)) {");
      if (v[i].flt) {
        t("      PR<%d> whole;", LP);
        t("      {");
        t("      PR<%d>& n = whole;", LP);
      }
      if (!emit_op(k)) return false;
      if (v[i].mode >= 0) emit_fix(i);
      if (v[i].flt) {
        t("      }");
        t("      n = floats(whole);");
      }
      t("    } else {");
      if (v[i].mode == B_CONSTANT) {
        t("      fill(n, (int)0x%08xu);", (uint32_t)v[i].c);
      } else if (v[i].mode == B_MIRROR) {
        // 1, 2 or 4 rows back
        t("      const int d = r - mirror_near(r, g.H);");
        t("      n = st.r%d[%d];", i, D - 1);
        if (D >= 2) t("      if (d == 2) n = st.r%d[%d];", i, D - 2);
        if (D >= 4) t("      if (d == 4) n = st.r%d[%d];", i, D - 4);
      } else {
        t("      n = st.r%d[%d];", i, D - 1);
      }
      t("    }");
      emit_push(i);
      if ((v[i].mode == B_MIRROR || v[i].mode == B_REPLICATE) && D > 1) {
        // rows above the image, once the rows they repeat are known
        auto set = [&](const std::string& top, const std::string& any, int back) {
          if (back < D)
            t("    if ((V == kTop && %s) || (V == kAny && %s)) st.r%d[%d] = st.r%d[%d];", top.c_str(), any.c_str(), i,
              D - 1 - back, i, D - 1);
        };
        const std::string tr = fmt("from_top + %d", gv.ext);
        if (v[i].mode == B_REPLICATE) {
          for (int j = 1; j < D; ++j) set(tr + " == 0", "r == 0", j);
        } else {
          // row -1 reads row 1, row -2 row 2 (at the latest in the step of the
          // first output row); images of one or two rows repeat
          auto mirror = [&](int j, int back) {
            set(tr + fmt(" == %d", j), fmt("r == %d", j), back);
            if (gv.ext == j && back < D)
              t("    if (COL && V == kMid && t == 0) st.r%d[%d] = st.r%d[%d];", i, D - 1 - back, i, D - 1);
          };
          if (v[i].ry >= 1) {
            set("false", "r == 0 && g.H == 1", 1);
            mirror(1, 2);
          }
          if (v[i].ry >= 2) {
            set("false", "r == 0 && g.H <= 2", 2);
            mirror(2, 4);
          }
        }
      }
      t("  }");
      if (slide[k]) emit_slide_start(k);
    }
    t("  if (S >= %d && (V != kAny || t >= first)) {", 2 * E);
    for (int i = 0; i < nv; ++i) {
      const GVal& gv = P.vals[i];
      if (!gv.store || gv.df == DF_BUF) continue;
      t("    emit_row<%d, SX_LP, COL, %s>(st.r%d[%d], io.ptr[%d], io.pitch[%d], t, g, off[%d]);", gv.df,
        (nt >> i) & 1 ? "true" : "false", i, v[i].depth - 1 - gv.ext, gv.io, gv.io, gv.io);
    }
    for (int k = 0; k < P.nops; ++k) {
      const GOp& o = P.ops[k];
      if (!is_reduce_op(o.kind)) continue;
      const int in = o.in[0];
      std::string add = o.kind == OP_SUMS     ? fmt("sums_add(red.q%d, v, in)", k)
                        : o.kind == OP_MINMAX ? fmt("minmax_add(red.q%d, v, in)", k)
                        : o.kind == OP_MMCOUNT
                            ? fmt("mmcount_add(red.q%d, v, in)", k)
                            : fmt("hist_add<%d, %d, %d>(red.hist, v, in)", o.p0, o.p1, o.p2);
      t("    if (!COL || t < own) own_pixels<COL>(st.r%d[%d], g, [&](int v, bool in) { %s; });", in, v[in].depth - 1 - P.vals[in].ext,
        add.c_str());
    }
    t("  }");
    t("}");
    emit_items(ins);
    t("}  // namespace hvx");
    if (nred) emit_reducing_entry();
    else emit_entry();
    return true;
  }
};

}  // namespace

bool emit_stream(const GProg& P, uint32_t nt, GenSource* out, std::string* why) {
  Planner p(P, nt, why);
  if (!p.plan()) return false;
  if (!p.emit()) return false;
  out->text = p.t.s;
  out->form = GEN_STREAM;
  out->tw = (64 - 2 * p.halo) * p.LP;
  out->th = kUnroll;
  out->red = p.nred > 0;
  out->lds_words = 0;
  out->ext = p.E;
  return true;
}

}  // namespace hvx
