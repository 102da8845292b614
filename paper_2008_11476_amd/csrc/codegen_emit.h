// Source emission shared by the forms of generated kernels (codegen.cpp: tiles
// and points; codegen_stream.cpp: streamed strips).
#pragma once
#include <cstdarg>
#include <cstdio>
#include <string>
#include <vector>

#include "codegen.h"

namespace hvx {

struct GenSource {
  std::string text;
  int form = 0;
  int tw = 0, th = 0;  // output tile (GEN_TILES); columns of a strip, and what a band's rows are a multiple of (GEN_STREAM)
  int ext = 0;         // rows a band reads beyond its own, on each side (GEN_STREAM)
  bool red = false;    // reduces global operators over the image
  int lds_words = 0;   // static LDS of one work-group
};

inline std::string vfmt(const char* f, va_list ap) {
  va_list again;
  va_copy(again, ap);
  const int n = vsnprintf(nullptr, 0, f, again);
  va_end(again);
  std::string s(n > 0 ? n : 0, '\0');
  if (n > 0) vsnprintf(&s[0], (size_t)n + 1, f, ap);
  return s;
}
inline std::string fmt(const char* f, ...) __attribute__((format(printf, 1, 2)));
inline std::string fmt(const char* f, ...) {
  va_list ap;
  va_start(ap, f);
  std::string s = vfmt(f, ap);
  va_end(ap);
  return s;
}

struct Text {
  std::string s;
  void operator()(const char* f, ...) __attribute__((format(printf, 2, 3))) {
    va_list ap;
    va_start(ap, f);
    s += vfmt(f, ap);
    va_end(ap);
    s += '\n';
  }
};

// an operator that reads its input at window offsets
inline bool is_local(int kind) { return !is_point_op(kind) && !is_global_op(kind); }

// A Convolve mask that is the outer product of a column and a row of
// integers, m[j][i] = a[j] b[i], as those two factors (b divided by the gcd
// of its entries; every integer factorisation is a multiple of that one).
// Summing each window column with the weights a and then the column sums
// with the weights b gives the same 32-bit wrapped sum as the mask itself,
// since the two double sums are equal as integers.
bool conv_rank_one(const GOp& o, int a[5], int b[5]);

// Includes, user kernels as functions (gx_expr<k>) and each operator as a
// constant (gop<k>); `header` is the device header the form needs.
void emit_prelude(Text& t, const GProg& P, const char* header, std::string* why, bool* ok);

// The streaming form of program P without the prelude (codegen_stream.cpp);
// false, with the reason, for a program it does not cover.
bool emit_stream(const GProg& P, uint32_t nt, GenSource* out, std::string* why);

}  // namespace hvx
