// Both stages of a request with their projections inside, for the calls that are held to fp32 (fp32 storage, and bf16 shapes
// outside the bf16 matrix-core set): the m links over a history, and rows over the m links.  A workgroup takes one head of one
// user (of several, where users are many and their rows few); projected queries, keys and values never exist in memory, and a
// request is two launches (three with a history of more than kChunkKeys items) where projections and attentions as kernels of
// their own (generic.hip) are four.
//
// fp32 products on the bf16 matrix instruction.  An fp32 number is the sum of three bf16 numbers, x = x0 + x1 + x2 (each the
// remainder rounded to nearest: at most 2^-8 and 2^-17 of x), and a product is taken as x0 y0 + x0 y1 + x1 y0 + x1 y1 +
// x0 y2 + x2 y0 with fp32 sums: what is left out is 2^-27 of |x y| in the root mean square and 2^-24 at most, of either sign.
// Six instructions of 32 cycles for 16 terms, against eight of 64 for the fp32 instruction (v_mfma_f32_32x32x2_f32), and fewer
// roundings of the accumulator: six per 16 terms instead of eight.  bf16 inputs are one plane, their products one instruction.
// The sum of the planes is exact where none of them lies under the smallest bf16 number (2^-133), as the third one of a number
// below 2^-110 would.  So with fp32 storage whatever is split is taken 2^24 times as large (kUp), or 2^48 times as sums of two such
// come, and is exact down to the smallest number; the units of sums (kSum, kUnit) are taken out where it costs least.  (About 100 of the
// kernels' some 1200 vector instructions a tile at d = 128: 16 users of 777 items and 1001 candidates 32.1 -> 33.0 us, the smallest
// request 15.3 -> 15.6.)  With bf16 storage everything is taken as it is: what results are rounded to, nine bits, is held from 2^-124 on.
// Where an operand is infinite, or rounds to infinity (fp32: from 2^104 on, being 2^24 times as large), its remainders are NaN; a
// sum may pass the range too (fp32: from 2^79 on, a logit or result from 2^55 on).  A result that is not finite is computed again
// with the fp32 instruction (`exact`) and taken from there, so that infinities stay where they are and no other row's bits change.
// The bf16 matrix instruction rounds downward a little more often than upward (the mean of its result and that of its negated operands
// is -1.2e-8 where accumulator and products are near one; the fp32 instruction's is zero), which over many items adds up: the mean
// of 4096 items' values was 6.9e-7 off, 3.6e-7 with the fp32 instruction.  So every other item of a history is taken negated, row
// and weight, and every other tile's result.  (fp32 storage only; bf16 results are rounded to 2^-9.)
//
// Fragments as in mfma.hpp.  A head narrower than 32 columns has its columns repeated over the 32 lanes of a weight fragment,
// which makes room for the planes: at d/h = 8 a lane's slots of one key fragment hold two planes, and the 32 rows of a value
// fragment three; at d/h = 16 its rows hold two.
#pragma once

#include <algorithm>
#include <type_traits>

#include "fused_grid.hpp"
#include "mfma.hpp"

namespace lime {
namespace {

__device__ __forceinline__ f32x16 zeros() {
  f32x16 x;
#pragma unroll
  for (int i = 0; i < 16; ++i) x[i] = 0.f;
  return x;
}
__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0); }

template <typename T>
constexpr int kPlanes = sizeof(T) == 4 ? 3 : 1;

// Eight numbers of a lane as planes.
template <int NP>
struct Planes {
  bf16x8 p[NP];
};
// Two numbers rounded to a register of two bf16 numbers, and the remainders.
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ unsigned rounded_pair(float a, float b) {
  bf16x2 p;
  p[0] = static_cast<__bf16>(a), p[1] = static_cast<__bf16>(b);
  return __builtin_bit_cast(unsigned, p);
}
__device__ __forceinline__ unsigned take_pair(float& a, float& b) {
  unsigned p = rounded_pair(a, b);
  asm("" : "+v"(p));  // (one conversion of the pair: the compiler would convert each number once more for its remainder)
  a -= __uint_as_float(p << 16), b -= __uint_as_float(p & 0xffff0000u);
  return p;
}
// How much larger what is split is; what a projection's sum, of rows and weights so much larger, stands for is kSum of it, what a
// product of such sums with other numbers so much larger stands for is kUnit of it.
template <typename T>
constexpr float kUp = sizeof(T) == 4 ? 0x1p24f : 1.f;
template <typename T>
constexpr float kDown = 1.f / kUp<T>;
template <typename T>
constexpr float kSum = kDown<T> * kDown<T>;
template <typename T>
constexpr float kUnit = kSum<T> * kDown<T>;
__device__ __forceinline__ Planes<3> split(const float (&x)[8]) {
  u32x4 p[3];
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    float a = x[2 * t], b = x[2 * t + 1];
    p[0][t] = take_pair(a, b);
    p[1][t] = take_pair(a, b);
    p[2][t] = rounded_pair(a, b);
  }
  return {{__builtin_bit_cast(bf16x8, p[0]), __builtin_bit_cast(bf16x8, p[1]), __builtin_bit_cast(bf16x8, p[2])}};
}
struct Half {
  float x[8];
};
__device__ __forceinline__ Half half_of(const f32x16& d, int f) {  // registers 8f .. 8f + 7
  Half h;
#pragma unroll
  for (int t = 0; t < 8; ++t) h.x[t] = d[8 * f + t];
  return h;
}
__device__ __forceinline__ Planes<3> split_half(const f32x16& d, int f) { return split(half_of(d, f).x); }
// The six terms of a product, small ones first: where a sum takes the small terms of all its products before the large ones,
// they are not rounded to the precision of the large sum one by one.
constexpr int kTerm[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
// c[i] += a[i] b[i], the accumulators in turn.
template <int N>
__device__ __forceinline__ void products(const Planes<3> (&a)[N], const Planes<3> (&b)[N], f32x16 (&c)[N]) {
#pragma unroll
  for (int t = 0; t < 6; ++t)
#pragma unroll
    for (int i = 0; i < N; ++i) c[i] = mfma32(a[i].p[kTerm[t][0]], b[i].p[kTerm[t][1]], c[i]);
}
template <int N>
__device__ __forceinline__ void products(const Planes<1> (&a)[N], const Planes<1> (&b)[N], f32x16 (&c)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) c[i] = mfma32(a[i].p[0], b[i].p[0], c[i]);
}

__device__ __forceinline__ Planes<3> planes_of(u32x4 a, u32x4 b, float times) {
  float x[8];
#pragma unroll
  for (int t = 0; t < 4; ++t) x[t] = __uint_as_float(a[t]) * times, x[4 + t] = __uint_as_float(b[t]) * times;
  return split(x);
}

// COLS columns of 32 rows on their way from memory to fragments (lane (n, g): columns 16 kk + 8 g .. + 7 of row n).  A load of
// fragments would touch 32 rows, and a compute unit takes 90 cycles for such an instruction (128 of them, 5.6 us, at 16 x 777
// rows of 512 bytes); 128 bytes of each of eight rows take 16.  So whole lines go to registers, in pieces of 128 bytes a row,
// and through 4 KiB of LDS of the wave's own, whose 16-byte units are swizzled by the row.  Rows shorter than that are read as
// fragments.
template <typename T, int COLS>
struct RowTile {
  static constexpr int kSteps = COLS / 16, kPiece = 128 / sizeof(T), kPieces = COLS / kPiece, kStepsPerPiece = kPiece / 16;
  static constexpr bool kLines = COLS * sizeof(T) >= 128;
  static constexpr int kUnits = sizeof(T) == 4 ? 2 : 1;  // 16-byte units of a fragment per lane
  u32x4 v[kLines ? kPieces * 4 : kSteps * kUnits];

  // `row`: the address of a row's first column, for the row's number 0 .. 31
  template <typename F>
  __device__ __forceinline__ void load(F row, int lane) {
    if constexpr (kLines) {
      const T* p[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = row(8 * i + lane / 8) + lane % 8 * (16 / static_cast<int>(sizeof(T)));
#pragma unroll
      for (int q = 0; q < kPieces; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) v[4 * q + i] = *reinterpret_cast<const u32x4*>(p[i] + q * kPiece);
    } else {
      const T* p = row(lane & 31) + 8 * (lane >> 5);
#pragma unroll
      for (int kk = 0; kk < kSteps; ++kk)
#pragma unroll
        for (int u = 0; u < kUnits; ++u) v[kk * kUnits + u] = *reinterpret_cast<const u32x4*>(p + 16 * kk + 4 * u);
    }
  }
  // this lane's part of the fragments of a piece, by way of LDS
  struct Piece {
    u32x4 u[kLines ? kStepsPerPiece : 1][kUnits];
  };
  __device__ __forceinline__ Piece piece(unsigned char* own, int lane, int q) const {
    Piece r;
    if constexpr (kLines) {
      unsigned char* const dst = own + lane / 8 * 128 + (lane % 8 ^ lane / 8) * 16;
      const unsigned char* const src = own + (lane & 31) * 128;
      wave_lds_fence();
#pragma unroll
      for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4*>(dst + i * 1024) = v[4 * q + i];
      wave_lds_fence();
#pragma unroll
      for (int k = 0; k < kStepsPerPiece; ++k)
#pragma unroll
        for (int j = 0; j < kUnits; ++j)
          r.u[k][j] = *reinterpret_cast<const u32x4*>(src + (((2 * k + (lane >> 5)) * kUnits + j) ^ (lane & 7)) * 16);
      wave_lds_fence();
    }
    return r;
  }
  // Calls ahead(kk + 1) and then use(kk, planes) for every 16 columns: what a step needs is asked for a step ahead.  (fp32: of
  // `times` the row)
  template <typename A, typename F>
  __device__ __forceinline__ void each(unsigned char* own, int lane, float times, A ahead, F use) const {
    Piece now = piece(own, lane, 0);
    ahead(0);
    Planes<kPlanes<T>> p = step(now, 0, times);
#pragma unroll
    for (int kk = 0; kk < kSteps; ++kk) {
      if (kLines && (kk + 1) % kStepsPerPiece == 0 && kk + 1 < kSteps) now = piece(own, lane, (kk + 1) / kStepsPerPiece);
      if (kk + 1 < kSteps) ahead(kk + 1);
      __builtin_amdgcn_sched_barrier(0);
      use(kk, p);
      if (kk + 1 < kSteps) p = step(now, kk + 1, times);
    }
  }
  __device__ __forceinline__ Planes<kPlanes<T>> step(const Piece& now, int kk, float times) const {
    if constexpr (kLines) {
      return planes(now.u[kk % kStepsPerPiece], times);
    } else {
      u32x4 u[kUnits];
#pragma unroll
      for (int j = 0; j < kUnits; ++j) u[j] = v[kk * kUnits + j];
      return planes(u, times);
    }
  }
  __device__ static __forceinline__ Planes<kPlanes<T>> planes(const u32x4 (&u)[kUnits], float times) {
    if constexpr (sizeof(T) == 4) return planes_of(u[0], u[1], times);
    else return {{__builtin_bit_cast(bf16x8, u[0])}};
  }
};

// 32 rows times 32 columns with the fp32 instruction, for results that are not finite from the planes.  `row` and `col`: this lane's.
// ROWS_KEPT: lane = row, registers = columns; otherwise lane = column, registers = rows.
template <typename T, int D, bool ROWS_KEPT>
__device__ __forceinline__ f32x16 exact_block(const T* row, const T* col, int g) {
  f32x16 acc = zeros();
#pragma unroll 1
  for (int k = g; k < D; k += 2) {
    const float x = to_float(row[k]), w = to_float(col[k * D]);
    acc = ROWS_KEPT ? mfma_f32(w, x, acc) : mfma_f32(x, w, acc);
  }
  return acc;
}

__device__ __forceinline__ bool not_finite(float x) { return !(fabsf(x) < INFINITY); }
// Whether any is not finite (or, for nothing, their sum).
template <typename V>
__device__ __forceinline__ bool any_not_finite(const V& x, int count) {
  float z[2] = {x[0], x[1]};
#pragma unroll
  for (int i = 2; i < count; ++i) z[i % 2] += x[i];
  return not_finite(z[0] + z[1]);
}

__device__ __forceinline__ bool either_lane(bool x) { return pair_max(x ? 1.f : 0.f) != 0.f; }

// What a head of DH columns looks like in 32-wide blocks.
template <int DH>
struct Head {
  static constexpr int DB = (DH + 31) / 32;              // blocks
  static constexpr int KF = DH == 8 ? 1 : DH / 16;       // key fragments of 16 columns (d/h = 8: the planes share it)
  static constexpr int VP = DH == 8 ? 1 : DH == 16 ? 2 : 3;  // value fragments per 16 keys and block
  static constexpr int QUADS = DH / 8;                   // registers of a result that count, in fours, per lane
};

// Two operands whose summed index are a head's columns, from half an accumulator block (lane = row, registers = columns).  At
// d/h = 8 the slots of a fragment hold two planes of four columns: (0, 1) x (0, 0), (0, 1) x (1, 1) and (0, 2) x (2, 0).
template <int DH, bool LEFT>
__device__ __forceinline__ Planes<3> column_planes(const float (&x)[8]) {
  if constexpr (DH == 8) {
    float y[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) y[t] = x[t & 3];
    const Planes<3> s = split(y);  // (both halves alike)
    Planes<3> r;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      r.p[0][t] = LEFT ? s.p[t < 4 ? 0 : 1][t] : s.p[0][t];
      r.p[1][t] = LEFT ? s.p[t < 4 ? 0 : 1][t] : s.p[1][t];
      r.p[2][t] = LEFT ? s.p[t < 4 ? 0 : 2][t] : s.p[t < 4 ? 2 : 0][t];
    }
    return r;
  } else {
    return split(x);
  }
}
// Term t of such a product.
template <int DH>
constexpr int kColumnTerms = DH == 8 ? 3 : 6;
template <int DH>
__device__ __forceinline__ f32x16 column_term(int t, const Planes<3>& a, const Planes<3>& b, f32x16 c) {
  return DH == 8 ? mfma32(a.p[2 - t], b.p[2 - t], c) : mfma32(a.p[kTerm[t][0]], b.p[kTerm[t][1]], c);
}

// The values' fragments (lane = column, slots = keys) of one block and 16 keys, and their product with weights.
template <int DH>
__device__ __forceinline__ Planes<Head<DH>::VP> value_planes(const Planes<3>& s, int n) {
  if constexpr (DH == 8) {
    Planes<1> r;
#pragma unroll
    for (int t = 0; t < 8; ++t) r.p[0][t] = n < 8 ? s.p[0][t] : n < 16 ? s.p[1][t] : n < 24 ? s.p[2][t] : static_cast<__bf16>(0.f);
    return r;
  } else if constexpr (DH == 16) {
    Planes<2> r;
#pragma unroll
    for (int t = 0; t < 8; ++t) r.p[0][t] = n < 16 ? s.p[0][t] : s.p[1][t], r.p[1][t] = n < 16 ? s.p[2][t] : static_cast<__bf16>(0.f);
    return r;
  } else {
    return s;
  }
}
// Term t of the values' product with weights (which plane of the values, which of the weights).
template <int DH>
constexpr int kValueTerms = DH == 8 ? 3 : DH == 16 ? 4 : 6;
template <int DH>
__device__ __forceinline__ f32x16 value_term(int t, const Planes<Head<DH>::VP>& v, const Planes<3>& w, f32x16 c) {
  if constexpr (DH == 8) return mfma32(v.p[0], w.p[2 - t], c);
  else if constexpr (DH == 16) return t == 0 ? mfma32(v.p[0], w.p[2], c) : t == 1 ? mfma32(v.p[1], w.p[0], c) : mfma32(v.p[0], w.p[3 - t], c);
  else return mfma32(v.p[kTerm[t][0]], w.p[kTerm[t][1]], c);
}

// A head's result in DH / 2 registers (lane half g: columns 8q + 4g + r, register 4q + r): the rows that hold planes added up.
template <int DH>
__device__ __forceinline__ void head_result(const f32x16 (&acc)[Head<DH>::DB], float (&x)[DH / 2]) {
#pragma unroll
  for (int i = 0; i < DH / 2; ++i) {
    const f32x16& s = acc[i / 16];
    const int j = i % 16;
    x[i] = DH == 8 ? s[j] + (s[4 + j] + s[8 + j]) : DH == 16 ? s[j] + s[8 + j] : s[j];
  }
}

template <typename OutT>
__device__ __forceinline__ void store_quad(OutT* dst, const float (&x)[4]) {
  if constexpr (sizeof(OutT) == 4) {
    *reinterpret_cast<float4*>(dst) = make_float4(x[0], x[1], x[2], x[3]);
  } else {
    bf16x4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = static_cast<__bf16>(x[r]);
    *reinterpret_cast<bf16x4*>(dst) = v;
  }
}

// `times` e^x for unit x, to a unit in the last place without the handling of its ends: 2^(x log2 e) from the product rounded,
// times what the rounding left out (x log2 e = t + r, e^x = 2^t (1 + r ln 2)).  NaN where x is infinite, zero below 2^-126.
// (unit, times: powers of two)
__device__ __forceinline__ float exp_finite(float x, float unit, float times) {
  const float kLog2e = 1.44269502f * unit, kLog2eRest = 1.92596303e-8f * unit, kLn2 = 0.693147182f;
  const float t = x * kLog2e;
  const float r = fmaf(x, kLog2eRest, fmaf(x, kLog2e, -t));
  const float p = __builtin_amdgcn_exp2f(t);
  return p * fmaf(r, kLn2 * times, times);
}
// `times` x / (1 + e^-x) for unit x, the quotient corrected once.  (Past 88 the exponential is as good as infinite; NaN where x is
// infinite.)
__device__ __forceinline__ float silu_finite(float x, float unit, float times) {
  const float den = 1.f + exp_finite(fminf(-x, 88.f / unit), unit, 1.f);
  const float r = __builtin_amdgcn_rcpf(den), y = x * (unit * times), q = y * r;
  return fmaf(fmaf(-den, q, y), r, q);
}
__device__ __forceinline__ float silu(float x) { return x / (1.f + expf(-x)); }
// The logit (as the sum that stands for it) of a key that does not count, in place of -infinity where NaN asks for the exact way.
// kLowLogit: maxima below it (which no finite operands of ordinary size give) take that way too.
constexpr float kMaskedLogit = -2e38f, kLowLogit = -1e38f;

// A head's columns of three weight matrices in LDS, kUp times as large, as planes in rows: [matrix][DB][planes][D][columns, 32 at most].
// Fetched in whole lines (a load instruction costs a compute unit 16 cycles, whatever it brings: column by column they were 2.8
// of the 19.6 us of the history kernel at 16 x 777 rows), and read as fragments through the transposing LDS read.
template <typename T, int D, int DH>
struct Weights {
  static constexpr int NP = kPlanes<T>, DB = Head<DH>::DB, kCols = std::min(DH, 32), kPitch = 2 * kCols, kPlane = D * kPitch;
  static constexpr int kBytes = 3 * DB * NP * kPlane;
  static constexpr int kPerUnit = 16 / sizeof(T), kRowUnits = DH / kPerUnit, kTotal = 3 * D * kRowUnits;
  static constexpr int kMine = (kTotal + kThreads - 1) / kThreads;
  u32x4 v[kMine];
  // the matrices' first rows, at the head's first column
  __device__ __forceinline__ void load(const T* w0, const T* w1, const T* w2, int tid) {
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int u = tid + i * kThreads;
      if (kTotal % kThreads == 0 || u < kTotal) {
        const T* from = u < D * kRowUnits ? w0 : u < 2 * D * kRowUnits ? w1 : w2;
        v[i] = *reinterpret_cast<const u32x4*>(from + u / kRowUnits % D * D + u % kRowUnits * kPerUnit);
      }
    }
  }
  __device__ __forceinline__ void park(unsigned char* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
      const int u = tid + i * kThreads;
      if (kTotal % kThreads != 0 && u >= kTotal) continue;
      const int col = u % kRowUnits * kPerUnit, matrix = u / (D * kRowUnits);
      unsigned char* dst = lds + (matrix * DB + col / 32) * NP * kPlane + u / kRowUnits % D * kPitch + col % 32 * 2;
      if constexpr (NP == 3) {
        float x[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) x[t] = __uint_as_float(v[i][t % 4]) * kUp<T>;
        const Planes<3> p = split(x);  // (both halves alike)
#pragma unroll
        for (int k = 0; k < 3; ++k) *reinterpret_cast<bf16x4*>(dst + k * kPlane) = __builtin_shufflevector(p.p[k], p.p[k], 0, 1, 2, 3);
      } else {
        *reinterpret_cast<u32x4*>(dst) = v[i];
      }
    }
  }
  // rows 16 kk .. of 32 columns as a fragment, a narrow head's columns repeated (see column_fragment)
  __device__ static __forceinline__ Planes<NP> fragment(const unsigned char* lds, int matrix, int ob, int kk, int lane) {
    const int chunk = ((lane >> 4 & 1) * 4 + lane % 4) % (kCols / 4);
    const unsigned char* p = lds + (matrix * DB + ob) * NP * kPlane + 16 * kk * kPitch + (8 * (lane >> 5) + lane % 16 / 4) * kPitch + chunk * 8;
    auto at = [](const unsigned char* q) {
      return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(q)));
    };
    Planes<NP> r;
#pragma unroll
    for (int k = 0; k < NP; ++k)
      r.p[k] = __builtin_shufflevector(at(p + k * kPlane), at(p + k * kPlane + 4 * kPitch), 0, 1, 2, 3, 4, 5, 6, 7);
    return r;
  }
};

__device__ __forceinline__ void park_block(float* dst, const f32x16& x, int lane) {
#pragma unroll
  for (int i = 0; i < 16; ++i) dst[i * 64 + lane] = x[i];
}

// One 32 x 32 block of a projection of the links, its sum over k shared out to SPLITS waves, each with COLS = D / SPLITS
// columns of the 32 link rows.  Lane = row, registers = columns (rows_kept, uniform), or lane = column, registers = rows.
template <typename W, typename T, int COLS>
__device__ __forceinline__ f32x16 partial_block(const RowTile<T, COLS>& x, const unsigned char* weights, int matrix, int ob, int part,
                                                unsigned char* own, bool rows_kept, int lane) {
  f32x16 acc[1] = {zeros()};
  Planes<kPlanes<T>> w[2];
  x.each(own, lane, kUp<T>, [&](int kk) { w[kk & 1] = W::fragment(weights, matrix, ob, part * (COLS / 16) + kk, lane); },
         [&](int kk, const Planes<kPlanes<T>>& p) {
           const Planes<kPlanes<T>> a[1] = {p}, b[1] = {w[kk & 1]};
           if (rows_kept) products(b, a, acc);
           else products(a, b, acc);
         });
  return acc[0];
}

template <int NP>
__device__ __forceinline__ Planes<NP> parked(const bf16x8* src, int lane) {
  Planes<NP> r;
#pragma unroll
  for (int k = 0; k < NP; ++k) r.p[k] = src[k * 64 + lane];
  return r;
}
template <int NP>
__device__ __forceinline__ void park(bf16x8* dst, const Planes<NP>& x, int lane) {
#pragma unroll
  for (int k = 0; k < NP; ++k) dst[k * 64 + lane] = x.p[k];
}

// The widths the kernels are built for.
#define LIME_FUSED_SHAPES(CASE) \
  CASE(32, 8) CASE(32, 16) CASE(32, 32) CASE(64, 8) CASE(64, 16) CASE(64, 32) CASE(64, 64) CASE(128, 16) CASE(128, 32)
inline bool fused_shape(int d, int h) {
#define LIME_CASE(D, DH) \
  if (d == D && d == DH * h) return true;
  LIME_FUSED_SHAPES(LIME_CASE)
#undef LIME_CASE
  return false;
}

// Waves per SIMD: two workgroups on a compute unit where their registers fit, nearly (in fp32 at d = 64 the rows kernel spills 12:
// 128 users, C = 512, d = 64, h = 8 38.7 us with them, 43.1 with one workgroup; at d = 128 88.5 and 61.3).
constexpr int fused_waves(int D, int DH) { return DH < 32 && D < 128 ? 4 : 2; }

// Workgroups that read the same rows (the heads of one user's) on one XCD: consecutive blocks go to consecutive XCDs.
__device__ __forceinline__ int block_on_xcd(int total) {
  const int per = (total + 7) / 8;
  return static_cast<int>(blockIdx.x) % 8 * per + static_cast<int>(blockIdx.x) / 8;
}

}  // namespace
}  // namespace lime
