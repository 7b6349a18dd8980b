// The products of the translation GEMMs on the 16-bit matrix cores (device
// code, gfx950).
//
// v_mfma_f32_16x16x32 takes 16-bit operands at 16 times the rate of the
// float32 MFMA, forms every product exactly and adds in float32.  A float32 x
// is the sum of three bfloat16 values (x0 the rounding of x, x1 that of
// x - x0, x2 the rest: 8 significant bits each, the remainders are exact), so
// a b = a0 b0 + (a0 b1 + a1 b0) + (a0 b2 + a1 b1 + a2 b0) up to 2^-26 |a b|,
// below the rounding of one float32 product: six MFMAs of 32 products take
// the place of eight float32 MFMAs of 4 products (96 against 256 matrix-core
// cycles for 16 x 16 x 32), and an output entry is rounded 6 times per 32
// products instead of 32 times.
//
// Operand forms (OP):
//   OP_F32   float32 operators, split in registers as they arrive; 3 planes
//   OP_P4    precise plans' directional operators: four bfloat16 planes (32
//            bits) formed at plan time from the float64 operator; 9 products
//   OP_F16   FP16X3 plans: two float16 planes, scaled per operator and per column
//   OP_BF16  BF16X3 plans: two bfloat16 planes
//
// Complex numbers are planar inside a step: a step of 32 complex k takes the
// real and the imaginary parts of the operator rows and of the columns as
// separate fragments, for a tile of 16 complex rows
//   Re += Are Xre - Aim Xim,   Im += Are Xim + Aim Xre.
// A split operator entry thus serves four products where the interleaved form
// (rows (Re, -Im), (Im, Re)) would split every entry twice.  The three sums of
// a step start from zero (the small products first) and are added to the
// tile's sums on the vector unit, so an output entry is rounded to its full
// size once or twice per step and not once per MFMA.
//
// K comes in chunks of 8 complex entries (ranks are padded to 8): the four
// 16-lane groups of a wave take one chunk each, so a full step has 4 chunks.
// Of the last K / 8 mod 4 chunks, one or two make a merged step of half the
// MFMAs: lane groups below rem take a chunk's (Are, Aim) against Xre, the next
// rem groups i A = (-Aim, Are) against Xim, the others a zero column chunk;
// three make a full step whose fourth group takes a zero column chunk.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace dfmm {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));  // an MFMA accumulator tile
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
constexpr int PREC_F16 = 1, PREC_BF16 = 2;

enum { OP_F32 = 0, OP_F16 = 1, OP_BF16 = 2, OP_P4 = 3 };
template <int OP>
struct OpForm {
  static constexpr int AW = OP == OP_P4 ? 8 : 4;   // float4 of an operator row's chunk (8 complex entries)
  static constexpr int PA = OP == OP_P4 ? 4 : (OP == OP_F32 ? 3 : 2);  // operator planes
  static constexpr int PB = OP == OP_P4 || OP == OP_F32 ? 3 : 2;       // column planes
  static constexpr int CU = 2 * PB;                // 16-byte LDS units of a column's chunk
};

// Chunks of a staged column of K complex entries: an odd number of chunks gets
// one of zeros for the lane groups without a chunk of their own.
__host__ __device__ inline int col_chunks(int K) { return (K / 8 + 1) / 2 * 2; }
// Its 16-byte LDS units: odd, so that the 16 columns that a wave reads at one
// chunk fall in different banks.
__host__ __device__ inline int col_units(int K, int pb) { return col_chunks(K) * 2 * pb + 1; }

// two float32 as two bfloat16 in a word, the first in the low half
__device__ __forceinline__ unsigned pack_bf16(float a, float b) {
  const v2f v = {a, b};
  return __builtin_bit_cast(unsigned, __builtin_convertvector(v, v2bf));
}
__device__ __forceinline__ float lo_bf16(unsigned w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

// x = hi + lo with hi the 16-bit rounding of x and lo that of the (exact) remainder
template <int PREC>
__device__ __forceinline__ void split_pair(float a, float b, unsigned& hi, unsigned& lo) {
  if constexpr (PREC == PREC_F16) {
    const _Float16 ha = _Float16(a), hb = _Float16(b);
    const _Float16 la = _Float16(a - float(ha)), lb = _Float16(b - float(hb));
    hi = unsigned(__builtin_bit_cast(unsigned short, ha)) | (unsigned(__builtin_bit_cast(unsigned short, hb)) << 16);
    lo = unsigned(__builtin_bit_cast(unsigned short, la)) | (unsigned(__builtin_bit_cast(unsigned short, lb)) << 16);
  } else {
    hi = pack_bf16(a, b);
    lo = pack_bf16(a - lo_bf16(hi), b - hi_bf16(hi));
  }
}

// the planes of two values, one word per plane
template <int OP, int P>
__device__ __forceinline__ void split_planes(float a, float b, unsigned (&w)[P]) {
  if constexpr (OP == OP_F16) {
    split_pair<PREC_F16>(a, b, w[0], w[1]);
  } else {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      w[p] = pack_bf16(a, b);
      if (p + 1 < P) {
        a -= lo_bf16(w[p]);
        b -= hi_bf16(w[p]);
      }
    }
  }
}

template <int PREC>
__device__ __forceinline__ v4f mfma16(v4u a, v4u b, v4f c) {
  if constexpr (PREC == PREC_F16)
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0,
                                                   0);
}
template <int OP>
__device__ __forceinline__ v4f mfma_op(v4u a, v4u b, v4f c) {
  return mfma16<OP == OP_F16 ? PREC_F16 : PREC_BF16>(a, b, c);
}

// the plane pairs (a, b) of a product, smallest first
template <int OP>
struct Products;
template <>
struct Products<OP_F32> {
  static constexpr int n = 6, a[6] = {2, 0, 1, 1, 0, 0}, b[6] = {0, 2, 1, 0, 1, 0};
};
template <>
struct Products<OP_P4> {
  static constexpr int n = 9, a[9] = {3, 2, 1, 2, 0, 1, 1, 0, 0}, b[9] = {0, 1, 2, 0, 2, 1, 0, 1, 0};
};
template <>
struct Products<OP_F16> {
  static constexpr int n = 3, a[3] = {1, 0, 0}, b[3] = {0, 1, 0};
};
template <>
struct Products<OP_BF16> : Products<OP_F16> {};

// The steps of a K-long row, and this lane's place in them.
struct OpRows {
  int nf, rem, ns;  // full steps; chunks of the merged last step (0: none); steps
  int nq, last;     // steps of four stored chunks; chunks stored in the step after them
  int kr, j;        // this lane's chunk in a full step and row / column in a tile
  __device__ __forceinline__ OpRows(int K, int lane) {
    const int nch = K / 8;
    nq = nch / 4;
    last = nch % 4;
    rem = last == 3 ? 0 : last;
    nf = nq + (last == 3 ? 1 : 0);
    ns = nf + (rem ? 1 : 0);
    kr = lane >> 4;
    j = lane & 15;
  }
  // whether this lane takes i A in the merged step
  __device__ __forceinline__ bool turned() const { return kr >= rem; }
};

// One wave's operator rows: a tile of 16 rows (8 where the operator ends on a
// half tile) holds, per step, the float4 t of chunk c of row j at
// (t nc + c) rows + j, nc chunks in the step.
template <int OP>
struct OpTile {
  static constexpr int AW = OpForm<OP>::AW;
  const float4* p;   // the tile
  int step;          // float4 of a step of four chunks
  int v4, vl;        // this lane's chunk and row in such a step / in the step after them
  int t4, tl;        // float4 from one t to the next, likewise
  int nq;
  __device__ __forceinline__ OpTile(const OpRows& o, const float4* __restrict__ tile, int rows) {
    const int row = o.j & (rows - 1);
    p = tile;
    step = 4 * AW * rows;
    v4 = o.kr * rows + row;
    // lane groups without a chunk of their own repeat one (their column chunk is zeros)
    vl = (o.last == 2 ? (o.kr & 1) : min(o.kr, max(o.last - 1, 0))) * rows + row;
    t4 = 4 * rows;
    tl = o.last * rows;
    nq = o.nq;
  }
};
template <int OP>
__device__ __forceinline__ void load_rows(const float4* __restrict__ p, int v, int ts, float4 (&raw)[OpForm<OP>::AW]) {
#pragma unroll
  for (int t = 0; t < OpForm<OP>::AW; ++t) raw[t] = (p + t * ts)[v];
}
template <int OP>
__device__ __forceinline__ void load_first(const OpTile<OP>& r, float4 (&raw)[OpForm<OP>::AW]) {
  const bool four = r.nq > 0;
  load_rows<OP>(r.p, four ? r.v4 : r.vl, four ? r.t4 : r.tl, raw);
}

// operator fragments of a step (turned lanes: of i A)
template <int OP>
struct Frag {
  v4u re[OpForm<OP>::PA], im[OpForm<OP>::PA];
};
template <int OP, bool MERGED>
__device__ __forceinline__ void make_frag(const float4 (&raw)[OpForm<OP>::AW], bool turned, Frag<OP>& f) {
  constexpr int PA = OpForm<OP>::PA;
  if constexpr (OP == OP_F32) {
    float4 v[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      v[t] = raw[t];
      if constexpr (MERGED) {
        const float4 w = v[t];
        v[t] = make_float4(turned ? -w.y : w.x, turned ? w.x : w.y, turned ? -w.w : w.z, turned ? w.z : w.w);
      }
    }
#pragma unroll
    for (int t = 0; t < 4; ++t) {  // two complex entries
      unsigned r[PA], i[PA];
      split_planes<OP>(v[t].x, v[t].z, r);
      split_planes<OP>(v[t].y, v[t].w, i);
#pragma unroll
      for (int p = 0; p < PA; ++p) {
        f.re[p][t] = r[p];
        f.im[p][t] = i[p];
      }
    }
  } else {  // stored as planes: unit 2 p + part
#pragma unroll
    for (int p = 0; p < PA; ++p) {
      f.re[p] = __builtin_bit_cast(v4u, raw[2 * p]);
      f.im[p] = __builtin_bit_cast(v4u, raw[2 * p + 1]);
      if constexpr (MERGED) {
        const v4u r = f.re[p], i = f.im[p], sg = {0x80008000u, 0x80008000u, 0x80008000u, 0x80008000u};
        f.re[p] = turned ? (i ^ sg) : r;
        f.im[p] = turned ? r : i;
      }
    }
  }
}

// A step's sums of one tile of 16 columns: Re = p - q, Im = i.  xb: this lane's
// column at its chunk (merged last step: its imaginary parts in turned lanes, q
// unused).
struct StepSums {
  v4f p, q, i;
};
template <int OP>
__device__ __forceinline__ StepSums step_full(const Frag<OP>& f, const v4u* xb) {
  using P = Products<OP>;
  constexpr int PB = OpForm<OP>::PB;
  v4u xr[PB], xi[PB];
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    xr[p] = xb[2 * p];
    xi[p] = xb[2 * p + 1];
  }
  StepSums s;
  s.p = s.q = s.i = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < P::n; ++k) {
    s.p = mfma_op<OP>(f.re[P::a[k]], xr[P::b[k]], s.p);
    s.i = mfma_op<OP>(f.re[P::a[k]], xi[P::b[k]], s.i);
    s.q = mfma_op<OP>(f.im[P::a[k]], xi[P::b[k]], s.q);
    s.i = mfma_op<OP>(f.im[P::a[k]], xr[P::b[k]], s.i);
  }
  return s;
}
template <int OP>
__device__ __forceinline__ StepSums step_merged(const Frag<OP>& f, const v4u* xb) {
  using P = Products<OP>;
  constexpr int PB = OpForm<OP>::PB;
  v4u x[PB];
#pragma unroll
  for (int p = 0; p < PB; ++p) x[p] = xb[2 * p];
  StepSums s;
  s.p = s.q = s.i = v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < P::n; ++k) {
    s.p = mfma_op<OP>(f.re[P::a[k]], x[P::b[k]], s.p);
    s.i = mfma_op<OP>(f.im[P::a[k]], x[P::b[k]], s.i);
  }
  return s;
}

// units of this lane's chunk of step s in a staged column (zero chunk: the last)
template <int OP>
__device__ __forceinline__ int step_unit(const OpRows& o, int s) {
  constexpr int CU = OpForm<OP>::CU;
  if (s < o.nf) return (4 * s + o.kr) * CU;  // the fourth group of a cut step takes the zero chunk
  const int c = o.rem == 2 ? (o.kr & 1) : (o.kr < 2 ? 0 : 1);
  return (4 * s + c) * CU + (o.kr >= o.rem ? 1 : 0);
}

// The products of one row tile: acc(n, sums, merged) takes the sums of every step
// and column tile n as they are done (so that one tile's are live at a time).  raw
// holds step 0 on entry and step 0 of the next tile rn on return: the rows of
// the step to come are in flight while one multiplies.
template <int OP, int NT, typename F>
__device__ __forceinline__ void tile_product(const OpRows& o, const OpTile<OP>& r, const OpTile<OP>& rn,
                                             const v4u* xcol, int cs, float4 (&raw)[OpForm<OP>::AW], F&& acc) {
  const int vn = rn.nq > 0 ? rn.v4 : rn.vl, tn = rn.nq > 0 ? rn.t4 : rn.tl;
  auto load = [&](int s) {  // step s, or the next tile's first past the last
    const bool in = s < o.ns, four = s < r.nq;
    const float4* p = in ? r.p + s * r.step : rn.p;
    const int v = in ? (four ? r.v4 : r.vl) : vn;
    const int t = in ? (four ? r.t4 : r.tl) : tn;
    load_rows<OP>(p, v, t, raw);
  };
  for (int s = 0; s < o.nf; ++s) {
    Frag<OP> f;
    make_frag<OP, false>(raw, false, f);
    load(s + 1);
    const v4u* xb = xcol + step_unit<OP>(o, s);
#pragma unroll
    for (int n = 0; n < NT; ++n) acc(n, step_full<OP>(f, xb + n * 16 * cs), std::false_type());
  }
  if (o.rem) {
    Frag<OP> f;
    make_frag<OP, true>(raw, o.turned(), f);
    load(o.ns);
    const v4u* xb = xcol + step_unit<OP>(o, o.nf);
#pragma unroll
    for (int n = 0; n < NT; ++n) acc(n, step_merged<OP>(f, xb + n * 16 * cs), std::true_type());
  }
}

// Largest value over the wave, by lane shuffles inside the vector unit.
__device__ __forceinline__ float wave_max(float v) {
  auto step = [&](auto ctrl) {
    const int w = __builtin_amdgcn_update_dpp(__float_as_int(v), __float_as_int(v), decltype(ctrl)::value, 0xF, 0xF, false);
    v = fmaxf(v, __int_as_float(w));
  };
  step(std::integral_constant<int, 0x111>());  // row_shr 1, 2, 4, 8: lane 15 of a row has the row's
  step(std::integral_constant<int, 0x112>());
  step(std::integral_constant<int, 0x114>());
  step(std::integral_constant<int, 0x118>());
  step(std::integral_constant<int, 0x142>());  // row_bcast 15, 31: lane 63 has the wave's
  step(std::integral_constant<int, 0x143>());
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Stage two complex entries at w, the word of a column's chunk that holds them
// (word q mod 4 of each unit of chunk q / 4 for float4 q of the column).
template <int OP>
__device__ __forceinline__ void stage_words(unsigned* w, float4 v) {
  constexpr int PB = OpForm<OP>::PB;
  unsigned r[PB], i[PB];
  split_planes<OP>(v.x, v.z, r);
  split_planes<OP>(v.y, v.w, i);
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    w[8 * p] = r[p];
    w[8 * p + 4] = i[p];
  }
}
template <int OP>
__device__ __forceinline__ int stage_word(int q) {
  return (q >> 2) * (4 * OpForm<OP>::CU) + (q & 3);
}
template <int OP>
__device__ __forceinline__ void stage_pair(unsigned* xc, int q, float4 v) {
  stage_words<OP>(xc + stage_word<OP>(q), v);
}

}  // namespace
}  // namespace dfmm
