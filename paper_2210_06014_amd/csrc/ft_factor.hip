// Factor pass: shared g per fiber, in-place chains, chunk maps, combine.
#include "ft_device.h"

namespace ft {
namespace {

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef double doublex4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Factor pass.  Each element x of a row, in order:
//     w = prod_{n != m} C(n)[i_n, :],  g = B(m) w,  e = x - a.g,
//     a <- a + (-lr lam) a + (lr e) g                       (Eq. (9), (10))
//
// The steps of a row are serial, but their expensive parts are not: a wavefront
// takes a row in blocks of 16 elements and solves a block's 16 steps at once.
// With rho = 1 - lr lam, gp = lr / rho, a_0 the row at the block's start, G the
// block's 16 x J matrix of g and e~_t = rho^-t e_t (t = 0..15), the steps are
//     (I + gp tril(G G^T, -1)) e~ = (rho^-t x_t) - G a_0,
//     a_nb = rho^nb (a_0 + gp G^T e~),
// the same result in another order of operations.  G and K = G G^T do not
// depend on a_0: they are matrix products (v_mfma_f32_16x16x4_f32) formed a
// block ahead; what stays serial is one product G a_0, a 16 x 16 forward
// substitution and one product G^T e~.
//
// What bounds it: issue.  An FP32 MFMA holds the VALU for its 32 cycles (16 of
// them and 64 FMAs take the sum of their times, in one wavefront or in four),
// so a block costs 24 MFMA (G and K at J = R = 32; 64 where a chunk map is
// carried too) plus the VALU work of the serial part, which dominates at
// J <= 16; there many chunks go four to a wavefront instead (quad_items).  The
// bf16 MFMA would run beside the VALU, but it truncates the terms of an
// instruction to the largest one's 24 bits: G from three bf16 parts per value
// took a tenth off a launch and doubled the error of A.  One item per wavefront
// otherwise, because a block's MFMA then serves one chain and the chain is 4
// times shorter than with an item per 16 lanes.  Against one step per element
// on 16 lanes (g by row broadcasts), us per launch: Netflix-shaped 8M elements,
// J = R = 32, modes 0 to 2: 828, 1048, 1048 -> 393, 500, 557; order 4 (3M, J = R = 32)
// 934 -> 241; order 6 (1M, BF16) 157 -> 59; order 8 (1M, J = 8, R = 16) 334
// -> 62; Netflix-shaped 5M, J = R = 16: 267 -> 154.
//
// Lane l = 16 g + i of the wavefront holds:
//   Gu[k]  G[i][jbase(g) + k], k < J / 4   (as the MFMA that forms G leaves it,
//          and as the operand of K = G G^T and of G N)
//   Gr[k]  G[sbase(g) + k][j], j = the lane's state index (through LDS)
//   L[s]   -gp K[i][s] for s < i, else 0   (through LDS, all rows of 16 alike)
//   a      the row's element j = 16 (g % 2) + i (J = 32), i % J otherwise, FP64,
//          as are its increments: the decay lr lam a is about a hundred ulps of
//          a and nearly constant, so rounding the running row to FP32 would
//          accumulate coherently.
// Values of other lanes are read by DPP row broadcasts, so a state vector is
// also kept rotated per row of 16: broadcast k then gives lane row g its
// jbase(g) + k.  Slots past the end of an item hold x = 0 and G = 0.

// Byte offset of row i of a C table, unsigned 32-bit: plan creation refuses
// I_n * R * 4 >= 2^31, so the product never wraps.
template <int R, class T>
__device__ __forceinline__ uint32_t row_bytes(int32_t i) {
  return (uint32_t)i * (uint32_t)(R * sizeof(T));
}

// K floats at byte offset `off` of a table (K * sizeof(T) bytes, aligned to
// that size: C rows are whole multiples of it), as loaded
template <int BYTES>
struct RawOf;
template <>
struct RawOf<4> {
  typedef uint32_t type;
};
template <>
struct RawOf<8> {
  typedef uint2 type;
};
template <>
struct RawOf<16> {
  typedef uint4 type;
};
template <>
struct RawOf<32> {
  struct type {
    uint4 a, b;
  };
};

template <class T, int K>
struct Slice {
  typename RawOf<K * (int)sizeof(T)>::type raw;
  __device__ __forceinline__ void load(const T* base, uint32_t off) {
    const char* p = reinterpret_cast<const char*>(base) + off;
    if constexpr (K * sizeof(T) == 32) {
      raw.a = *reinterpret_cast<const uint4*>(p);
      raw.b = *reinterpret_cast<const uint4*>(p + 16);
    } else {
      raw = *reinterpret_cast<const typename RawOf<K * (int)sizeof(T)>::type*>(p);
    }
  }
  __device__ __forceinline__ void widen(float (&o)[K]) const {
    uint32_t w[(K * sizeof(T)) / 4];
    __builtin_memcpy(w, &raw, sizeof(w));
    if constexpr (sizeof(T) == 4) {
#pragma unroll
      for (int k = 0; k < K; ++k) o[k] = __uint_as_float(w[k]);
    } else {
#pragma unroll
      for (int k = 0; k < K / 2; ++k) {
        o[2 * k] = __uint_as_float(w[k] << 16);
        o[2 * k + 1] = __uint_as_float(w[k] & 0xFFFF0000u);
      }
    }
  }
};

// Powers of rho that the blocks need, formed on the host in FP64.
struct RhoPow {
  double p[17];                // rho^nb
  float inv[16], inv_lo[16];   // rho^-t, to twice FP32's precision
};

// rho^-t x - u with one rounding (of the difference): x and rho^-t x are often
// much larger than the residual, and an FP32 product would round it by theirs.
// (With that product the error of A in relaxed passes of a learning regime was
// a tenth above that of one step per element.)
__device__ __forceinline__ float scaled_residual(float x, float inv, float inv_lo, float u) {
  return fmaf(x, inv_lo, fmaf(x, inv, -u));
}

template <int J>
struct Geo : JLayout<J> {
  static constexpr int NS = J >= 32 ? 8 : 4;    // values of Gr
  static constexpr int GS = J + 4;              // LDS row stride of G in floats
  static constexpr int LS = 20;                 // LDS row stride of L in floats
  __device__ static int sbase(int g) { return J >= 32 ? 8 * (g >> 1) : 4 * g; }
  __device__ static int jlane(int i, int g) { return J >= 32 ? 16 * (g & 1) + i : i % J; }
};

template <int J>
struct __align__(16) WaveLds {
  float G[16 * Geo<J>::GS];
  float L[16 * Geo<J>::LS];
  float T[16 * Geo<J>::LS];  // inverse of a map's block
  float P[8 * 12];
};

// `v` with the lanes of row g of 16 rotated so that lane i holds the value of
// lane (i + STEP g) % 16; J = 32 rotates rows 2 and 3 by 8
template <int C1, int C2, int C3>
__device__ __forceinline__ float rotate_rows(float v) {
  int r = __builtin_bit_cast(int, v);
  const int s = r;
  if constexpr (C1 != 0) r = __builtin_amdgcn_update_dpp(r, s, 0x120 + C1, 0x2, 0xf, false);
  if constexpr (C2 != 0) r = __builtin_amdgcn_update_dpp(r, s, 0x120 + C2, 0x4, 0xf, false);
  if constexpr (C3 != 0) r = __builtin_amdgcn_update_dpp(r, s, 0x120 + C3, 0x8, 0xf, false);
  return __builtin_bit_cast(float, r);
}
template <int J>
__device__ __forceinline__ float rotate_state(float v) {
  if constexpr (J >= 32) return rotate_rows<0, 8, 8>(v);
  else if constexpr (J >= 16) return rotate_rows<12, 8, 4>(v);
  else return rotate_rows<14, 12, 10>(v);
}
template <int C1, int C2, int C3>
__device__ __forceinline__ double rotate_rows(double v) {
  float w[2];
  __builtin_memcpy(w, &v, 8);
  w[0] = rotate_rows<C1, C2, C3>(w[0]);
  w[1] = rotate_rows<C1, C2, C3>(w[1]);
  __builtin_memcpy(&v, w, 8);
  return v;
}
template <int J>
__device__ __forceinline__ double rotate_state(double v) {
  if constexpr (J >= 32) return rotate_rows<0, 8, 8>(v);
  else if constexpr (J >= 16) return rotate_rows<12, 8, 4>(v);
  else return rotate_rows<14, 12, 10>(v);
}
template <int J, class V>
__device__ __forceinline__ V rotate_slots(V v) {
  if constexpr (J >= 32) return rotate_rows<0, 8, 8>(v);
  else return rotate_rows<12, 8, 4>(v);
}

// sums over lanes l, l ^ 32 and over l, l ^ 16; every lane ends with the same bits
__device__ __forceinline__ float sum_halves(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_rows(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ double sum_halves(double v) {
  uint32_t w[2];
  __builtin_memcpy(w, &v, 8);
  const auto lo = __builtin_amdgcn_permlane32_swap(w[0], w[0], false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(w[1], w[1], false, false);
  const uint32_t a[2] = {lo[0], hi[0]}, b[2] = {lo[1], hi[1]};
  double x, y;
  __builtin_memcpy(&x, a, 8);
  __builtin_memcpy(&y, b, 8);
  return x + y;
}
__device__ __forceinline__ double sum_rows(double v) {
  uint32_t w[2];
  __builtin_memcpy(w, &v, 8);
  const auto lo = __builtin_amdgcn_permlane16_swap(w[0], w[0], false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(w[1], w[1], false, false);
  const uint32_t a[2] = {lo[0], hi[0]}, b[2] = {lo[1], hi[1]};
  double x, y;
  __builtin_memcpy(&x, a, 8);
  __builtin_memcpy(&y, b, 8);
  return x + y;
}

// acc + sum_{k<K} src[lane k of the row] * v[k].  The trailing s_nop covers a
// consumer that reads the result through DPP, a permute or an MFMA: the
// compiler does not see the VALU write inside the block.
#define FT_BSUM_END "s_nop 1"
template <int K>
__device__ __forceinline__ float bsum(float src, const float* v) {
  float acc = 0.f;
  if constexpr (K == 8) {
    asm("s_nop 4\n\t" FT_DOT(0, 2) FT_DOT(1, 3) FT_DOT(2, 4) FT_DOT(3, 5) FT_DOT(4, 6) FT_DOT(5, 7) FT_DOT(6, 8)
            FT_DOT(7, 9) FT_BSUM_END
        : "+v"(acc)
        : "v"(src), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
  } else if constexpr (K == 4) {
    asm("s_nop 4\n\t" FT_DOT(0, 2) FT_DOT(1, 3) FT_DOT(2, 4) FT_DOT(3, 5) FT_BSUM_END
        : "+v"(acc)
        : "v"(src), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
  } else {
    static_assert(K == 2, "2, 4 or 8 broadcasts");
    asm("s_nop 4\n\t" FT_DOT(0, 2) FT_DOT(1, 3) FT_BSUM_END : "+v"(acc) : "v"(src), "v"(v[0]), "v"(v[1]));
  }
  return acc;
}

// the same in FP64 (a 64-bit DPP operand knows row_newbcast only, which is what is needed)
#define FT_DOT64(n, op) "v_fmac_f64_dpp %0, %1, %" #op FT_BC(n)
template <int K>
__device__ __forceinline__ double bsum(double src, const double* v) {
  double acc = 0.0;
  if constexpr (K == 8) {
    asm("s_nop 4\n\t" FT_DOT64(0, 2) FT_DOT64(1, 3) FT_DOT64(2, 4) FT_DOT64(3, 5) FT_DOT64(4, 6) FT_DOT64(5, 7)
            FT_DOT64(6, 8) FT_DOT64(7, 9) FT_BSUM_END
        : "+v"(acc)
        : "v"(src), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]), "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7]));
  } else if constexpr (K == 2) {
    asm("s_nop 4\n\t" FT_DOT64(0, 2) FT_DOT64(1, 3) FT_BSUM_END : "+v"(acc) : "v"(src), "v"(v[0]), "v"(v[1]));
  } else {
    static_assert(K == 4, "2, 4 or 8 broadcasts");
    asm("s_nop 4\n\t" FT_DOT64(0, 2) FT_DOT64(1, 3) FT_DOT64(2, 4) FT_DOT64(3, 5) FT_BSUM_END
        : "+v"(acc)
        : "v"(src), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]));
  }
  return acc;
}

// Forward substitution: z_i += L[s] z_s for s = 0..14 in turn (L[s] = 0 in
// lanes i <= s).  Each step reads the step before through DPP: two wait states.
#define FT_SUB(n, op) "v_fmac_f32_dpp %0, %0, %" #op FT_BC(n) "s_nop 1\n\t"
__device__ __forceinline__ float forward_substitute(float z, const float (&L)[16]) {
  asm("s_nop 4\n\t" FT_SUB(0, 1) FT_SUB(1, 2) FT_SUB(2, 3) FT_SUB(3, 4) FT_SUB(4, 5) FT_SUB(5, 6) FT_SUB(6, 7)
          FT_SUB(7, 8) FT_SUB(8, 9) FT_SUB(9, 10) FT_SUB(10, 11) FT_SUB(11, 12) FT_SUB(12, 13) FT_SUB(13, 14)
              FT_SUB(14, 15)
      : "+v"(z)
      : "v"(L[0]), "v"(L[1]), "v"(L[2]), "v"(L[3]), "v"(L[4]), "v"(L[5]), "v"(L[6]), "v"(L[7]), "v"(L[8]), "v"(L[9]),
        "v"(L[10]), "v"(L[11]), "v"(L[12]), "v"(L[13]), "v"(L[14]));
  return z;
}

// The same solution as r plus the rest that is returned here, with one rounding
// of its size: a lane's sum above passes through up to 15 of them.  The rest,
// L z, is small beside z, so it is summed again from the z found.
#define FT_LZ(n, acc, op) "v_fmac_f32_dpp %" #acc ", %0, %" #op FT_BC(n)
__device__ __forceinline__ float solve_rest(float r, const float (&L)[16]) {
  float z = r, c0 = 0.f, c1 = 0.f;
  asm("s_nop 4\n\t" FT_SUB(0, 3) FT_SUB(1, 4) FT_SUB(2, 5) FT_SUB(3, 6) FT_SUB(4, 7) FT_SUB(5, 8) FT_SUB(6, 9)
          FT_SUB(7, 10) FT_SUB(8, 11) FT_SUB(9, 12) FT_SUB(10, 13) FT_SUB(11, 14) FT_SUB(12, 15) FT_SUB(13, 16)
              FT_SUB(14, 17) FT_LZ(0, 1, 3) FT_LZ(1, 2, 4) FT_LZ(2, 1, 5) FT_LZ(3, 2, 6) FT_LZ(4, 1, 7) FT_LZ(5, 2, 8)
                  FT_LZ(6, 1, 9) FT_LZ(7, 2, 10) FT_LZ(8, 1, 11) FT_LZ(9, 2, 12) FT_LZ(10, 1, 13) FT_LZ(11, 2, 14)
                      FT_LZ(12, 1, 15) FT_LZ(13, 2, 16) FT_LZ(14, 1, 17)
      : "+v"(z), "+v"(c0), "+v"(c1)
      : "v"(L[0]), "v"(L[1]), "v"(L[2]), "v"(L[3]), "v"(L[4]), "v"(L[5]), "v"(L[6]), "v"(L[7]), "v"(L[8]), "v"(L[9]),
        "v"(L[10]), "v"(L[11]), "v"(L[12]), "v"(L[13]), "v"(L[14]));
  return c0 + c1;
}

// y[0..S-1] += (lane S's L[0..S-1]) * y[S]: one step of the rows of the inverse
// of a unit lower triangular 8 x 8 matrix I - L, lane i holding row i % 8
template <int S>
__device__ __forceinline__ void inverse_step(float (&y)[8], const float (&L)[8]) {
#define FT_INV(n) asm("v_fmac_f32_dpp %0, %1, %2 row_newbcast:" #n " row_mask:0xf bank_mask:0xf" : "+v"(y[s]) : "v"(L[s]), "v"(y[S]))
#pragma unroll
  for (int s = 0; s < S; ++s) {
    if constexpr (S == 1) FT_INV(1);
    if constexpr (S == 2) FT_INV(2);
    if constexpr (S == 3) FT_INV(3);
    if constexpr (S == 4) FT_INV(4);
    if constexpr (S == 5) FT_INV(5);
    if constexpr (S == 6) FT_INV(6);
    if constexpr (S == 7) FT_INV(7);
  }
#undef FT_INV
}

// Source of the blocks' G: the C rows of an element's other modes (w, then
// B(m) w), its fiber's g, or (NC, order 3 and J = R = 16) C rows formed from
// A and B on use.  `Idx` is what a lane loads for its slot, `Raw` the slices
// gathered with it; both are loaded blocks ahead of their use.
template <int N, int J, int R, class T, bool FIB, bool NC>
struct Source {
  static constexpr int KR = R / 4;
  static constexpr int NI = FIB ? 1 : N - 1;
  static constexpr int RK = FIB ? Geo<J>::NG : KR;
  using E = typename std::conditional<FIB, float, T>::type;  // element type of the gathered table
  struct Idx {
    uint32_t o[NI];
    float x;
  };
  struct Raw {
    Slice<E, RK> s[NI];
  };
  const int32_t* idx;
  int64_t nnz;
  const float* val;
  CPtrs<N, T> cp;
  const int32_t* fid;
  const float* gfib;
  NoC<N> nc;
  GForm<J, R, T> gf;
  float bn[NC ? N - 1 : 1][4];  // B(n) of the other modes as left operands (NC)
  int i, g;

  __device__ __forceinline__ void init(const T* Bm, int lane) {
    i = lane & 15;
    g = lane >> 4;
    if constexpr (!FIB) gf.load(Bm, i, g);
    if constexpr (NC)
#pragma unroll
      for (int k = 0; k < N - 1; ++k)
#pragma unroll
        for (int s = 0; s < 4; ++s) bn[k][s] = nc.B[k][(4 * g + s) * R + i];
  }
  // slot i of the block at position p0 of an item ending before pe (clamped to its last element)
  __device__ __forceinline__ void index(int64_t p0, int64_t pe, Idx& a) const { index_at(min(p0 + i, pe - 1), a); }
  __device__ __forceinline__ void index_at(int64_t p, Idx& a) const {
    a.x = val[p];
    if constexpr (FIB) {
      a.o[0] = (uint32_t)fid[p];
    } else {
#pragma unroll
      for (int k = 0; k < N - 1; ++k) a.o[k] = (uint32_t)idx[(int64_t)k * nnz + p];
    }
  }
  __device__ __forceinline__ void gather(const Idx& a, Raw& r) const {
    if constexpr (FIB) {
      // fibers number up to nnz: 64-bit offsets
      const float* row = gfib + (int64_t)a.o[0] * J;
      r.s[0].load(row, (uint32_t)(Geo<J>::jbase(g) * sizeof(float)));
    } else if constexpr (NC) {
#pragma unroll
      for (int k = 0; k < N - 1; ++k) r.s[k].load(nc.A[k] + (int64_t)a.o[k] * 16, (uint32_t)(4 * g * sizeof(float)));
    } else {
#pragma unroll
      for (int k = 0; k < N - 1; ++k)
        r.s[k].load(cp.p[k], row_bytes<R, T>((int32_t)a.o[k]) + (uint32_t)(KR * g * sizeof(T)));
    }
  }
  // G of the block (zero in slots from nb on)
  __device__ __forceinline__ void form(const Raw& r, int nb, float (&G)[Geo<J>::NG]) const {
    const bool ok = i < nb;
    if constexpr (FIB) {
      r.s[0].widen(G);
#pragma unroll
      for (int k = 0; k < Geo<J>::NG; ++k) G[k] = ok ? G[k] : 0.f;
    } else {
      float w[KR];
      if constexpr (NC) {
#pragma unroll
        for (int k = 0; k < N - 1; ++k) {
          float av[4];
          r.s[k].widen(av);
          floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < 4; ++s) c = __builtin_amdgcn_mfma_f32_16x16x4f32(bn[k][s], av[s], c, 0, 0, 0);
#pragma unroll
          for (int s = 0; s < 4; ++s) w[s] = k == 0 ? c[s] : w[s] * c[s];
        }
      } else {
        r.s[0].widen(w);
#pragma unroll
        for (int k = 1; k < N - 1; ++k) {
          float t[KR];
          r.s[k].widen(t);
#pragma unroll
          for (int s = 0; s < KR; ++s) w[s] *= t[s];
        }
      }
#pragma unroll
      for (int s = 0; s < KR; ++s) w[s] = ok ? w[s] : 0.f;
      gf.form(w, G);
    }
  }
};

// The shared intermediate of Section 3.2: g_f = B(m) w_f once per mode-m
// fiber f (w_f = prod_{n != m} C(n)[i_n, :] is the same for every element of
// the fiber), formed by the same code as the per-element path, so the factor
// pass gives the same bits either way.  A wavefront takes kFiberBlocks blocks
// of 16 fibers and gathers one block ahead.
constexpr int kFiberBlocks = 4;

template <int N, int J, int R, class T>
__global__ __launch_bounds__(256) void k_fiber_g(const int32_t* __restrict__ fib_idx, int64_t nfib, CPtrs<N, T> cp,
                                                 const T* __restrict__ Bm, float* __restrict__ gfib) {
  using Src = Source<N, J, R, T, false, false>;
  Src src;
  src.nnz = nfib;
  src.cp = cp;
  src.init(Bm, threadIdx.x & 63);
  const int64_t f0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * (16 * kFiberBlocks);
  if (f0 >= nfib) return;
  auto index = [&](int64_t f, typename Src::Idx& a) {
    const int64_t p = min(f + src.i, nfib - 1);
#pragma unroll
    for (int k = 0; k < N - 1; ++k) a.o[k] = (uint32_t)fib_idx[(int64_t)k * nfib + p];
  };
  typename Src::Idx ix[kFiberBlocks];
  typename Src::Raw raw;
#pragma unroll
  for (int b = 0; b < kFiberBlocks; ++b) index(f0 + 16 * b, ix[b]);
  src.gather(ix[0], raw);
#pragma unroll
  for (int b = 0; b < kFiberBlocks; ++b) {
    const typename Src::Raw cur = raw;
    if (b + 1 < kFiberBlocks) src.gather(ix[b + 1], raw);
    float G[Geo<J>::NG];
    src.form(cur, 16, G);
    const int64_t f = f0 + 16 * b + src.i;
    if (f < nfib) {
      float* dst = gfib + f * J + Geo<J>::jbase(src.g);
      if constexpr (Geo<J>::NG == 2) {
        *reinterpret_cast<floatx2*>(dst) = floatx2{G[0], G[1]};
      } else {
#pragma unroll
        for (int k = 0; k < Geo<J>::NG; k += 4)
          *reinterpret_cast<floatx4*>(dst + k) = floatx4{G[k], G[k + 1], G[k + 2], G[k + 3]};
      }
    }
  }
}

// One block ready for its serial part, and (MAP) G by columns for the chunk map.
template <int J, bool MAP>
struct Block {
  float Gu[Geo<J>::NG], Gr[Geo<J>::NS], L[16], x;
  float Gc[MAP ? Geo<J>::JT : 1][4];  // G[4 g + v][jmap(jt, i)]
};

// LDS is private to the wavefront, which executes its accesses in order; the
// fence keeps the compiler from moving reads of other lanes' values up.
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// -gp tril(K, -1) of a block into LDS, by rows
template <int J>
__device__ __forceinline__ void store_l(const float (&G)[Geo<J>::NG], float gp, int i, int g, float* lds_l) {
  floatx4 K = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < Geo<J>::NG; ++k) K = __builtin_amdgcn_mfma_f32_16x16x4f32(G[k], G[k], K, 0, 0, 0);
  floatx4 Lw;
#pragma unroll
  for (int v = 0; v < 4; ++v) Lw[v] = 4 * g + v < i ? -gp * K[v] : 0.f;
  *reinterpret_cast<floatx4*>(lds_l + i * Geo<J>::LS + 4 * g) = Lw;
}

// G and K of a block into LDS: G by slots, and -gp tril(K, -1) by rows.
template <int J>
__device__ __forceinline__ void store_block(const float (&G)[Geo<J>::NG], float gp, int i, int g, float* lds_g,
                                            float* lds_l) {
  using Q = Geo<J>;
  float* grow = lds_g + i * Q::GS + Q::jbase(g);
  if constexpr (Q::NG == 2) {
    *reinterpret_cast<floatx2*>(grow) = floatx2{G[0], G[1]};
  } else {
#pragma unroll
    for (int k = 0; k < Q::NG; k += 4)
      *reinterpret_cast<floatx4*>(grow + k) = floatx4{G[k], G[k + 1], G[k + 2], G[k + 3]};
  }
  store_l<J>(G, gp, i, g, lds_l);
}

// The same out of LDS in the layouts of the serial part.  G of the state
// product is read back as well (not taken from the MFMA result), because
// inline assembly reads it.
template <int J, bool MAP>
__device__ __forceinline__ void load_block(const float* lds_g, const float* lds_l, int i, int g, Block<J, MAP>& blk) {
  using Q = Geo<J>;
  const float* grow = lds_g + i * Q::GS + Q::jbase(g);
  if constexpr (Q::NG == 2) {
    const floatx2 u = *reinterpret_cast<const floatx2*>(grow);
    blk.Gu[0] = u[0];
    blk.Gu[1] = u[1];
  } else {
#pragma unroll
    for (int k = 0; k < Q::NG; k += 4) {
      const floatx4 u = *reinterpret_cast<const floatx4*>(grow + k);
#pragma unroll
      for (int v = 0; v < 4; ++v) blk.Gu[k + v] = u[v];
    }
  }
  const float* gcol = lds_g + Q::sbase(g) * Q::GS + Q::jlane(i, g);
#pragma unroll
  for (int k = 0; k < Q::NS; ++k) blk.Gr[k] = gcol[k * Q::GS];
  const float* lrow = lds_l + i * Q::LS;
#pragma unroll
  for (int s = 0; s < 16; s += 4) {
    const floatx4 u = *reinterpret_cast<const floatx4*>(lrow + s);
#pragma unroll
    for (int v = 0; v < 4; ++v) blk.L[s + v] = u[v];
  }
  if constexpr (MAP) {
#pragma unroll
    for (int jt = 0; jt < Q::JT; ++jt) {
      const int j = Q::jmap(jt, i);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float q = lds_g[(4 * g + v) * Q::GS + max(j, 0)];
        blk.Gc[jt][v] = j >= 0 ? q : 0.f;
      }
    }
  }
}

template <int J, bool MAP>
__device__ __forceinline__ void prepare_block(const float (&G)[Geo<J>::NG], float x, int nb, float gp, int i, int g,
                                              WaveLds<J>& lds, Block<J, MAP>& blk) {
  wave_lds_fence();
  store_block<J>(G, gp, i, g, lds.G, lds.L);
  wave_lds_fence();
  load_block<J, MAP>(lds.G, lds.L, i, g, blk);
  blk.x = i < nb ? x : 0.f;
}

// The serial part of a block: a <- rho^nb (a + gp G^T e~); inv, inv_lo are
// those of the lane's slot.  The rows of A take their increments in FP64 and an
// e~ of one rounding: in FP32, as the state of a chunk map has them, the error of A over
// rows of 700 elements in a learning regime (lr = 1e-2) is 3.7e-8 where one
// step per element has 3.3e-8; so it is 3.3e-8.
template <int J, bool MAP>
__device__ __forceinline__ void step_block(const Block<J, MAP>& blk, float inv, float inv_lo, double gp,
                                           double rho_nb, double& a) {
  using Q = Geo<J>;
  const float af = rotate_state<J>((float)a);
  const float u = sum_rows(sum_halves(bsum<Q::NG>(af, blk.Gu)));
  const float res = scaled_residual(blk.x, inv, inv_lo, u);
  double d;
  if constexpr (MAP) {
    float f = sum_halves(bsum<Q::NS>(rotate_slots<J>(forward_substitute(res, blk.L)), blk.Gr));
    if constexpr (J < 32) f = sum_rows(f);
    d = (double)f;
  } else {
    double Gd[Q::NS];
#pragma unroll
    for (int k = 0; k < Q::NS; ++k) Gd[k] = (double)blk.Gr[k];
    d = sum_halves(bsum<Q::NS>((double)rotate_slots<J>(res + solve_rest(res, blk.L)), Gd));
    if constexpr (J < 32) d = sum_rows(d);
  }
  a = rho_nb * fma(gp, d, a);
}

// T = (I + gp tril(K, -1))^-1 of a block, as the left operand of T Y: lane
// (i, g) gets T[i][4 g + v].  lds.L holds -gp tril(K, -1).  The two diagonal
// 8 x 8 blocks are inverted by substitution, lanes 0-31 the first and lanes
// 32-63 the second, so that one row broadcast serves both (28 FMAs; the whole
// 16 x 16 matrix by substitution takes 120); then T21 = T22 (-L21) T11, an
// entry per lane, through LDS.  T12 = 0 is stored once per item.
template <int J>
__device__ __forceinline__ void block_inverse(WaveLds<J>& lds, int lane, float (&Ti)[4]) {
  constexpr int LS = Geo<J>::LS;
  const int i = lane & 15, g = lane >> 4, h8 = 8 * (lane >> 5), r8 = i & 7;
  auto row8 = [](const float* p, float (&o)[8]) {
    const floatx4 u = *reinterpret_cast<const floatx4*>(p), v = *reinterpret_cast<const floatx4*>(p + 4);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      o[k] = u[k];
      o[4 + k] = v[k];
    }
  };
  float y[8], L[8];
  row8(lds.L + (h8 + r8) * LS + h8, L);
#pragma unroll
  for (int s = 0; s < 8; ++s) y[s] = s == r8 ? 1.f : 0.f;
  asm("s_nop 4" : "+v"(y[7]));
  inverse_step<7>(y, L);
  inverse_step<6>(y, L);
  inverse_step<5>(y, L);
  inverse_step<4>(y, L);
  inverse_step<3>(y, L);
  inverse_step<2>(y, L);
  inverse_step<1>(y, L);
  float* trow = lds.T + (h8 + r8) * LS + h8;
  *reinterpret_cast<floatx4*>(trow) = floatx4{y[0], y[1], y[2], y[3]};
  *reinterpret_cast<floatx4*>(trow + 4) = floatx4{y[4], y[5], y[6], y[7]};
  wave_lds_fence();
  const int k = lane >> 3, s = lane & 7;
  float q[8], acc = 0.f;
  row8(lds.L + (8 + k) * LS, q);
#pragma unroll
  for (int u = 0; u < 8; ++u) acc = fmaf(q[u], lds.T[u * LS + s], acc);
  lds.P[k * 12 + s] = acc;
  wave_lds_fence();
  acc = 0.f;
  row8(lds.T + (8 + k) * LS + 8, q);
#pragma unroll
  for (int u = 0; u < 8; ++u) acc = fmaf(q[u], lds.P[u * 12 + s], acc);
  lds.T[(8 + k) * LS + s] = acc;
  wave_lds_fence();
  const floatx4 t = *reinterpret_cast<const floatx4*>(lds.T + i * LS + 4 * g);
#pragma unroll
  for (int v = 0; v < 4; ++v) Ti[v] = t[v];
}

// The chunk map's block, a -> rho^T (I + Nm) a + v with Nm = prod (I - gp g g^T) - I:
//     Nm <- Nm - gp G^T (I + gp tril(K, -1))^-1 (G + G Nm).
// Nm is kept as MFMA results, rows and columns in jmap order: row 4 g + v of
// tile jt, column i of tile ct.  (Nm is M - I so that the small updates are
// not absorbed.)
template <int J>
__device__ __forceinline__ void map_block(const Block<J, true>& blk, WaveLds<J>& lds, float gp, int lane,
                                          floatx4 (&Nm)[Geo<J>::JT][Geo<J>::JT]) {
  using Q = Geo<J>;
  float Ti[4];
  block_inverse<J>(lds, lane, Ti);
#pragma unroll
  for (int ct = 0; ct < Q::JT; ++ct) {
    floatx4 Y = {blk.Gc[ct][0], blk.Gc[ct][1], blk.Gc[ct][2], blk.Gc[ct][3]};
#pragma unroll
    for (int k = 0; k < Q::NG; ++k)
      Y = __builtin_amdgcn_mfma_f32_16x16x4f32(blk.Gu[k], Nm[k / Q::VJ][ct][k % Q::VJ], Y, 0, 0, 0);
    floatx4 Z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 4; ++v) Z = __builtin_amdgcn_mfma_f32_16x16x4f32(Ti[v], Y[v], Z, 0, 0, 0);
    float Zs[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) Zs[v] = -gp * Z[v];
#pragma unroll
    for (int jt = 0; jt < Q::JT; ++jt)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        Nm[jt][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(blk.Gc[jt][v], Zs[v], Nm[jt][ct], 0, 0, 0);
  }
}

// What every item of a launch reads.
template <int N, int J, int R, class T, bool FIB, bool NC>
struct FactorArgs {
  const int32_t* idx;
  int64_t nnz;
  const float* val;
  CPtrs<N, T> cp;
  const T* Bm;
  float* Am;
  float* hvec;
  const int32_t* fid;
  const float* gfib;
  NoC<N> nc;
  float* maps;         // chunk maps, or the relaxed chunks' increments
  double* map_scale;
  const int64_t* row_ptr;
  double rho, gp;
  RhoPow pw;
  int block;           // elements per block (16; 1 where rho^-15 would leave the FP32 range)
  int quads;           // items taken four to a wavefront: kQuadChunks, kQuadRows
};

enum { ITEM_CHAIN, ITEM_RELAXED, ITEM_MAP };
enum { kQuadChunks = 1, kQuadRows = 2 };

// One work item on one wavefront.
//  CHAIN: the row (or the head of a long row) is updated in place; a head
//    writes the row's head vector, or A(m) itself when hvec is null (the
//    relaxed passes).
//  RELAXED: a chunk of a long row under FT_RELAXED runs from the row as its
//    head left it, a_H (in A(m); the merge that follows is the only other
//    writer) and stores its increment beyond the decay of a_H, weighted by the
//    decay of the row's later elements,
//        rho^T (a - rho^len a_H),   T = elements of the row after the chunk,
//    and the sum of ||g||^2 over its steps, J + 1 floats per chunk slot.
//  MAP: a chunk's affine map a -> rho^len (I + Nm) a + v; v is the state
//    reached from a = 0.
template <int KIND, int N, int J, int R, class T, bool FIB, bool NC>
__device__ __forceinline__ void factor_item(const FItem& it, const FactorArgs<N, J, R, T, FIB, NC>& F,
                                            WaveLds<J>& lds) {
  using Q = Geo<J>;
  constexpr bool MAP = KIND == ITEM_MAP;
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  if (it.len <= 0) return;
  Source<N, J, R, T, FIB, NC> src;
  src.idx = F.idx;
  src.nnz = F.nnz;
  src.val = F.val;
  src.cp = F.cp;
  src.fid = F.fid;
  src.gfib = F.gfib;
  src.nc = F.nc;
  src.init(F.Bm, lane);
  const int64_t pe = it.start + it.len;
  const int bs = F.block;
  const int jl = Q::jlane(i, g);
  const float gpf = (float)F.gp;
  const float inv = F.pw.inv[i], inv_lo = F.pw.inv_lo[i];
  double a = 0.0;
  if constexpr (!MAP) a = (double)F.Am[(int64_t)it.row * J + jl];
  floatx4 Nm[Q::JT][Q::JT];
  if constexpr (MAP) {
#pragma unroll
    for (int jt = 0; jt < Q::JT; ++jt)
#pragma unroll
      for (int ct = 0; ct < Q::JT; ++ct) Nm[jt][ct] = floatx4{0.f, 0.f, 0.f, 0.f};
    lds.T[(lane >> 3) * Q::LS + 8 + (lane & 7)] = 0.f;  // T12
  }
  float gg = 0.f;  // sum of ||g||^2 (RELAXED), this lane's part
  // Pipeline: the gathers of block b + 1 and the indices of block b + 2 are in
  // flight while block b is formed, and block b is formed (MFMA, LDS) beside
  // the serial part of block b - 1 (VALU).
  typename Source<N, J, R, T, FIB, NC>::Idx ix0, ix1;
  typename Source<N, J, R, T, FIB, NC>::Raw raw;
  src.index(it.start, pe, ix0);
  src.gather(ix0, raw);
  src.index(min(it.start + bs, pe - 1), pe, ix1);
  Block<J, MAP> cur;
  auto form = [&](int64_t p, Block<J, MAP>& blk) {
    const int nb = (int)min<int64_t>(bs, pe - p);
    float G[Q::NG];
    src.form(raw, nb, G);
    const float x = ix0.x;
    ix0 = ix1;
    src.gather(ix0, raw);
    src.index(min(p + 2 * bs, pe - 1), pe, ix1);
    if constexpr (KIND == ITEM_RELAXED)
#pragma unroll
      for (int k = 0; k < Q::NG; ++k) gg = fmaf(G[k], G[k], gg);
    prepare_block<J, MAP>(G, x, nb, gpf, i, g, lds, blk);
  };
  form(it.start, cur);
  int64_t p = it.start;
  if constexpr (MAP) {
    // (a map's own products keep the matrix cores busy: its blocks are formed one after another, which
    // leaves registers for three wavefronts per SIMD)
    for (;;) {
      step_block<J, MAP>(cur, inv, inv_lo, F.gp, F.pw.p[min<int64_t>(bs, pe - p)], a);
      map_block<J>(cur, lds, gpf, lane, Nm);
      p += bs;
      if (p >= pe) break;
      form(p, cur);
    }
  } else {
    // (two blocks in turn: copying one to the other is 30 instructions)
    const double rb = F.pw.p[bs];
    Block<J, MAP> nxt;
    while (p + 2 * bs < pe) {
      form(p + bs, nxt);
      step_block<J, MAP>(cur, inv, inv_lo, F.gp, rb, a);
      form(p + 2 * bs, cur);
      step_block<J, MAP>(nxt, inv, inv_lo, F.gp, rb, a);
      p += 2 * bs;
    }
    if (p + bs < pe) {
      form(p + bs, nxt);
      step_block<J, MAP>(cur, inv, inv_lo, F.gp, rb, a);
      cur = nxt;
      p += bs;
    }
    step_block<J, MAP>(cur, inv, inv_lo, F.gp, F.pw.p[pe - p], a);
  }

  // lanes that hold a copy of the state's element jl write it once
  const bool writer = J >= 32 ? g < 2 : g == 0 && i < J;
  if constexpr (KIND == ITEM_CHAIN) {
    float* dst = it.kind == ITEM_LIGHT || F.hvec == nullptr ? F.Am + (int64_t)it.row * J : F.hvec + (int64_t)it.slot * J;
    if (writer) dst[jl] = (float)a;
  } else if constexpr (KIND == ITEM_RELAXED) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) gg += __shfl_xor(gg, off);
    const double own = pow(F.rho, (double)it.len);
    const double after = pow(F.rho, (double)(F.row_ptr[it.row + 1] - pe));
    float* dst = F.maps + (int64_t)it.slot * (J + 1);
    if (writer) dst[jl] = (float)(after * (a - own * (double)F.Am[(int64_t)it.row * J + jl]));
    if (lane == 0) dst[J] = gg;
  } else {
    float* dst = F.maps + (int64_t)it.slot * (J * J + J);  // column-major
#pragma unroll
    for (int ct = 0; ct < Q::JT; ++ct) {
      const int c = Q::jmap(ct, i);
#pragma unroll
      for (int jt = 0; jt < Q::JT; ++jt) {
        const int r = Q::jmap(jt, 4 * g);
        if constexpr (Q::VJ == 4)
          *reinterpret_cast<floatx4*>(dst + c * J + r) = Nm[jt][ct];
        else if (c >= 0)
          *reinterpret_cast<floatx2*>(dst + c * J + r) = floatx2{Nm[jt][ct][0], Nm[jt][ct][1]};
      }
    }
    if (writer) dst[J * J + jl] = (float)a;
    if (lane == 0) F.map_scale[it.slot] = pow(F.rho, (double)it.len);
  }
}

// Four items on one wavefront (J <= 16), 16 lanes each, one step per element:
//     Nm <- Nm - gp g (g + Nm^T g)^T,   a <- a + gp (rho^-t x - a.g) g,
// a decaying by rho^16 at the end of a block (t: the step within it); lane l
// of a row of 16 holds column l of Nm (MAP) and element l of a (FP64, MAP:
// from a = 0).  Only where rho >= 1/2, as with blocks of 16.  G comes from the products that factor_item takes
// it from, a chunk's block after the other, through LDS, so that g is the same
// to the bit.  A step is 2 J row broadcasts and about 14 more instructions for
// four chunks, where a block of 16 elements on the matrix cores costs one
// chunk 20 of their instructions and 140 others, three quarters of them the
// same in the four rows of lanes: more work per second, but a chunk takes
// about twice as long.
template <int J>
struct __align__(16) QuadLds {
  static constexpr int S = 16 * Geo<J>::GS + 16;  // one chunk's block; the 16 spread the rows over the banks
  float G[4 * S];
};

template <int KIND, int N, int J, int R, class T, bool FIB, bool NC>
__device__ __forceinline__ void quad_items(const FItem* __restrict__ items, int64_t k0, int64_t n_items,
                                           const FactorArgs<N, J, R, T, FIB, NC>& F, QuadLds<J>& lds) {
  static_assert(J <= 16, "a row of 16 lanes holds the state");
  using Q = Geo<J>;
  using Src = Source<N, J, R, T, FIB, NC>;
  constexpr bool MAP = KIND == ITEM_MAP;
  // all four gathers ahead of the steps where they fit in registers, else two at a time
  constexpr bool PIPE = Src::NI * Src::RK * (int)sizeof(typename Src::E) <= 48;
  constexpr int NR = PIPE ? 4 : 2;
  if (k0 >= n_items) return;
  const int lane = threadIdx.x & 63, l = lane & 15, row = lane >> 4;
  FItem it{0, 0, 0, 0, 0};
  if (k0 + row < n_items) it = items[k0 + row];
  Src src;
  src.idx = F.idx;
  src.nnz = F.nnz;
  src.val = F.val;
  src.cp = F.cp;
  src.fid = F.fid;
  src.gfib = F.gfib;
  src.nc = F.nc;
  src.init(F.Bm, lane);
  int most = it.len;
  most = max(most, __shfl_xor(most, 16));
  most = __builtin_amdgcn_readfirstlane(max(most, __shfl_xor(most, 32)));
  double a = 0.0;
  if constexpr (!MAP)
    if (it.len > 0) a = (double)F.Am[(int64_t)it.row * J + l % J];
  float Nc[MAP ? J : 1];
#pragma unroll
  for (int j = 0; j < (MAP ? J : 1); ++j) Nc[j] = 0.f;
  float gg = 0.f;
  const float gpf = (float)F.gp;
  const double rhol = F.pw.p[l + 1];
  // slot l of the block at t0 of this row's chunk (clamped to its last element; an empty item reads element 0)
  auto index = [&](int t0, typename Src::Idx& ix) {
    src.index_at(it.start + min(t0 + l, max(it.len - 1, 0)), ix);
  };
  auto gather = [&](const typename Src::Idx& ix, int q, typename Src::Raw& r) {
    typename Src::Idx o;
#pragma unroll
    for (int k = 0; k < Src::NI; ++k) o.o[k] = (uint32_t)__shfl((int)ix.o[k], 16 * q + l);
    src.gather(o, r);
  };
  typename Src::Idx ix0, ix1;
  typename Src::Raw raw[NR];
  index(0, ix0);
#pragma unroll
  for (int q = 0; q < NR; ++q) gather(ix0, q, raw[q]);
  index(16, ix1);
  for (int t0 = 0; t0 < most; t0 += 16) {
    wave_lds_fence();
    static_for<0, 4>([&](auto QQ) {
      constexpr int q = decltype(QQ)::value;
      float G[Q::NG];
      src.form(raw[q % NR], min(max(__builtin_amdgcn_readlane(it.len, 16 * q) - t0, 0), 16), G);
      if constexpr (q + NR < 4) gather(ix0, q + NR, raw[q % NR]);
      if constexpr (KIND == ITEM_RELAXED) {
        float z = 0.f;
#pragma unroll
        for (int k = 0; k < Q::NG; ++k) z = fmaf(G[k], G[k], z);
        z = sum_rows(sum_halves(z));
        gg += row == q ? z : 0.f;
      }
      float* grow = lds.G + q * QuadLds<J>::S + l * Q::GS + Q::jbase(row);
#pragma unroll
      for (int k = 0; k < Q::NG; k += 2) *reinterpret_cast<floatx2*>(grow + k) = floatx2{G[k], G[k + 1]};
    });
    const float x = ix0.x;
    ix0 = ix1;
#pragma unroll
    for (int q = 0; q < NR; ++q) gather(ix0, q, raw[q]);
    index(t0 + 32, ix1);
    wave_lds_fence();
    float gs[16];
#pragma unroll
    for (int s = 0; s < 16; ++s) gs[s] = lds.G[row * QuadLds<J>::S + s * Q::GS + l % J];
    static_for<0, 16>([&](auto S) {
      constexpr int s = decltype(S)::value;
      const float g = gs[s];  // 0 past the end of the chunk
      if constexpr (MAP) {
        float h = g;
        dot_bcast<J>(h, g, Nc);
        axpy_bcast<J>(Nc, g, -gpf * h);
      }
      const float e = gpf * scaled_residual(bcast16<s>(x), F.pw.inv[s], F.pw.inv_lo[s], group_sum<J>((float)a * g));
      a = fma((double)e, (double)g, a);
    });
    const int nb = it.len - t0;
    const double part = __shfl(rhol, 16 * row + min(max(nb - 1, 0), 15));
    a *= nb >= 16 ? F.pw.p[16] : nb > 0 ? part : 1.0;
  }
  if (it.len <= 0) return;
  if constexpr (KIND == ITEM_CHAIN) {
    float* dst = it.kind == ITEM_LIGHT || F.hvec == nullptr ? F.Am + (int64_t)it.row * J : F.hvec + (int64_t)it.slot * J;
    if (l < J) dst[l] = (float)a;
  } else if constexpr (KIND == ITEM_RELAXED) {
    gg = group_sum<16>(gg);
    const double own = pow(F.rho, (double)it.len);
    const double after = pow(F.rho, (double)(F.row_ptr[it.row + 1] - (it.start + it.len)));
    float* dst = F.maps + (int64_t)it.slot * (J + 1);
    if (l < J) dst[l] = (float)(after * (a - own * (double)F.Am[(int64_t)it.row * J + l]));
    if (l == 0) dst[J] = gg;
  } else {
    float* dst = F.maps + (int64_t)it.slot * (J * J + J);  // column-major
    if (l < J) {
#pragma unroll
      for (int j = 0; j < J; j += 4)
        *reinterpret_cast<floatx4*>(dst + l * J + j) = floatx4{Nc[j], Nc[j + 1], Nc[j + 2], Nc[j + 3]};
      dst[J * J + l] = (float)a;
    }
    if (l == 0) F.map_scale[it.slot] = pow(F.rho, (double)it.len);
  }
}

// A long row, or the head of one, by a workgroup: wavefronts 1 to 3 form its
// blocks in turn (gathers, MFMA) and leave them in LDS, a round of three ahead
// of wavefront 0, which only takes the serial parts.  A lone wavefront issues
// an instruction about every five cycles, so a chain that also forms its blocks
// takes 1900 cycles per block (J = 8) to 2400 (J = 32); the serial part alone
// is a third of that, and the head of a long row is what a launch waits for.
// G and x are stored as FP64, so that the chain converts neither.  (T = (I + gp
// tril(K, -1))^-1 formed by wavefronts 1 to 3 in place of the substitution is
// slower where the launch is full of such rows: 1000 rows of 8000 elements,
// J = 32, g shared, 318 us against 283; 240 with the sums of a block in FP32.)
template <int J>
struct __align__(16) TeamLds {
  static constexpr int GS = J + 2;  // row stride of G in doubles
  double G[2][3][16 * GS];
  double x[2][3][16];              // rho^-t x
  float L[2][3][16 * Geo<J>::LS];
};

template <int J>
struct TeamBlock {
  double Gu[Geo<J>::NG], Gr[Geo<J>::NS], x;
  float L[16];
  __device__ __forceinline__ void load(const TeamLds<J>& lds, int h, int q, int i, int g) {
    using Q = Geo<J>;
    const double* grow = lds.G[h][q] + i * TeamLds<J>::GS + Q::jbase(g);
#pragma unroll
    for (int k = 0; k < Q::NG; ++k) Gu[k] = grow[k];
    const double* gcol = lds.G[h][q] + Q::sbase(g) * TeamLds<J>::GS + Q::jlane(i, g);
#pragma unroll
    for (int k = 0; k < Q::NS; ++k) Gr[k] = gcol[k * TeamLds<J>::GS];
    const float* lrow = lds.L[h][q] + i * Q::LS;
#pragma unroll
    for (int s = 0; s < 16; s += 4) {
      const floatx4 u = *reinterpret_cast<const floatx4*>(lrow + s);
#pragma unroll
      for (int v = 0; v < 4; ++v) L[s + v] = u[v];
    }
    x = lds.x[h][q][i];
  }
  __device__ __forceinline__ void step(double gp, double rho_nb, double& a) const {
    using Q = Geo<J>;
    const double r = x - sum_rows(sum_halves(bsum<Q::NG>(rotate_state<J>(a), Gu)));
    const double e = r + (double)solve_rest((float)r, L);
    double d = sum_halves(bsum<Q::NS>(rotate_slots<J>(e), Gr));
    if constexpr (J < 32) d = sum_rows(d);
    a = rho_nb * fma(gp, d, a);
  }
};

template <int N, int J, int R, class T, bool FIB, bool NC>
__device__ __forceinline__ void team_item(const FItem& it, const FactorArgs<N, J, R, T, FIB, NC>& F, TeamLds<J>& lds) {
  using Q = Geo<J>;
  using Src = Source<N, J, R, T, FIB, NC>;
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (it.len <= 0) return;
  const int64_t pe = it.start + it.len;
  const int bs = F.block;
  const int nblk = (it.len + bs - 1) / bs, rounds = (nblk + 2) / 3;
  const int jl = Q::jlane(i, g);
  if (wave == 0) {
    __builtin_amdgcn_s_setprio(3);
    double a = (double)F.Am[(int64_t)it.row * J + jl];
    const double rb = F.pw.p[bs];
    for (int r = 0; r <= rounds; ++r) {
      if (r > 0) {
        const int h = (r - 1) & 1, b0 = 3 * (r - 1);
        TeamBlock<J> blk[2];
        blk[0].load(lds, h, 0, i, g);
        static_for<0, 3>([&](auto S) {
          constexpr int q = decltype(S)::value;
          if (b0 + q < nblk) {
            // (a slot past the last block holds an old one, which is not used)
            if constexpr (q < 2) blk[(q + 1) & 1].load(lds, h, q + 1, i, g);
            const int64_t left = pe - it.start - (int64_t)(b0 + q) * bs;
            blk[q & 1].step(F.gp, left >= bs ? rb : F.pw.p[left], a);
          }
        });
      }
      __syncthreads();
    }
    __builtin_amdgcn_s_setprio(0);
    float* dst = it.kind == ITEM_LIGHT || F.hvec == nullptr ? F.Am + (int64_t)it.row * J : F.hvec + (int64_t)it.slot * J;
    if (J >= 32 ? g < 2 : g == 0 && i < J) dst[jl] = (float)a;
    return;
  }
  Src src;
  src.idx = F.idx;
  src.nnz = F.nnz;
  src.val = F.val;
  src.cp = F.cp;
  src.fid = F.fid;
  src.gfib = F.gfib;
  src.nc = F.nc;
  src.init(F.Bm, lane);
  const float gpf = (float)F.gp;
  const double inv = (double)F.pw.inv[i] + (double)F.pw.inv_lo[i];
  const int step = 3 * bs, w = wave - 1;
  int64_t p = it.start + (int64_t)w * bs;
  typename Src::Idx ix0, ix1;
  typename Src::Raw raw;
  src.index(min(p, pe - 1), pe, ix0);
  src.gather(ix0, raw);
  src.index(min(p + step, pe - 1), pe, ix1);
  for (int r = 0; r <= rounds; ++r) {
    if (p < pe) {
      const int nb = (int)min<int64_t>(bs, pe - p), h = r & 1;
      float G[Q::NG];
      src.form(raw, nb, G);
      const float x = ix0.x;
      ix0 = ix1;
      src.gather(ix0, raw);
      src.index(min(p + 2 * step, pe - 1), pe, ix1);
      double* grow = lds.G[h][w] + i * TeamLds<J>::GS + Q::jbase(g);
#pragma unroll
      for (int k = 0; k < Q::NG; ++k) grow[k] = (double)G[k];
      if (g == 0) lds.x[h][w][i] = i < nb ? (double)x * inv : 0.0;
      store_l<J>(G, gpf, i, g, lds.L[h][w]);
      p += step;
    }
    __syncthreads();
  }
}

// A pack: a block of 16 slots shared by whole short rows.  The rows' steps are
// independent, so K is masked to pairs of one row; each slot reads its own
// row's state, and the rows' sums of e~_t g_t are one product over the slots,
// Delta^T = G^T (e~_s [row s = row t]), in FP64 as the steps of a longer row.  (A row of five elements in a block of
// its own costs as much as one of 16: order 4, 300k such rows, J = R = 32,
// 554 -> 253 us per pass; Netflix-shaped 5M mode 0, J = R = 16: 279 -> 171.)  Rows share sums in
// which another row's terms carry a factor 0, so a pack with a value that is
// not finite is left alone (false): its rows are then taken one by one.
template <int N, int J, int R, class T, bool FIB, bool NC>
__device__ __forceinline__ bool pack_item(const Pack* __restrict__ pk, const FactorArgs<N, J, R, T, FIB, NC>& F,
                                          WaveLds<J>& lds) {
  using Q = Geo<J>;
  using Src = Source<N, J, R, T, FIB, NC>;
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  Src src;
  src.idx = F.idx;
  src.nnz = F.nnz;
  src.val = F.val;
  src.cp = F.cp;
  src.fid = F.fid;
  src.gfib = F.gfib;
  src.nc = F.nc;
  src.init(F.Bm, lane);
  const int n = pk->n;
  typename Src::Idx ix;
  typename Src::Raw raw;
  src.index(pk->start, pk->start + n, ix);
  src.gather(ix, raw);
  const int row = pk->row[i], at = pk->at[i];
  const int4 row4 = *reinterpret_cast<const int4*>(&pk->row[4 * g]);
  const int rows[4] = {row4.x, row4.y, row4.z, row4.w};  // of slots 4 g + v
  float* arow = F.Am + (int64_t)row * J + Q::jbase(g);
  float as[Q::NG];
#pragma unroll
  for (int k = 0; k < Q::NG; ++k) as[k] = arow[k];
  float G[Q::NG];
  src.form(raw, n, G);
  float u = G[0] * as[0];
#pragma unroll
  for (int k = 1; k < Q::NG; ++k) u = fmaf(G[k], as[k], u);
  u = sum_rows(sum_halves(u));
  wave_lds_fence();
  float* grow = lds.G + i * Q::GS + Q::jbase(g);
#pragma unroll
  for (int k = 0; k < Q::NG; k += 2) *reinterpret_cast<floatx2*>(grow + k) = floatx2{G[k], G[k + 1]};
  floatx4 K = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < Q::NG; ++k) K = __builtin_amdgcn_mfma_f32_16x16x4f32(G[k], G[k], K, 0, 0, 0);
  const float gpf = (float)F.gp;
  floatx4 Lw;
#pragma unroll
  for (int v = 0; v < 4; ++v) Lw[v] = 4 * g + v < i && rows[v] == row ? -gpf * K[v] : 0.f;
  *reinterpret_cast<floatx4*>(lds.L + i * Q::LS + 4 * g) = Lw;
  wave_lds_fence();
  float L[16];
#pragma unroll
  for (int s = 0; s < 16; s += 4) {
    const floatx4 x = *reinterpret_cast<const floatx4*>(lds.L + i * Q::LS + s);
#pragma unroll
    for (int v = 0; v < 4; ++v) L[s + v] = x[v];
  }
  // rho^-t and rho^count by the slot's place in its row: lane t holds the t-th power
  const float inv = __shfl(F.pw.inv[i], at & 15), inv_lo = __shfl(F.pw.inv_lo[i], at & 15);
  const double rc = __shfl(F.pw.p[i < 15 ? i + 1 : 16], max((at >> 8) - 1, 0));
  const float res = scaled_residual(i < n ? ix.x : 0.f, inv, inv_lo, u);
  const float e = res + solve_rest(res, L);
  if (__any(!(fabsf(e) <= 3.402823466e38f))) return false;
  const float er = rotate_rows<12, 8, 4>(e);  // broadcast v gives lane row g slot 4 g + v
  doublex4 d[Q::JT];
#pragma unroll
  for (int jt = 0; jt < Q::JT; ++jt) d[jt] = doublex4{0.0, 0.0, 0.0, 0.0};
  static_for<0, 4>([&](auto VV) {
    constexpr int v = decltype(VV)::value;
    const float ev = bcast16<v>(er);
    const double em = rows[v] == row ? (double)ev : 0.0;
#pragma unroll
    for (int jt = 0; jt < Q::JT; ++jt) {
      const int j = Q::jmap(jt, 4 * (i & 3) + (i >> 2));  // (row 4 v + g of an FP64 result is in lanes of row g)
      const float q = lds.G[(4 * g + v) * Q::GS + max(j, 0)];
      d[jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(j >= 0 ? (double)q : 0.0, em, d[jt], 0, 0, 0);
    }
  });
  if ((at & 255) == 0 && i < n) {
#pragma unroll
    for (int k = 0; k < Q::NG; ++k)
      arow[k] = (float)(rc * fma(F.gp, d[k / Q::VJ][k % Q::VJ], (double)as[k]));
  }
  return true;
}

// LDS of a workgroup: a part of its own for each wavefront (a workgroup at the
// end of the rows has wavefronts with four rows beside others with a pack), or
// all of it for a team.
template <int J, bool QUAD>
union SlotLds {
  WaveLds<J> wave;
  QuadLds<J> quad;
};
template <int J>
union SlotLds<J, false> {
  WaveLds<J> wave;
};
template <int J, bool QUAD = false>
union FactorLds {
  SlotLds<J, QUAD> slot[4];
  TeamLds<J> team;
};

// Entry k of the in-place items that a wavefront takes, from item k0 on: a row
// (or four), or past the rows a pack.
template <bool QUAD, int N, int J, int R, class T, bool FIB, bool NC>
__device__ __forceinline__ void wave_items(int64_t k, int64_t k0, const FItem* __restrict__ items, int64_t n_items,
                                           const Pack* __restrict__ packs, int64_t n_packs,
                                           const FactorArgs<N, J, R, T, FIB, NC>& F, FactorLds<J, QUAD>& lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int64_t rows = n_items - k0;
  if constexpr (QUAD) {
    if (F.quads & kQuadRows) {
      rows = (rows + 3) / 4;
      if (k < rows) {
        quad_items<ITEM_CHAIN>(items, k0 + 4 * k, n_items, F, lds.slot[wave].quad);
        return;
      }
    }
  }
  FItem it{0, 0, 0, 0, ITEM_LIGHT};
  const Pack* pk = nullptr;
  int t = 0;
  if (k < rows) {
    it = items[k0 + k];
  } else {
    if (k - rows >= n_packs) return;
    pk = packs + (k - rows);
    if (pack_item(pk, F, lds.slot[wave].wave)) return;
  }
  for (;;) {
    if (pk) {
      it.start = pk->start + t;
      it.len = pk->at[t] >> 8;
      it.row = pk->row[t];
      t += it.len;
    }
    factor_item<ITEM_CHAIN>(it, F, lds.slot[wave].wave);
    if (!pk || t >= pk->n) return;
  }
}

// Chunks of a launch that a workgroup takes: one per wavefront, or four.
template <int KIND, bool QUAD, int N, int J, int R, class T, bool FIB, bool NC>
__device__ __forceinline__ void chunk_items(int64_t b, const FItem* __restrict__ items, int64_t n_items,
                                            const FactorArgs<N, J, R, T, FIB, NC>& F, FactorLds<J, QUAD>& lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t k = b * 4 + wave;
  if constexpr (QUAD) {
    if (F.quads & kQuadChunks) {
      quad_items<KIND>(items, 4 * k, n_items, F, lds.slot[wave].quad);
      return;
    }
  }
  if (k < n_items) factor_item<KIND>(items[k], F, lds.slot[wave].wave);
}

// In-place items alone: the first `teams` workgroups take a long row each, the
// items after the padded list of those follow, one or four per wavefront; the
// hardware dispatcher balances the items (the lists are sorted by length, so
// that a workgroup's end together).
template <bool QUAD, int N, int J, int R, class T, bool FIB, bool NC = false>
__global__ __launch_bounds__(256) void k_factor_apply(const FItem* __restrict__ items, int64_t n_items, int64_t teams,
                                                      const Pack* __restrict__ packs, int64_t n_packs,
                                                      FactorArgs<N, J, R, T, FIB, NC> F) {
  __shared__ FactorLds<J, QUAD> lds;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b = block_id();
  if (b < teams) {
    team_item(items[b], F, lds.team);
    return;
  }
  wave_items((b - teams) * 4 + wave, (teams + 3) / 4 * 4, items, n_items, packs, n_packs, F, lds);
}

// Chunks of long rows: their maps, or (RELAXED) their increments.
template <int KIND, bool QUAD, int N, int J, int R, class T, bool FIB, bool NC = false>
__global__ __launch_bounds__(256, KIND == ITEM_MAP ? 3 : 1) void k_factor_compose(const FItem* __restrict__ items,
                                                                                  int64_t n_items,
                                                                                  FactorArgs<N, J, R, T, FIB, NC> F) {
  __shared__ FactorLds<J, QUAD> lds;
  chunk_items<KIND>(block_id(), items, n_items, F, lds);
}

// The in-place items and the chunk maps of one exact factor pass in one
// launch.  They are independent (a map starts from the identity, not from
// its row's head).  The first `teams` workgroups take the heads of the long
// rows, the next map_blocks the chunk maps, the rest the short rows: the long
// serial heads start at once and run while the maps keep the SIMDs busy, and
// the short items fill in where the maps run out.
template <bool QUAD, int N, int J, int R, class T, bool FIB, bool NC = false>
__global__ __launch_bounds__(256, 3) void k_factor_fused(int64_t teams, int64_t map_blocks,
                                                      const FItem* __restrict__ apply_items, int64_t n_apply,
                                                      const FItem* __restrict__ compose_items, int64_t n_compose,
                                                      const Pack* __restrict__ packs, int64_t n_packs,
                                                      FactorArgs<N, J, R, T, FIB, NC> F) {
  __shared__ FactorLds<J, QUAD> lds;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b = block_id();
  if (b < teams) {
    team_item(apply_items[b], F, lds.team);
  } else if (b < teams + map_blocks) {
    chunk_items<ITEM_MAP>(b - teams, compose_items, n_compose, F, lds);
  } else {
    wave_items((b - teams - map_blocks) * 4 + wave, (teams + 3) / 4 * 4, apply_items, n_apply, packs, n_packs, F, lds);
  }
}

// Fold `count` consecutive maps (earliest first) into one, in order:
//   (s2, N2, v2) o (s1, N1, v1) = (s1 s2, N1 + N2 + N2 N1, s2 (v1 + N2 v1) + v2),
// with s = rho^length kept in FP64.  Only rows with more maps than the last
// fold takes in sequence (below) pass through here.
//
// A wavefront per fold and 16 columns: the columns of the running map are
// independent of each other, stay in MFMA results and are the right operand of
// the next product as they are; each later map is read as the left operand and
// once in the layout of the results, one map ahead.  What bounds it is the
// latency of this chain (16 MFMA of 32 cycles per map at J = 32) and of the
// launches, so a row has few levels: 16 maps per fold, and one launch for all
// last folds.  Against a tree in LDS by a workgroup and a last fold per level,
// us per pass: J = 32 (rows of up to 900 maps) 84 -> 31, J = 16 38 -> 20.
constexpr int kMaxFanin = 16;

template <int J>
struct MapRegs {
  static constexpr int JT = (J + 15) / 16;
  floatx4 d[JT];       // rows 16 jt + 4 g + v, column 16 ct + i (result layout)
  float a[JT][JT][4];  // row 16 it + i, columns 16 jt + 4 g + v (left operand)
  float v[JT];         // vector, entry 16 it + i, every row of 16 lanes alike
  double s;
  __device__ __forceinline__ void load(const float* __restrict__ maps, const double* __restrict__ scale, int64_t slot,
                                       int ct, int i, int g, bool left) {
    const float* m = maps + slot * (J * J + J);
    const bool ok = J >= 16 || (i < J && 4 * g < J);  // J = 8: a quarter of the tile
    const int ic = J >= 16 ? i : i % J, gc = J >= 16 ? g : g % 2;
#pragma unroll
    for (int jt = 0; jt < JT; ++jt) {
      const floatx4 x = *reinterpret_cast<const floatx4*>(m + (16 * ct + ic) * J + 16 * jt + 4 * gc);
#pragma unroll
      for (int u = 0; u < 4; ++u) d[jt][u] = ok ? x[u] : 0.f;
    }
    if (left)
#pragma unroll
      for (int it = 0; it < JT; ++it)
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float x = m[(16 * jt + 4 * gc + u) * J + 16 * it + ic];
            a[it][jt][u] = ok ? x : 0.f;
          }
#pragma unroll
    for (int it = 0; it < JT; ++it) v[it] = m[J * J + 16 * it + ic];
    s = scale[slot];
  }
};

template <int J>
__global__ __launch_bounds__(256) void k_combine(const CItem* __restrict__ items, int64_t n_items,
                                                 float* __restrict__ maps, double* __restrict__ map_scale) {
  constexpr int JT = MapRegs<J>::JT;
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int64_t k = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (k >= n_items * JT) return;
  const CItem it = items[k / JT];
  const int ct = (int)(k % JT);
  MapRegs<J> P, cur, nxt;
  P.load(maps, map_scale, it.in_off, ct, i, g, false);
  if (it.count > 1) nxt.load(maps, map_scale, it.in_off + 1, ct, i, g, true);
  for (int c = 1; c < it.count; ++c) {
    cur = nxt;
    if (c + 1 < it.count) nxt.load(maps, map_scale, it.in_off + c + 1, ct, i, g, true);
    floatx4 acc[JT];
#pragma unroll
    for (int rt = 0; rt < JT; ++rt) acc[rt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int rt = 0; rt < JT; ++rt)
          acc[rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(cur.a[rt][jt][u], P.d[jt][u], acc[rt], 0, 0, 0);
    if (ct == 0) {
      // N2 v1: lane (i, g) adds its four columns per tile, then the four rows of lanes
      float w[JT][4];
#pragma unroll
      for (int jt = 0; jt < JT; ++jt)
#pragma unroll
        for (int u = 0; u < 4; ++u) w[jt][u] = __shfl(P.v[jt], 4 * g + u);
#pragma unroll
      for (int rt = 0; rt < JT; ++rt) {
        float z = 0.f;
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
          for (int u = 0; u < 4; ++u) z = fmaf(cur.a[rt][jt][u], w[jt][u], z);
        z = sum_rows(sum_halves(z));
        P.v[rt] = (float)(cur.s * ((double)P.v[rt] + (double)z)) + cur.v[rt];
      }
    }
#pragma unroll
    for (int rt = 0; rt < JT; ++rt) P.d[rt] = (P.d[rt] + cur.d[rt]) + acc[rt];
    P.s *= cur.s;
  }
  float* dst = maps + it.out_off * (J * J + J);
  if (J >= 16 || (i < J && 4 * g < J)) {
#pragma unroll
    for (int jt = 0; jt < JT; ++jt)
      *reinterpret_cast<floatx4*>(dst + (16 * ct + i) * J + 16 * jt + 4 * g) = P.d[jt];
    if (ct == 0 && g == 0)
#pragma unroll
      for (int rt = 0; rt < JT; ++rt) dst[J * J + 16 * rt + i] = P.v[rt];
  }
  if (ct == 0 && lane == 0) map_scale[it.out_off] = P.s;
}

// The last fold at J = 32, a wavefront per row: lane (i, g) takes row
// 16 (g % 2) + i of a map and the 16 columns from 16 (g / 2) on, which the
// state is kept spread for.  16 loads and FMAs per lane and map where a
// 16-lane group per row takes 64 (16 maps: 16 us -> 8 us).
__global__ __launch_bounds__(256) void k_combine_final32(const CItem* __restrict__ items, int64_t n_items,
                                                         const float* __restrict__ maps,
                                                         const double* __restrict__ map_scale,
                                                         const float* __restrict__ hvec, float* __restrict__ Am) {
  constexpr int J = 32, D = 4;  // maps in flight
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int64_t k = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (k >= n_items) return;
  const CItem it = items[k];
  const int row = 16 * (g & 1) + i;
  double a = (double)hvec[(int64_t)it.heavy * J + row];
  float N[D][16], v[D];
  double s[D];
  auto load = [&](int c, float (&n)[16], float& vv, double& sc) {
    const int64_t slot = it.in_off + min(c, it.count - 1);
    const float* m = maps + slot * (J * J + J);
#pragma unroll
    for (int q = 0; q < 16; ++q) n[q] = m[(16 * (g >> 1) + q) * J + row];
    vv = m[J * J + row];
    sc = map_scale[slot];
  };
  static_for<0, D>([&](auto S) { load(decltype(S)::value, N[decltype(S)::value], v[decltype(S)::value], s[decltype(S)::value]); });
  for (int c0 = 0; c0 < it.count; c0 += D) {
    static_for<0, D>([&](auto S) {
      constexpr int d = decltype(S)::value;
      if (c0 + d < it.count) {
        const uint32_t af = __float_as_uint((float)a);
        const auto h = __builtin_amdgcn_permlane16_swap(af, af, false, false);  // every row: a_0..15, a_16..31
        const float as = __uint_as_float(g < 2 ? h[0] : h[1]);
        float z = bsum<8>(as, N[d]);
        z += bsum<8>(__builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__float_as_int(as), 0x128, 0xf, 0xf, true)),
                     N[d] + 8);
        z = sum_halves(z);
        a = s[d] * (a + (double)z) + (double)v[d];
        load(c0 + d + D, N[d], v[d], s[d]);
      }
    });
  }
  if (g < 2) Am[(int64_t)it.row * J + row] = (float)a;
}

// Last fold of a heavy row: its remaining maps, earliest first, applied to
// the head vector (the row's state after its first chunk),
//     a <- s (a + N a) + v,
// J^2 work per map where composing two maps costs J^3.  One 16-lane group
// per row; lane i holds a_i in FP64 and row i of the maps in flight (D of
// them, loaded ahead of the dependent chain).  Rows of a wavefront have
// similar map counts (the list is sorted by count); steps past a row's count
// leave it unchanged.
template <int J>
__global__ __launch_bounds__(256) void k_combine_final(const CItem* __restrict__ items, int64_t n_items,
                                                       const float* __restrict__ maps,
                                                       const double* __restrict__ map_scale,
                                                       const float* __restrict__ hvec, float* __restrict__ Am) {
  static_assert(J <= 16, "J = 32 has a wavefront per row");
  constexpr int MS = J * J + J;
  constexpr int D = 4;
  const int l = threadIdx.x & 15;
  const int64_t gid = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
  CItem it{0, 0, 0, 0, 0, 0};
  if (gid < n_items) it = items[gid];
  double a = (it.count > 0 && l < J) ? (double)hvec[(int64_t)it.heavy * J + l] : 0.0;
  int maxc = it.count;
  maxc = max(maxc, __shfl_xor(maxc, 16));
  maxc = max(maxc, __shfl_xor(maxc, 32));
  // row l of map k (entry (l, q) at q J + l); lanes past J (J = 8) read row
  // J - 1 and discard it.  Past the row's count: its last map.
  auto load = [&](int k, float (&Nr)[J], float& v, double& sc) {
    const int64_t slot = it.in_off + min(k, max(it.count - 1, 0));
    const float* mp = maps + slot * MS;
    const int i = min(l, J - 1);
#pragma unroll
    for (int q = 0; q < J; ++q) Nr[q] = mp[q * J + i];
    v = mp[J * J + i];
    sc = map_scale[slot];
  };
  float Nq[D][J], vq[D];
  double sq[D];
  static_for<0, D>([&](auto S) { load(decltype(S)::value, Nq[decltype(S)::value], vq[decltype(S)::value],
                                      sq[decltype(S)::value]); });
  for (int k0 = 0; k0 < maxc; k0 += D) {
    static_for<0, D>([&](auto S) {
      constexpr int d = decltype(S)::value;
      const int k = k0 + d;
      if (k < maxc) {
        float acc = 0.f;
        dot_bcast<J>(acc, (float)a, Nq[d]);
        if (k < it.count) a = sq[d] * (a + (double)acc) + (double)vq[d];
        load(k + D, Nq[d], vq[d], sq[d]);
      }
    });
  }
  if (it.count > 0 && l < J) Am[(int64_t)it.row * J + l] = (float)a;
}

// FT_RELAXED merge of a long row's chunk increments, in two fixed levels so
// that rows of many thousand chunks spread over many workgroups and the sums
// do not depend on timing.  Both levels sum `count` consecutive records of
// J + 1 values (the increment, then sum ||g||^2) in FP64: thread (sub, j)
// adds records sub, sub + S, sub + 2 S, ... (S = 256 / J; a wavefront reads
// 64 / J consecutive records, one contiguous run), then the S partial sums
// are added in a fixed tree order in LDS.
template <int J, class In>
__device__ __forceinline__ void sum_records(const In* __restrict__ base, int count, double (&ssum)[256 / J][J + 1]) {
  constexpr int S = 256 / J;
  const int t = threadIdx.x, j = t % J, sub = t / J;
  double s = 0.0, G = 0.0;
#pragma unroll 4
  for (int k = sub; k < count; k += S) {
    s += (double)base[(int64_t)k * (J + 1) + j];
    if (j == 0) G += (double)base[(int64_t)k * (J + 1) + J];
  }
  ssum[sub][j] = s;
  if (j == 0) ssum[sub][J] = G;
  __syncthreads();
  for (int stride = S / 2; stride >= 1; stride /= 2) {
    if (sub < stride) {
      ssum[sub][j] += ssum[sub + stride][j];
      if (j == 0) ssum[sub][J] += ssum[sub + stride][J];
    }
    __syncthreads();
  }
}

// Level 1: one workgroup per group of at most kRelaxGroup consecutive chunks
// of one row; writes the group's FP64 record.
template <int J>
__global__ __launch_bounds__(256) void k_relaxed_group(const CItem* __restrict__ items, const float* __restrict__ incr,
                                                       double* __restrict__ part) {
  __shared__ double ssum[256 / J][J + 1];
  const CItem it = items[blockIdx.x];
  sum_records<J>(incr + it.in_off * (J + 1), it.count, ssum);
  const int t = threadIdx.x;
  if (t <= J) part[it.out_off * (J + 1) + t] = ssum[0][t];
}

// Level 2: one workgroup per long row, over its groups' records.  a_H (the
// row after its head) is in A(m); the row becomes
//     a_H + omega ((rho^(L - head) - 1) a_H + sum),
//     omega = min(1, 1 / (lr sum ||g||^2)).
template <int J>
__global__ __launch_bounds__(256) void k_relaxed_merge(const CItem* __restrict__ items, const double* __restrict__ part,
                                                       float* __restrict__ Am, double lr, double rho) {
  __shared__ double ssum[256 / J][J + 1];
  const CItem it = items[blockIdx.x];
  sum_records<J>(part + it.in_off * (J + 1), it.count, ssum);
  const int t = threadIdx.x;
  if (t < J) {
    const double lg = lr * ssum[0][J];
    const double omega = lg > 1.0 ? 1.0 / lg : 1.0;
    const double decay = pow(rho, (double)it.out_off);  // out_off: elements after the head
    float* a = Am + (int64_t)it.row * J + t;
    const double aH = (double)*a;
    *a = (float)(aH + omega * ((decay - 1.0) * aH + ssum[0][t]));
  }
}

// workgroups for n items, one per wavefront or four
int64_t item_blocks(int64_t n, bool quad) { return quad ? (n + 15) / 16 : (n + 3) / 4; }

// CALL(true) or CALL(false): a kernel with the four-item paths, or without
#define FT_QUAD(quad, J, CALL)                     \
  do {                                             \
    if constexpr (J <= 16) {                       \
      if (quad) CALL(true);                        \
      else CALL(false);                            \
    } else {                                       \
      CALL(false);                                 \
    }                                              \
  } while (0)

template <int N, int J, int R, class T, bool FIB, bool NC = false>
hipError_t factor_launch(const ft_plan* P, int m, const ft_params* p, const Scratch& S, double lr, double lam,
                         hipStream_t s) {
  const ModeMeta& M = P->meta[m];
  const ModeDev& D = P->dev[m];
  FactorArgs<N, J, R, T, FIB, NC> F{};
  F.idx = D.idx;
  F.nnz = P->nnz;
  F.val = D.val;
  F.cp = others<N, T>(p, m);
  F.Bm = Store<T>::B(p, m);
  F.Am = p->A[m];
  F.hvec = S.hvec;
  F.fid = D.fid;
  F.gfib = S.gfib;
  if (NC)
    for (int k = 0; k < N - 1; ++k) {
      F.nc.A[k] = p->A[(m + 1 + k) % N];
      F.nc.B[k] = p->B[(m + 1 + k) % N];
    }
  F.maps = S.maps;
  F.map_scale = S.map_scale;
  F.row_ptr = D.row_ptr;
  F.rho = 1.0 - lr * lam;
  F.gp = lr / F.rho;
  // rho^-15 scales the values of a block: with rho >= 1/2 it stays below 2^15;
  // a decay above that (lr lam > 1/2) is stepped element by element
  F.block = F.rho >= 0.5 ? 16 : 1;
  F.pw.p[0] = 1.0;
  for (int k = 1; k <= 16; ++k) F.pw.p[k] = F.pw.p[k - 1] * F.rho;
  for (int k = 0; k < F.block; ++k) {
    const double inv = 1.0 / F.pw.p[k];
    F.pw.inv[k] = (float)inv;
    F.pw.inv_lo[k] = (float)(inv - (double)F.pw.inv[k]);
  }
  // the list of in-place items: n_team for a workgroup each (padded to a multiple of four), then one per wavefront,
  // the shortest rows as packs (or, where blocks are single elements, on their own)
  const int64_t n_packs = F.block == 16 ? M.n_packs : 0, n_apply = n_packs > 0 ? M.n_wave : M.n_apply;
  const int64_t n_rows = n_apply - (M.n_team + 3) / 4 * 4;
  if (F.block == 16) {
    if (quad_chunks(N, J, P->relaxed, M.n_compose)) F.quads |= kQuadChunks;
    if (quad_rows(N, J, P->relaxed, n_rows, M.row_elems, M.n_compose)) F.quads |= kQuadRows;
  }
  // (a launch of rows, or of chunks, alone needs the four-item paths for these only)
  const int rows4 = F.quads & kQuadRows, chunks4 = F.quads & kQuadChunks;
  const int64_t row_waves = rows4 ? (n_rows + 3) / 4 : n_rows;
  const int64_t apply_blocks = M.n_team + (row_waves + n_packs + 3) / 4;
  const int64_t compose_blocks = item_blocks(M.n_compose, chunks4);
#define FT_APPLY(Q)                                                                                                  \
  hipLaunchKernelGGL((k_factor_apply<Q, N, J, R, T, FIB, NC>), block_grid(apply_blocks), dim3(256), 0, s, D.apply, \
                     n_apply, M.n_team, D.packs, n_packs, F)
#define FT_RELAXED_CHUNKS(Q)                                                                                     \
  hipLaunchKernelGGL((k_factor_compose<ITEM_RELAXED, Q, N, J, R, T, FIB, NC>), block_grid(compose_blocks),     \
                     dim3(256), 0, s, D.compose, M.n_compose, F)
#define FT_MAPS(Q)                                                                                               \
  hipLaunchKernelGGL((k_factor_compose<ITEM_MAP, Q, N, J, R, T, FIB, NC>), block_grid(compose_blocks), dim3(256), \
                     0, s, D.compose, M.n_compose, F)
#define FT_FUSED(Q)                                                                                                 \
  hipLaunchKernelGGL((k_factor_fused<Q, N, J, R, T, FIB, NC>), block_grid(apply_blocks + compose_blocks),         \
                     dim3(256), 0, s, M.n_team, compose_blocks, D.apply, n_apply, D.compose, M.n_compose, D.packs, \
                     n_packs, F)
  if (FIB) {
    KTimer tm(P, FT_K_FIBER_G, s);
    const int64_t per_block = 4 * 16 * kFiberBlocks;  // fibers of a workgroup
    hipLaunchKernelGGL((k_fiber_g<N, J, R, T>), dim3((unsigned)((M.n_fibers + per_block - 1) / per_block)), dim3(256),
                       0, s, D.fib_idx, M.n_fibers, F.cp, F.Bm, S.gfib);
  }
  if constexpr (!NC) {
    if (P->relaxed) {
      // short rows and heads (in place), then the chunks from the rows as their heads left them, then the
      // two merge levels; long rows are read in their dealt order
      if (D.fidx) F.idx = D.fidx;
      if (D.fval) F.val = D.fval;
      F.hvec = nullptr;
      if (M.n_apply > 0) {
        KTimer tm(P, FT_K_FACTOR_APPLY, s);
        FT_QUAD(rows4, J, FT_APPLY);
      }
      if (M.n_compose > 0) {
        KTimer tm(P, FT_K_FACTOR_COMPOSE, s);
        FT_QUAD(chunks4, J, FT_RELAXED_CHUNKS);
      }
      if (M.n_relax > 0) {
        KTimer tm(P, FT_K_COMBINE, s);
        double* part = relax_partials(P, S, m);
        hipLaunchKernelGGL((k_relaxed_group<J>), dim3((unsigned)M.n_relax_groups), dim3(256), 0, s, D.relax,
                           S.maps, part);
        hipLaunchKernelGGL((k_relaxed_merge<J>), dim3((unsigned)M.n_relax), dim3(256), 0, s,
                           D.relax + M.n_relax_groups, part, p->A[m], lr, F.rho);
      }
      return hipGetLastError();
    }
  }
  if (M.n_compose > 0 && M.n_apply > 0 && P->fused) {
    KTimer tm(P, FT_K_FACTOR_FUSED, s);
    FT_QUAD(F.quads, J, FT_FUSED);
  } else {
    if (M.n_compose > 0) {
      KTimer tm(P, FT_K_FACTOR_COMPOSE, s);
      FT_QUAD(chunks4, J, FT_MAPS);
    }
    if (M.n_apply > 0) {
      KTimer tm(P, FT_K_FACTOR_APPLY, s);
      FT_QUAD(rows4, J, FT_APPLY);
    }
  }
#undef FT_APPLY
#undef FT_RELAXED_CHUNKS
#undef FT_MAPS
#undef FT_FUSED
  for (size_t L = 0; L < M.level_len.size(); ++L) {
    KTimer tm(P, FT_K_COMBINE, s);
    const int64_t nc = M.level_ncomp[L], nf = M.level_len[L] - nc;
    if (nc > 0)
      hipLaunchKernelGGL((k_combine<J>), dim3((unsigned)((nc * MapRegs<J>::JT + 3) / 4)), dim3(256), 0, s,
                         D.levels + M.level_off[L], nc, S.maps, S.map_scale);
    if (nf > 0) {
      const CItem* last = D.levels + M.level_off[L] + nc;
      if constexpr (J == 32)
        hipLaunchKernelGGL(k_combine_final32, dim3((unsigned)((nf + 3) / 4)), dim3(256), 0, s, last, nf, S.maps,
                           S.map_scale, S.hvec, p->A[m]);
      else
        hipLaunchKernelGGL((k_combine_final<J>), dim3((unsigned)((nf + 15) / 16)), dim3(256), 0, s, last, nf, S.maps,
                           S.map_scale, S.hvec, p->A[m]);
    }
  }
  return hipGetLastError();
}

template <int N, int J, int R, class T>
hipError_t factor_impl(const ft_plan* P, int m, const ft_params* p, const Scratch& S, double lr, double lam,
                       hipStream_t s) {
  if (P->no_c_cache) {
    if constexpr (N == 3 && J == 16 && R == 16 && std::is_same<T, float>::value)
      return factor_launch<N, J, R, T, false, true>(P, m, p, S, lr, lam, s);
    else
      return hipErrorInvalidValue;  // rejected at plan creation and in the parameter checks
  }
  return P->meta[m].use_fiber ? factor_launch<N, J, R, T, true>(P, m, p, S, lr, lam, s)
                              : factor_launch<N, J, R, T, false>(P, m, p, S, lr, lam, s);
}

}  // namespace

int max_fanin() { return kMaxFanin; }

hipError_t launch_factor(const ft_plan* P, int m, const ft_params* p, const Scratch& S, double lr, double lam,
                         hipStream_t s) {
#define X(n, j, r)                                                                             \
  case key(n, j, r):                                                                           \
    return bf16(p) ? factor_impl<n, j, r, uint16_t>(P, m, p, S, lr, lam, s)                   \
                   : factor_impl<n, j, r, float>(P, m, p, S, lr, lam, s);
  FT_DISPATCH()
#undef X
}

}  // namespace ft
