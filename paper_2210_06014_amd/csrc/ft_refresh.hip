// C refresh (MFMA) and BF16 casts.
#include "ft_device.h"

namespace ft {
namespace {

// ---------------------------------------------------------------------------
// C = A B  (I x J) (J x R) on the matrix cores, TPW tiles of 16 rows per
// wavefront.  The refresh streams A in and C out (a few flops per byte), so
// the layout is chosen for the loads: the sum over k may run in any order,
// and lane (i, g) of a tile (row i = lane % 16, group g = lane / 16) takes
// the k values whose A entries are contiguous in its row, so that A arrives
// in 16-byte loads covering whole row pieces; every load of a wavefront is
// issued before its first MFMA.

constexpr int kRefreshTiles = 4;  // 16-row tiles per wavefront

// FP32, v_mfma_f32_16x16x4_f32: lane (i, g) supplies A[i][k] and B[k][col]
// for one k per instruction and receives D[4 g + v][col], col = lane % 16.
// For J a multiple of 16 its k values are 16 h + 4 g + u (h < J / 16,
// u < 4: float4 loads); for J = 8 they are 2 g + u.
template <int J>
__device__ __forceinline__ int refresh_k(int g, int kb) {
  if constexpr (J % 16 == 0)
    return 16 * (kb / 4) + 4 * g + (kb % 4);
  else
    return (J / 4) * g + kb;
}

// The modes of one launch (blockIdx.y): one, or all of them when every C is
// refreshed, so that a model's first refresh is one launch.
struct RefreshArgs {
  const float* A[FT_MAX_ORDER];
  const float* B[FT_MAX_ORDER];
  void* A16[FT_MAX_ORDER];
  void* B16[FT_MAX_ORDER];
  void* C[FT_MAX_ORDER];  // FP32, or BF16
  int64_t I[FT_MAX_ORDER];
};

template <int J, int R>
__global__ __launch_bounds__(256) void k_refresh(RefreshArgs args) {
  const float* __restrict__ A = args.A[blockIdx.y];
  const float* __restrict__ B = args.B[blockIdx.y];
  float* __restrict__ C = static_cast<float*>(args.C[blockIdx.y]);
  const int64_t I = args.I[blockIdx.y];
  static_assert(J % 4 == 0, "J is a multiple of 4");
  constexpr int KPL = J / 4;  // k values per lane
  constexpr int CT = (R + 15) / 16;
  constexpr int TPW = kRefreshTiles;
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int64_t tile0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * TPW;
  if (tile0 * 16 >= I) return;
  float b[CT][KPL];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct) {
    const int col = ct * 16 + li;
#pragma unroll
    for (int kb = 0; kb < KPL; ++kb) b[ct][kb] = col < R ? B[refresh_k<J>(lg, kb) * R + col] : 0.f;
  }
  float a[TPW][KPL];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int64_t row = (tile0 + t) * 16 + li;
    const bool ok = row < I;
    const float* ar = A + (ok ? row : 0) * J;
    if constexpr (J % 16 == 0) {
#pragma unroll
      for (int h = 0; h < J / 16; ++h) {
        const floatx4 v = *reinterpret_cast<const floatx4*>(ar + 16 * h + 4 * lg);
#pragma unroll
        for (int u = 0; u < 4; ++u) a[t][4 * h + u] = ok ? v[u] : 0.f;
      }
    } else {
#pragma unroll
      for (int kb = 0; kb < KPL; ++kb) a[t][kb] = ok ? ar[refresh_k<J>(lg, kb)] : 0.f;
    }
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int64_t row0 = (tile0 + t) * 16;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < KPL; ++kb) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][kb], b[ct][kb], acc, 0, 0, 0);
      const int col = ct * 16 + li;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = row0 + lg * 4 + v;
        if (r < I && col < R) C[r * R + col] = acc[v];
      }
    }
  }
}

// BF16 storage: A16 = bf16(A), B16 = bf16(B), C16 = bf16(A16 B16) in one launch,
// with v_mfma_f32_16x16x16_bf16 (FP32 accumulation): a lane rounds the master
// values that it supplies to the product and stores them (three launches,
// casts first, took 12 us on a 10,000-row mode, this one 5).  Lane (i, g)
// supplies four k values per instruction: with J a multiple of 32 they are
// 8 g + 4 kb + u (8 consecutive values of a row cover both instructions),
// otherwise 16 kb + 4 g + u; k beyond J supplies zeros.  The result layout is
// that of the FP32 tile.
typedef short shortx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint16_t f2bf(float f) {
  // round to nearest even on the upper 16 bits (IEEE-754 binary32 -> bfloat16); NaN stays NaN
  const uint32_t u = __float_as_uint(f);
  const uint32_t nan = (u >> 16) | 0x40u, num = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
  return (uint16_t)((u & 0x7FFFFFFFu) > 0x7F800000u ? nan : num);
}

template <int J>
__device__ __forceinline__ int refresh_k16(int g, int kb, int u) {
  if constexpr (J % 32 == 0)
    return 32 * (kb / 2) + 8 * g + 4 * (kb % 2) + u;
  else
    return 16 * kb + 4 * g + u;
}

template <int J, int R>
__global__ __launch_bounds__(256) void k_refresh_bf16(RefreshArgs args) {
  constexpr int CT = (R + 15) / 16;
  constexpr int KB = (J + 15) / 16;
  constexpr int TPW = kRefreshTiles;
  const float* __restrict__ A = args.A[blockIdx.y];
  const float* __restrict__ B = args.B[blockIdx.y];
  uint16_t* __restrict__ A16 = static_cast<uint16_t*>(args.A16[blockIdx.y]);
  uint16_t* __restrict__ B16 = static_cast<uint16_t*>(args.B16[blockIdx.y]);
  uint16_t* __restrict__ C = static_cast<uint16_t*>(args.C[blockIdx.y]);
  const int64_t I = args.I[blockIdx.y];
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int64_t tile0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * TPW;
  if (tile0 * 16 >= I) return;
  // loads from clamped addresses, masked afterwards, so that all are in flight together
  float bv[CT][KB][4], av[TPW][KB][4];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        bv[ct][kb][u] = B[min(refresh_k16<J>(lg, kb, u), J - 1) * R + min(ct * 16 + li, R - 1)];
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const float* ar = A + min((tile0 + t) * 16 + li, I - 1) * J;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const int k = min(refresh_k16<J>(lg, kb, 0), J - 4);  // four consecutive values
#pragma unroll
      for (int u = 0; u < 4; ++u) av[t][kb][u] = ar[k + u];
    }
  }
  shortx4 b[CT][KB], a[TPW][KB];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool ok = ct * 16 + li < R && refresh_k16<J>(lg, kb, u) < J;
        b[ct][kb][u] = ok ? (short)f2bf(bv[ct][kb][u]) : (short)0;
      }
#pragma unroll
  for (int t = 0; t < TPW; ++t)
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool ok = (tile0 + t) * 16 + li < I && refresh_k16<J>(lg, kb, u) < J;
        a[t][kb][u] = ok ? (short)f2bf(av[t][kb][u]) : (short)0;
      }
  if (tile0 == 0) {  // the first wavefront stores B16: its lanes hold every entry once
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int col = ct * 16 + li, k = refresh_k16<J>(lg, kb, u);
          if (col < R && k < J) B16[k * R + col] = (uint16_t)b[ct][kb][u];
        }
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int64_t row = (tile0 + t) * 16 + li;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
      const int k = refresh_k16<J>(lg, kb, 0);
      if (row < I && k < J) __builtin_memcpy(A16 + row * J + k, &a[t][kb], 8);
    }
  }
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    const int64_t row0 = (tile0 + t) * 16;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
      floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kb = 0; kb < KB; ++kb) acc = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a[t][kb], b[ct][kb], acc, 0, 0, 0);
      const int col = ct * 16 + li;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = row0 + lg * 4 + v;
        if (r < I && col < R) C[r * R + col] = f2bf(acc[v]);
      }
    }
  }
}

}  // namespace

bool supported(int N, int J, int R) {
  switch (key(N, J, R)) {
#define X(n, j, r) \
  case key(n, j, r): return true;
    FT_CONFIGS(X)
#undef X
    default: return false;
  }
}

// modes n0 .. n1 - 1
hipError_t launch_refresh(const ft_plan* P, int n0, int n1, const ft_params* p, hipStream_t s) {
  RefreshArgs a{};
  int64_t most = 0;
  for (int n = n0; n < n1; ++n) {
    a.A[n - n0] = p->A[n];
    a.B[n - n0] = p->B[n];
    a.A16[n - n0] = p->A16[n];
    a.B16[n - n0] = p->B16[n];
    a.C[n - n0] = bf16(p) ? p->C16[n] : p->C[n];
    a.I[n - n0] = P->desc.dims[n];
    most = std::max(most, P->desc.dims[n]);
  }
  if (n1 <= n0) return hipSuccess;
  const int64_t waves = ((most + 15) / 16 + kRefreshTiles - 1) / kRefreshTiles;
  const dim3 grid((unsigned)((waves + 3) / 4), (unsigned)(n1 - n0));
  KTimer tm(P, FT_K_REFRESH, s);
  switch (P->J * 64 + P->R) {
#define X(j, r)                                                                          \
  case j * 64 + r:                                                                       \
    if (bf16(p))                                                                         \
      hipLaunchKernelGGL((k_refresh_bf16<j, r>), grid, dim3(256), 0, s, a);              \
    else                                                                                 \
      hipLaunchKernelGGL((k_refresh<j, r>), grid, dim3(256), 0, s, a);                   \
    return hipGetLastError();
    X(8, 8) X(16, 16) X(32, 32) X(8, 16)
#undef X
    default: return hipErrorInvalidValue;
  }
}

}  // namespace ft
