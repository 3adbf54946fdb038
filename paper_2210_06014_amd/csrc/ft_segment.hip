// Segment passes: core gradient, loss, forward, gradient, predict.
#include <mutex>

#include "ft_device.h"

namespace ft {
namespace {

// ---------------------------------------------------------------------------
// Segment passes (core gradient, loss, forward, gradient).  A wavefront takes
// segments gw, gw + nw, ... (a fixed assignment), R/4 lanes per element.

// groups of P elements per trip: fewer at high order, where each element
// holds N - 1 indices in registers
template <int N>
constexpr int trip_unroll() {
  return N > 4 ? 2 : 4;
}

// Values per lane in the segment passes: one 16-byte load of a C row, 4 FP32
// or 8 BF16 values, so a row takes R/4 (FP32) or R/8 (BF16) lanes.
template <class T>
constexpr int vpl() {
  return 16 / (int)sizeof(T);
}

__device__ __forceinline__ void load16(const float* p, float (&o)[4]) {
  const floatx4 u = *reinterpret_cast<const floatx4*>(p);
#pragma unroll
  for (int c = 0; c < 4; ++c) o[c] = u[c];
}
__device__ __forceinline__ void load16(const uint16_t* p, float (&o)[8]) {
  const uint4 u = *reinterpret_cast<const uint4*>(p);
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    o[2 * c] = __uint_as_float(w[c] << 16);
    o[2 * c + 1] = __uint_as_float(w[c] & 0xFFFF0000u);
  }
}

// a 16-byte slice as loaded, widened to its 4 FP32 or 8 BF16 values
template <class T>
__device__ __forceinline__ void widen(const uint4& u, float (&o)[vpl<T>()]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int c = 0; c < 4; ++c) o[c] = __uint_as_float(w[c]);
  } else {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      o[2 * c] = __uint_as_float(w[c] << 16);
      o[2 * c + 1] = __uint_as_float(w[c] & 0xFFFF0000u);
    }
  }
}

// prod over the gathered 16-byte slices (lane q of the element) of its C
// rows, in table order; zero for an invalid slot.  Invalid slots carry index
// 0 (a valid row), so the loads need no branch and are all in flight together.
template <int N, int R, class T>
__device__ __forceinline__ void gather_slices(const CPtrs<N, T>& cp, const int32_t (&ik)[N > 1 ? N - 1 : 1], bool vld,
                                              int q, float (&w)[vpl<T>()]) {
  constexpr int V = vpl<T>();
  const uint32_t qb = (uint32_t)(16 * q);
  load16(reinterpret_cast<const T*>(reinterpret_cast<const char*>(cp.p[0]) +
                                    ((uint32_t)ik[0] * (uint32_t)(R * sizeof(T)) + qb)),
         w);
#pragma unroll
  for (int k = 1; k < N - 1; ++k) {
    float t[V];
    load16(reinterpret_cast<const T*>(reinterpret_cast<const char*>(cp.p[k]) +
                                      ((uint32_t)ik[k] * (uint32_t)(R * sizeof(T)) + qb)),
           t);
#pragma unroll
    for (int c = 0; c < V; ++c) w[c] *= t[c];
  }
#pragma unroll
  for (int c = 0; c < V; ++c) w[c] = vld ? w[c] : 0.f;
}

// Indices and values of one trip: trip_unroll groups of P elements of a
// segment from position t0.  Each element is loaded once, by lane
// (element - t0) % 64, and handed to the R/4 lanes that gather for it by a
// cross-lane permute (the LDS crossbar), so that an index load carries 64
// distinct addresses: the address units, which bound these passes, see a
// quarter of the index loads.  Positions past the end are clamped to the
// segment's last element (a valid address), so the loads need no branch.
// A trip of fewer than 32 elements (R = 32 at high orders) would waste most
// of such loads, so there each lane loads its own elements' indices.
template <int N, int P>
struct Trip {
  static constexpr int U = trip_unroll<N>();
  static constexpr bool PERMUTE = U * P >= 32;
  static constexpr int NL = PERMUTE ? (U * P + 63) / 64 : U;  // element loads per lane
  int32_t ik[NL][N > 1 ? N - 1 : 1];
  float xv[NL];
};

template <int N, int P, bool PERM>
__device__ __forceinline__ void load_trip(Trip<N, P>& L, const Seg& S, int t0, int lane,
                                          const int32_t* __restrict__ idx, int64_t nnz, const float* __restrict__ xs,
                                          const int32_t* __restrict__ perm) {
  const int last = max(S.len - 1, 0);
  const int slot = lane / (64 / P);
#pragma unroll
  for (int h = 0; h < Trip<N, P>::NL; ++h) {
    const uint32_t o = (uint32_t)min(Trip<N, P>::PERMUTE ? t0 + 64 * h + lane : t0 + h * P + slot, last);
#pragma unroll
    for (int k = 0; k < N - 1; ++k) L.ik[h][k] = (idx + (int64_t)k * nnz + S.start)[o];
    L.xv[h] = PERM ? xs[(perm + S.start)[o]] : (xs + S.start)[o];
  }
}

// indices and value of element u P + slot of a trip, from the lane that loaded it
template <int N, int P, int u>
__device__ __forceinline__ void trip_elem(const Trip<N, P>& L, int slot, int32_t (&ik)[N > 1 ? N - 1 : 1],
                                          float& xv) {
  if constexpr (Trip<N, P>::PERMUTE) {
    constexpr int h = (u * P) / 64;
    const int src = (u * P + slot) & 63;
#pragma unroll
    for (int k = 0; k < N - 1; ++k) ik[k] = __shfl(L.ik[h][k], src);
    xv = __shfl(L.xv[h], src);
  } else {
#pragma unroll
    for (int k = 0; k < N - 1; ++k) ik[k] = L.ik[u][k];
    xv = L.xv[u];
  }
}

// A wavefront walks its segments gw, gw + nw, ... trip by trip.  While the
// gathers of one trip are in flight it already loads the indices of the next
// trip (the first trip of its next segment at a segment's end, whose
// descriptor was read one segment ahead), so that every trip costs one memory
// round trip instead of two.  A segment of length 0 stands in past the last.

// MODE 0: s = sum e w (core gradient); MODE 1: t = sum -e w (gradient of 1/2 sum e^2);
// MODE 2: t = sum delta w with delta from the caller (input order, via perm).
template <int N, int J, int R, int MODE, class T>
__global__ __launch_bounds__(256) void k_segsum(const Seg* __restrict__ segs, int64_t nseg,
                                                const int32_t* __restrict__ idx, int64_t nnz,
                                                const float* __restrict__ val, CPtrs<N, T> cp,
                                                const T* __restrict__ Cm, const T* __restrict__ Am,
                                                const float* __restrict__ up, const int32_t* __restrict__ perm,
                                                float* __restrict__ partials, float* __restrict__ tseg) {
  constexpr int V = vpl<T>();
  constexpr int QL = R / V;
  constexpr int P = 64 / QL;
  constexpr int GJ = (J + P - 1) / P;
  constexpr int U = trip_unroll<N>();
  __shared__ float red[4][J * R];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = lane / QL, q = lane % QL;
  const int64_t nw = (int64_t)gridDim.x * 4;
  const float* xs = MODE == 2 ? up : val;
  float Gp[GJ][V];
#pragma unroll
  for (int u = 0; u < GJ; ++u)
#pragma unroll
    for (int c = 0; c < V; ++c) Gp[u][c] = 0.f;
  // C(m) slice and A(m) entries of a segment's row
  auto row_loads = [&](const Seg& X, float (&cr)[V], float (&ar)[GJ]) {
    if (MODE != 2) load16(Cm + (int64_t)X.row * R + V * q, cr);
#pragma unroll
    for (int u = 0; u < GJ; ++u) {
      const int j = slot + P * u;
      ar[u] = j < J ? to_f(Am[(int64_t)X.row * J + j]) : 0.f;
    }
  };
  int64_t sg = (int64_t)blockIdx.x * 4 + wave;
  if (sg < nseg) {
    const Seg none{0, 0, 0};
    Seg S = segs[sg];
    Seg Sq = sg + nw < nseg ? segs[sg + nw] : none;
    float crow[V];
#pragma unroll
    for (int c = 0; c < V; ++c) crow[c] = 0.f;
    float arow[GJ];
    row_loads(S, crow, arow);
    Trip<N, P> cur;
    load_trip<N, P, MODE == 2>(cur, S, 0, lane, idx, nnz, xs, perm);
    float acc[V];
#pragma unroll
    for (int c = 0; c < V; ++c) acc[c] = 0.f;
    int t0 = 0;
    for (;;) {
      int32_t ik[U][N > 1 ? N - 1 : 1];
      float xv[U];
      bool vl[U];
      static_for<0, U>([&](auto UU) {
        constexpr int u = decltype(UU)::value;
        trip_elem<N, P, u>(cur, slot, ik[u], xv[u]);
        vl[u] = t0 + u * P + slot < S.len;
      });
      float w[U][V];
#pragma unroll
      for (int u = 0; u < U; ++u) gather_slices<N, R, T>(cp, ik[u], vl[u], q, w[u]);
      const bool seg_end = t0 + P * U >= S.len;
      const Seg& Sn = seg_end ? Sq : S;
      Trip<N, P> nxt;
      load_trip<N, P, MODE == 2>(nxt, Sn, seg_end ? 0 : t0 + P * U, lane, idx, nnz, xs, perm);
      float crow_n[V], arow_n[GJ];
#pragma unroll
      for (int c = 0; c < V; ++c) crow_n[c] = crow[c];
#pragma unroll
      for (int u = 0; u < GJ; ++u) arow_n[u] = arow[u];
      if (seg_end) row_loads(Sq, crow_n, arow_n);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float d;
        if (MODE == 2) {
          d = vl[u] ? xv[u] : 0.f;
        } else {
          float xh = crow[0] * w[u][0];
#pragma unroll
          for (int c = 1; c < V; ++c) xh = fmaf(crow[c], w[u][c], xh);
          xh = group_sum<QL>(xh);
          d = vl[u] ? (MODE == 0 ? xv[u] - xh : xh - xv[u]) : 0.f;
        }
#pragma unroll
        for (int c = 0; c < V; ++c) acc[c] = fmaf(d, w[u][c], acc[c]);
      }
      if (seg_end) {
#pragma unroll
        for (int off = QL; off < 64; off <<= 1)
#pragma unroll
          for (int c = 0; c < V; ++c) acc[c] += __shfl_xor(acc[c], off);
        if (tseg && slot == 0)
#pragma unroll
          for (int c = 0; c < V; ++c) tseg[sg * R + V * q + c] = acc[c];
#pragma unroll
        for (int u = 0; u < GJ; ++u) {
          const int j = slot + P * u;
          if (j < J)
#pragma unroll
            for (int c = 0; c < V; ++c) Gp[u][c] = fmaf(arow[u], acc[c], Gp[u][c]);
        }
        sg += nw;
        if (sg >= nseg) break;
        S = Sq;
        Sq = sg + nw < nseg ? segs[sg + nw] : none;
#pragma unroll
        for (int c = 0; c < V; ++c) {
          crow[c] = crow_n[c];
          acc[c] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < GJ; ++u) arow[u] = arow_n[u];
        t0 = 0;
      } else {
        t0 += P * U;
      }
      cur = nxt;
    }
  }
#pragma unroll
  for (int u = 0; u < GJ; ++u) {
    const int j = slot + P * u;
    if (j < J)
#pragma unroll
      for (int c = 0; c < V; ++c) red[wave][j * R + V * q + c] = Gp[u][c];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < J * R; e += 256)
    partials[(int64_t)blockIdx.x * J * R + e] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
}

// Short rows.  A row of ten elements leaves most of a wavefront idle in the
// walk above (a trip is 64 elements at R = 16, 32 at R = 32), so where a mode
// has many, the plan lists its rows of at most kShortSeg elements apart, by
// descending length, and here the 64 / (R / V) slots of a wavefront take a row
// each: a slot's lanes load the indices of 8 elements at a time and gather them
// one after another, with no sum over the slots.  The rows' contribution to G,
// sum_slot a_slot s_slot^T, is a product over the slots on the matrix cores.
// Mode 0 of the Netflix-shaped tensors (400k rows, half the elements in rows of
// ten): 8M elements, J = R = 32, 240 -> 134 us for both kernels; 5M, J = R = 16, 158 -> 59 us.
template <int N, int J, int R, int MODE, class T>
__global__ __launch_bounds__(256) void k_segshort(const Seg* __restrict__ segs, int64_t seg0, int64_t nseg,
                                                  const int32_t* __restrict__ idx, int64_t nnz,
                                                  const float* __restrict__ val, CPtrs<N, T> cp,
                                                  const T* __restrict__ Cm, const T* __restrict__ Am,
                                                  const float* __restrict__ up, const int32_t* __restrict__ perm,
                                                  float* __restrict__ partials, float* __restrict__ tseg) {
  constexpr int V = vpl<T>();
  constexpr int QL = R / V;
  constexpr int P = 64 / QL;
  constexpr int EB = 8;                        // elements of a slot per batch of index loads
  constexpr int NL = (EB + QL - 1) / QL;       // index loads per lane and batch
  constexpr int U = trip_unroll<N>();          // elements of a slot gathered together
  constexpr int JT = (J + 15) / 16, RT = (R + 15) / 16;
  constexpr int SR = R + 4;
  __shared__ float red[4][J * R];
  __shared__ __align__(16) float sums[4][P * SR];
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = lane / QL, q = lane % QL;
  const float* xs = MODE == 2 ? up : val;
  floatx4 G[JT][RT];
#pragma unroll
  for (int jt = 0; jt < JT; ++jt)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) G[jt][rt] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int64_t ngrp = (nseg + P - 1) / P, nw = (int64_t)gridDim.x * 4;
  for (int64_t grp = (int64_t)blockIdx.x * 4 + wave; grp < ngrp; grp += nw) {
    const int64_t k = grp * P + slot;
    Seg S = segs[seg0 + min(k, nseg - 1)];
    if (k >= nseg) S.len = 0;
    const int maxlen = __builtin_amdgcn_readfirstlane(S.len);  // slot 0's: the list is sorted
    float crow[V];
#pragma unroll
    for (int c = 0; c < V; ++c) crow[c] = 0.f;
    if (MODE != 2) load16(Cm + (int64_t)S.row * R + V * q, crow);
    // A(m) of the slots 4 t + g as the left operand of G
    float av[P / 4][JT];
#pragma unroll
    for (int t = 0; t < P / 4; ++t) {
      const int64_t row = __shfl(S.row, (4 * t + g) * QL);
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        const float a = to_f(Am[row * J + 16 * jt + (J >= 16 ? i : i % J)]);
        av[t][jt] = (J >= 16 || i < J) ? a : 0.f;
      }
    }
    float acc[V];
#pragma unroll
    for (int c = 0; c < V; ++c) acc[c] = 0.f;
    struct Batch {
      int32_t ik[NL][N > 1 ? N - 1 : 1];
      float xv[NL];
    };
    const int last = max(S.len - 1, 0);
    auto load = [&](int t0, Batch& b) {
#pragma unroll
      for (int h = 0; h < NL; ++h) {
        const uint32_t o = (uint32_t)min(t0 + q + QL * h, last);
#pragma unroll
        for (int n = 0; n < N - 1; ++n) b.ik[h][n] = (idx + (int64_t)n * nnz + S.start)[o];
        b.xv[h] = MODE == 2 ? xs[(perm + S.start)[o]] : (xs + S.start)[o];
      }
    };
    Batch cur;
    load(0, cur);
    for (int t0 = 0; t0 < maxlen; t0 += EB) {
      Batch nxt;
      load(t0 + EB, nxt);
      static_for<0, EB / U>([&](auto HH) {
        constexpr int u0 = decltype(HH)::value * U;
        if (t0 + u0 < maxlen) {
          float w[U][V], xv[U];
          bool vl[U];
          static_for<0, U>([&](auto UU) {
            constexpr int u = decltype(UU)::value, e = u0 + u, h = e / QL;
            const int from = slot * QL + e % QL;
            int32_t ik[N > 1 ? N - 1 : 1];
#pragma unroll
            for (int n = 0; n < N - 1; ++n) ik[n] = QL > 1 ? __shfl(cur.ik[h][n], from) : cur.ik[h][n];
            xv[u] = QL > 1 ? __shfl(cur.xv[h], from) : cur.xv[h];
            vl[u] = t0 + e < S.len;
            gather_slices<N, R, T>(cp, ik, vl[u], q, w[u]);
          });
#pragma unroll
          for (int u = 0; u < U; ++u) {
            float d;
            if (MODE == 2) {
              d = vl[u] ? xv[u] : 0.f;
            } else {
              float xh = crow[0] * w[u][0];
#pragma unroll
              for (int c = 1; c < V; ++c) xh = fmaf(crow[c], w[u][c], xh);
              xh = group_sum<QL>(xh);
              d = vl[u] ? (MODE == 0 ? xv[u] - xh : xh - xv[u]) : 0.f;
            }
#pragma unroll
            for (int c = 0; c < V; ++c) acc[c] = fmaf(d, w[u][c], acc[c]);
          }
        }
      });
      cur = nxt;
    }
    if (tseg && k < nseg)
#pragma unroll
      for (int c = 0; c < V; ++c) tseg[(seg0 + k) * R + V * q + c] = acc[c];
    // (the wavefront's own LDS, in order)
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int c = 0; c < V; c += 4)
      *reinterpret_cast<floatx4*>(&sums[wave][slot * SR + V * q + c]) =
          floatx4{acc[c], acc[c + 1], acc[c + 2], acc[c + 3]};
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int t = 0; t < P / 4; ++t)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const float sv = sums[wave][(4 * t + g) * SR + 16 * rt + (R >= 16 ? i : i % R)];
        const float sr = (R >= 16 || i < R) ? sv : 0.f;
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
          G[jt][rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[t][jt], sr, G[jt][rt], 0, 0, 0);
      }
  }
#pragma unroll
  for (int jt = 0; jt < JT; ++jt)
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j = 16 * jt + 4 * g + v, r = 16 * rt + i;
        if (j < J && r < R) red[wave][j * R + r] = G[jt][rt][v];
      }
  __syncthreads();
  for (int e = threadIdx.x; e < J * R; e += 256)
    partials[(int64_t)blockIdx.x * J * R + e] = ((red[0][e] + red[1][e]) + red[2][e]) + red[3][e];
}

// ---------------------------------------------------------------------------
// Segment passes with the C row of the first index column reused along runs.
// Within a row of mode m the elements are sorted by the index of mode m + 1
// (column 0 of idx), so consecutive elements repeat it in runs (at order 3 the
// fibers of the third mode).  Here the P slots of a wavefront (R/V lanes
// each) take contiguous pieces of a segment, so that a run stays within a
// slot, and a slot gathers the column-0 row only where that index changes:
// per element it gathers the rows of the other columns, per run one more.
// With u = C(m)[row] * C(m+1)[j] formed once per run,
//     xhat = u . prod_{k >= 1} C[i_k]                        (per element)
//     s = sum_x e_x w_x = sum_runs C(m+1)[j] * t_run,  t_run = sum_{x in run} e_x prod_{k >= 1} C[i_k].
// MODE 0, 1, 2 as in k_segsum; MODE 3: loss (FP64 sum of e^2) and, with out,
// xhat stored at the element's input position.  The walk, the partials and
// the fixed summation order are otherwise those of k_segsum: a wavefront
// takes segments gw, gw + nw, ..., and each trip of U steps loads the indices
// of the next trip (across segment boundaries) while its gathers are in
// flight.
template <int N, int J, int R, int MODE, class T>
__global__ __launch_bounds__(256) void k_segrun(const Seg* __restrict__ segs, int64_t nseg,
                                                const int32_t* __restrict__ idx, int64_t nnz,
                                                const float* __restrict__ val, CPtrs<N, T> cp,
                                                const T* __restrict__ Cm, const T* __restrict__ Am,
                                                const float* __restrict__ up, const int32_t* __restrict__ perm,
                                                float* __restrict__ partials, float* __restrict__ tseg,
                                                double* __restrict__ dpart, float* __restrict__ out) {
  static_assert(N >= 3, "run reuse needs a column besides the first");
  constexpr int V = vpl<T>();
  constexpr int QL = R / V;               // lanes per element
  constexpr int P = 64 / QL;              // slots per wavefront
  constexpr int GJ = (J + P - 1) / P;
  constexpr int U = N > 4 ? 2 : 4;        // steps per trip
  constexpr int NL = (U + QL - 1) / QL;   // element loads per lane per trip
  constexpr int NI = N - 1;
  constexpr bool LOSS = MODE == 3;
  constexpr bool PERM = MODE == 2;
  __shared__ float red[LOSS ? 1 : 4][LOSS ? 1 : J * R];
  __shared__ double dred[4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = lane / QL, q = lane % QL;
  const int64_t nw = (int64_t)gridDim.x * 4;
  const float* xs = PERM ? up : val;
  float Gp[LOSS ? 1 : GJ][V];
#pragma unroll
  for (int u = 0; u < (LOSS ? 1 : GJ); ++u)
#pragma unroll
    for (int c = 0; c < V; ++c) Gp[u][c] = 0.f;
  double sse = 0.0;
  // loads of one trip: lane q of a slot loads the slot's elements q, q + QL, ... of the trip
  struct Ld {
    int32_t ik[NL][NI];
    float xv[NL];
  };
  auto load_trip = [&](Ld& L, const Seg& X, int k0) {
    const int Ls = (X.len + P - 1) / P;
    const int last = max(X.len - 1, 0);
#pragma unroll
    for (int h = 0; h < NL; ++h) {
      const uint32_t o = (uint32_t)min(slot * Ls + k0 + q + QL * h, last);
#pragma unroll
      for (int k = 0; k < NI; ++k) L.ik[h][k] = (idx + (int64_t)k * nnz + X.start)[o];
      L.xv[h] = PERM ? xs[(perm + X.start)[o]] : (xs + X.start)[o];
    }
  };
  auto row_loads = [&](const Seg& X, float (&cr)[V], float (&ar)[LOSS ? 1 : GJ]) {
    if (MODE != 2) load16(Cm + (int64_t)X.row * R + V * q, cr);
    if constexpr (!LOSS) {
#pragma unroll
      for (int u = 0; u < GJ; ++u) {
        const int j = slot + P * u;
        ar[u] = j < J ? to_f(Am[(int64_t)X.row * J + j]) : 0.f;
      }
    }
  };
  int64_t sg = (int64_t)blockIdx.x * 4 + wave;
  if (sg < nseg) {
    const Seg none{0, 0, 0};
    Seg S = segs[sg];
    Seg Sq = sg + nw < nseg ? segs[sg + nw] : none;
    float crow[V], arow[LOSS ? 1 : GJ];
#pragma unroll
    for (int c = 0; c < V; ++c) crow[c] = 0.f;
    row_loads(S, crow, arow);
    Ld cur;
    load_trip(cur, S, 0);
    int Ls = (S.len + P - 1) / P;
    int b = slot * Ls, e = min(S.len, b + Ls);
    // run state of this slot: the column-0 index and row of the current run,
    // u = crow * c1, the run's partial sum t, the segment's sum s
    int32_t jprev = -1;
    float c1[V], uu[V], t[V], s[V];
#pragma unroll
    for (int c = 0; c < V; ++c) c1[c] = uu[c] = t[c] = s[c] = 0.f;
    int k0 = 0;
    for (;;) {
      int32_t ik[U][NI];
      float xv[U];
      bool vl[U], nr[U];
      static_for<0, U>([&](auto UU) {
        constexpr int u = decltype(UU)::value;
        constexpr int h = u / QL;
        const int src = slot * QL + (u % QL);
#pragma unroll
        for (int k = 0; k < NI; ++k) ik[u][k] = QL > 1 ? __shfl(cur.ik[h][k], src) : cur.ik[h][k];
        xv[u] = QL > 1 ? __shfl(cur.xv[h], src) : cur.xv[h];
        vl[u] = b + k0 + u < e;
      });
      // a step starts a run where its column-0 index differs from the step before
      nr[0] = vl[0] && ik[0][0] != jprev;
#pragma unroll
      for (int u = 1; u < U; ++u) nr[u] = vl[u] && ik[u][0] != ik[u - 1][0];
      // gathers: the rows of columns 1.. for every step, the column-0 row where a run starts
      // slices are kept as loaded (four registers, FP32 or BF16) and widened
      // where used; at order 4 and up the per-element product is formed here
      constexpr bool PROD = NI > 2;
      uint4 w2r[U], cnr[U];
      float w2p[PROD ? U : 1][PROD ? V : 1];
      const uint32_t qb = (uint32_t)(16 * q);
      auto slice = [&](int k, int32_t i) {
        return *reinterpret_cast<const uint4*>(reinterpret_cast<const char*>(cp.p[k]) +
                                               ((uint32_t)i * (uint32_t)(R * sizeof(T)) + qb));
      };
#pragma unroll
      for (int u = 0; u < U; ++u) {
        w2r[u] = slice(1, ik[u][1]);
        if constexpr (PROD) {
          widen<T>(w2r[u], w2p[u]);
#pragma unroll
          for (int k = 2; k < NI; ++k) {
            float tk[V];
            widen<T>(slice(k, ik[u][k]), tk);
#pragma unroll
            for (int c = 0; c < V; ++c) w2p[u][c] *= tk[c];
          }
        }
        cnr[u] = make_uint4(0u, 0u, 0u, 0u);
        if (nr[u]) cnr[u] = slice(0, ik[u][0]);
      }
      // the next trip's indices (the next segment's first trip at a segment's end)
      const bool seg_end = k0 + U >= Ls;
      const Seg& Sn = seg_end ? Sq : S;
      Ld nxt;
      load_trip(nxt, Sn, seg_end ? 0 : k0 + U);
      float crow_n[V], arow_n[LOSS ? 1 : GJ];
#pragma unroll
      for (int c = 0; c < V; ++c) crow_n[c] = crow[c];
#pragma unroll
      for (int u = 0; u < (LOSS ? 1 : GJ); ++u) arow_n[u] = arow[u];
      if (seg_end) row_loads(Sq, crow_n, arow_n);
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float w2[V];
        if constexpr (PROD) {
#pragma unroll
          for (int c = 0; c < V; ++c) w2[c] = w2p[u][c];
        } else {
          widen<T>(w2r[u], w2);
        }
        if (nr[u]) {
          // close the previous run: s += C(m+1)[j] * t
          float cn[V];
          widen<T>(cnr[u], cn);
#pragma unroll
          for (int c = 0; c < V; ++c) {
            s[c] = fmaf(c1[c], t[c], s[c]);
            t[c] = 0.f;
            c1[c] = cn[c];
            uu[c] = crow[c] * c1[c];
          }
        }
        if (vl[u]) jprev = ik[u][0];
        float d;
        if constexpr (MODE == 2) {
          d = vl[u] ? xv[u] : 0.f;
        } else {
          float xh = uu[0] * w2[0];
#pragma unroll
          for (int c = 1; c < V; ++c) xh = fmaf(uu[c], w2[c], xh);
          xh = group_sum<QL>(xh);
          if constexpr (LOSS) {
            if (vl[u] && q == 0) {
              const float er = xv[u] - xh;
              sse += (double)er * (double)er;
              if (out) out[perm[S.start + (b + k0 + u)]] = xh;
            }
            d = 0.f;
          } else {
            d = vl[u] ? (MODE == 0 ? xv[u] - xh : xh - xv[u]) : 0.f;
          }
        }
        if constexpr (!LOSS) {
#pragma unroll
          for (int c = 0; c < V; ++c) t[c] = fmaf(d, w2[c], t[c]);
        }
      }
      if (seg_end) {
        if constexpr (!LOSS) {
#pragma unroll
          for (int c = 0; c < V; ++c) s[c] = fmaf(c1[c], t[c], s[c]);
#pragma unroll
          for (int off = QL; off < 64; off <<= 1)
#pragma unroll
            for (int c = 0; c < V; ++c) s[c] += __shfl_xor(s[c], off);
          if (tseg && slot == 0)
#pragma unroll
            for (int c = 0; c < V; ++c) tseg[sg * R + V * q + c] = s[c];
#pragma unroll
          for (int u = 0; u < GJ; ++u) {
            const int j = slot + P * u;
            if (j < J)
#pragma unroll
              for (int c = 0; c < V; ++c) Gp[u][c] = fmaf(arow[u], s[c], Gp[u][c]);
          }
        }
        sg += nw;
        if (sg >= nseg) break;
        S = Sq;
        Sq = sg + nw < nseg ? segs[sg + nw] : none;
        Ls = (S.len + P - 1) / P;
        b = slot * Ls;
        e = min(S.len, b + Ls);
        jprev = -1;
#pragma unroll
        for (int c = 0; c < V; ++c) {
          crow[c] = crow_n[c];
          c1[c] = uu[c] = t[c] = s[c] = 0.f;
        }
#pragma unroll
        for (int u = 0; u < (LOSS ? 1 : GJ); ++u) arow[u] = arow_n[u];
        k0 = 0;
      } else {
        k0 += U;
      }
      cur = nxt;
    }
  }
  if constexpr (LOSS) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) sse += __shfl_xor(sse, off);
    if (lane == 0) dred[wave] = sse;
    __syncthreads();
    if (threadIdx.x == 0 && dpart) dpart[blockIdx.x] = ((dred[0] + dred[1]) + dred[2]) + dred[3];
  } else {
#pragma unroll
    for (int u = 0; u < GJ; ++u) {
      const int j = slot + P * u;
      if (j < J)
#pragma unroll
        for (int c = 0; c < V; ++c) red[wave][j * R + V * q + c] = Gp[u][c];
    }
    __syncthreads();
    for (int x = threadIdx.x; x < J * R; x += 256)
      partials[(int64_t)blockIdx.x * J * R + x] = ((red[0][x] + red[1][x]) + red[2][x]) + red[3][x];
  }
}

// Core gradient without the C cache (the Table 5 comparison; N = 3,
// J = R = 16): one segment per 16-lane group.  Lane r forms C(n)[i, r] of the
// other modes from their A rows, C(m)[row, r] once per segment, then
// s_r = sum_x e_x w_r and G[:, r] += a_row s_r.  The sixteen groups' partials
// of a workgroup are summed in a fixed order.
template <int N>
__global__ __launch_bounds__(256) void k_core_nc(const Seg* __restrict__ segs, int64_t nseg,
                                                 const int32_t* __restrict__ idx, int64_t nnz,
                                                 const float* __restrict__ val, NoC<N> nc,
                                                 const float* __restrict__ Am, const float* __restrict__ Bm,
                                                 float* __restrict__ partials) {
  constexpr int J = 16, R = 16;
  __shared__ float red[16][J * R];
  const int l = threadIdx.x & 15, grp = threadIdx.x >> 4;
  float Bc[N - 1][16];
  load_nc_cols<N>(nc, l, Bc);
  float Bmc[16], Gc[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    Bmc[j] = Bm[j * R + l];
    Gc[j] = 0.f;
  }
  const int64_t ng = (int64_t)gridDim.x * 16;
  for (int64_t sg = (int64_t)blockIdx.x * 16 + grp; sg < nseg; sg += ng) {
    const Seg S = segs[sg];
    const float arow = Am[(int64_t)S.row * J + l];
    float crow = 0.f;
    dot_bcast16(crow, arow, Bmc);  // C(m)[row, l]
    float sacc = 0.f;
    for (int t0 = 0; t0 < S.len; t0 += 16) {
      const int64_t p = S.start + min(t0 + l, S.len - 1);
      const float xv = val[p];
      int ix[N - 1];
#pragma unroll
      for (int k = 0; k < N - 1; ++k) ix[k] = idx[(int64_t)k * nnz + p];
      float w[16][1];
      gather_w_nc<N>(nc, Bc, ix, l, t0, S.len, w);
      static_for<0, 16>([&](auto SS) {
        constexpr int s = decltype(SS)::value;
        const float xh = group_sum<16>(crow * w[s][0]);
        const float e = bcast16<s>(xv) - xh;
        sacc = fmaf(e, w[s][0], sacc);  // w = 0 past the end of the segment
      });
    }
    axpy_bcast16(Gc, arow, sacc);  // G[j][l] += a_j s_l
  }
#pragma unroll
  for (int j = 0; j < 16; ++j) red[grp][j * R + l] = Gc[j];
  __syncthreads();
  for (int e = threadIdx.x; e < J * R; e += 256) {
    float acc = 0.f;
#pragma unroll
    for (int g = 0; g < 16; ++g) acc += red[g][e];
    partials[(int64_t)blockIdx.x * J * R + e] = acc;
  }
}

// Sum of the workgroup partials in a fixed order, then optionally the core
// step B <- B + lr (G / |Omega| - lam B) (Algorithm 5).  A workgroup takes 16
// entries of J x R and sums the partials in 64 chains of 16 lanes: kFold
// slices, four chains per slice, each over every fourth partial of its slice,
// so that 2048 partials are 32 independent loads per lane.  Bound by the
// latency of these loads and by the launch itself: as two launches, slices
// over all entries first, 5 + 5 us at any size; as one launch of 16 entries per
// workgroup 5 us (the same sums in the same order).
constexpr int kFold = 16;

__global__ __launch_bounds__(1024) void k_fold_update(const float* __restrict__ partials, int nparts, int JR,
                                                      float* __restrict__ Bm, float* __restrict__ Gout, float lr,
                                                      float lam, float inv_nnz, int update) {
  __shared__ float red[4 * kFold][16], fold[kFold][16];
  const int c = threadIdx.x & 15, q = threadIdx.x >> 4;
  const int e = blockIdx.x * 16 + c;  // JR is a multiple of 64
  const int per = (nparts + kFold - 1) / kFold;
  const int b0 = (q >> 2) * per, b1 = min(nparts, b0 + per);
  float s = 0.f;
#pragma unroll 16
  for (int b = b0 + (q & 3); b < b1; b += 4) s += partials[(int64_t)b * JR + e];
  red[q][c] = s;
  __syncthreads();
  if (q < kFold) fold[q][c] = ((red[4 * q][c] + red[4 * q + 1][c]) + red[4 * q + 2][c]) + red[4 * q + 3][c];
  __syncthreads();
  if (q > 0) return;
  s = 0.f;
#pragma unroll
  for (int b = 0; b < kFold; ++b) s += fold[b][c];
  if (Gout) Gout[e] = s;
  if (update) {
    const float b = Bm[e];
    Bm[e] = b + lr * (s * inv_nnz - lam * b);
  }
}

// dA(m)[i, j] = sum_r B(m)[j, r] t_i[r], t_i = sum of the row's segment sums:
// 16 rows per wavefront, lane (i, g) summing a slice of row i's segments, and
// B t on the matrix cores.  The segment sums are added in FP64, so that a
// row's error is that of its segments (FP32, at most 512 elements each)
// however many it has: added in FP32, 678 segments of 192 elements had twice
// the error of the same row in 254 of 512.  What bounds the launch is the
// latency of the longest row's loads: eight are in flight, and a row of more
// than kSerialSegs segments is summed by the whole wavefront, 16 segments at a
// time and then over 16 lanes in a fixed tree (about 2 us a row, which fewer
// segments do not repay: with 16 in place of 128, 40 us).  Planted shape, 1M
// elements, J = R = 16, us per mode: 26 in one chain per row, 19 so.
constexpr int kSerialSegs = 128;

template <int J, int R, class T>
__global__ __launch_bounds__(256) void k_grad_rows(const int64_t* __restrict__ seg_first,
                                                   const int64_t* __restrict__ row_ptr,
                                                   const float* __restrict__ tseg, const T* __restrict__ Bm,
                                                   float* __restrict__ gA, int64_t I, int seg_len) {
  constexpr int KR = R / 4;
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int64_t row = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 16 + i;
  if (row - i >= I) return;
  GForm<J, R, T> gf;
  gf.load(Bm, i, g);
  const int64_t rc = min(row, I - 1);
  const int n = row < I ? (int)((row_ptr[rc + 1] - row_ptr[rc] + seg_len - 1) / seg_len) : 0;
  const int64_t first = seg_first[rc];
  double t[KR];
#pragma unroll
  for (int c = 0; c < KR; ++c) t[c] = 0.0;
  // segment sums k0, k0 + step, ... below count, eight loads in flight
  auto add = [&](const float* src, int k0, int step, int count, double (&s)[KR]) {
    for (int k = k0; k < count; k += 8 * step) {
      float x[8][KR];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int c = 0; c < KR; ++c) x[u][c] = src[(int64_t)min(k + u * step, count - 1) * R + c];
#pragma unroll
      for (int u = 0; u < 8; ++u)
#pragma unroll
        for (int c = 0; c < KR; ++c) s[c] += k + u * step < count ? (double)x[u][c] : 0.0;
    }
  };
  add(tseg + first * R + KR * g, 0, 1, n <= kSerialSegs ? n : 0, t);
  // (the four lanes of a row agree on n; the low 16 bits are those of the lanes of g = 0)
  for (uint32_t todo = (uint32_t)__ballot(n > kSerialSegs) & 0xFFFFu; todo; todo &= todo - 1) {
    const int r = __builtin_ctz(todo);
    const int nr = __shfl(n, r);
    const float* src = tseg + (int64_t)__shfl(first, r) * R + KR * g;
    double s[KR];
#pragma unroll
    for (int c = 0; c < KR; ++c) s[c] = 0.0;
    add(src, i, 16, nr, s);
#pragma unroll
    for (int off = 1; off < 16; off <<= 1)
#pragma unroll
      for (int c = 0; c < KR; ++c) s[c] += __shfl_xor(s[c], off);
    if (i == r)
#pragma unroll
      for (int c = 0; c < KR; ++c) t[c] = s[c];
  }
  float tf[KR], G[JLayout<J>::NG];
#pragma unroll
  for (int c = 0; c < KR; ++c) tf[c] = (float)t[c];
  gf.form(tf, G);
  if (row < I)
#pragma unroll
    for (int k = 0; k < JLayout<J>::NG; ++k) gA[row * J + JLayout<J>::jbase(g) + k] = G[k];
}

// Loss: per-element e^2 summed in FP64 (and, with out != nullptr, xhat stored
// at the element's input position).
template <int N, int R, class T>
__global__ __launch_bounds__(256) void k_loss(const Seg* __restrict__ segs, int64_t nseg,
                                              const int32_t* __restrict__ idx, int64_t nnz,
                                              const float* __restrict__ val, CPtrs<N, T> cp,
                                              const T* __restrict__ Cm, double* __restrict__ dpart,
                                              const int32_t* __restrict__ perm, float* __restrict__ out) {
  constexpr int V = vpl<T>();
  constexpr int QL = R / V;
  constexpr int P = 64 / QL;
  constexpr int U = trip_unroll<N>();
  __shared__ double red[4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = lane / QL, q = lane % QL;
  const int64_t nw = (int64_t)gridDim.x * 4;
  double sse = 0.0;
  int64_t sg = (int64_t)blockIdx.x * 4 + wave;
  if (sg < nseg) {
    const Seg none{0, 0, 0};
    Seg S = segs[sg];
    Seg Sq = sg + nw < nseg ? segs[sg + nw] : none;
    float crow[V];
    load16(Cm + (int64_t)S.row * R + V * q, crow);
    Trip<N, P> cur;
    load_trip<N, P, false>(cur, S, 0, lane, idx, nnz, val, nullptr);
    int t0 = 0;
    for (;;) {
      int32_t ik[U][N > 1 ? N - 1 : 1];
      float xv[U];
      bool vl[U];
      static_for<0, U>([&](auto UU) {
        constexpr int u = decltype(UU)::value;
        trip_elem<N, P, u>(cur, slot, ik[u], xv[u]);
        vl[u] = t0 + u * P + slot < S.len;
      });
      float w[U][V];
#pragma unroll
      for (int u = 0; u < U; ++u) gather_slices<N, R, T>(cp, ik[u], vl[u], q, w[u]);
      const bool seg_end = t0 + P * U >= S.len;
      const Seg& Sn = seg_end ? Sq : S;
      Trip<N, P> nxt;
      load_trip<N, P, false>(nxt, Sn, seg_end ? 0 : t0 + P * U, lane, idx, nnz, val, nullptr);
      float crow_n[V];
      if (seg_end) {
        load16(Cm + (int64_t)Sq.row * R + V * q, crow_n);
      } else {
#pragma unroll
        for (int c = 0; c < V; ++c) crow_n[c] = crow[c];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float xh = crow[0] * w[u][0];
#pragma unroll
        for (int c = 1; c < V; ++c) xh = fmaf(crow[c], w[u][c], xh);
        xh = group_sum<QL>(xh);
        if (vl[u] && q == 0) {
          const float e = xv[u] - xh;
          sse += (double)e * (double)e;
          if (out) out[perm[S.start + (t0 + u * P + slot)]] = xh;
        }
      }
      if (seg_end) {
        sg += nw;
        if (sg >= nseg) break;
        S = Sq;
        Sq = sg + nw < nseg ? segs[sg + nw] : none;
        t0 = 0;
      } else {
        t0 += P * U;
      }
#pragma unroll
      for (int c = 0; c < V; ++c) crow[c] = crow_n[c];
      cur = nxt;
    }
  }
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) sse += __shfl_xor(sse, off);
  if (lane == 0) red[wave] = sse;
  __syncthreads();
  if (threadIdx.x == 0 && dpart) dpart[blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// FP64 sums of squares of every A(n), one launch: workgroup (x, n) adds its
// share of A(n) in 16-byte loads (four bytes where A(n) starts off a 16-byte
// boundary), four accumulators per thread.  One launch of 16-byte loads
// instead of two per mode of four-byte ones: a 1e6 x 32 matrix 190 us -> 30 us.
struct SumsqArgs {
  const float* X[FT_MAX_ORDER];
  int64_t n[FT_MAX_ORDER];
};

__global__ __launch_bounds__(256) void k_sumsq(SumsqArgs a, double* __restrict__ dpart) {
  __shared__ double red[4];
  const float* __restrict__ X = a.X[blockIdx.y];
  const int64_t n = a.n[blockIdx.y];
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, nt = (int64_t)gridDim.x * 256;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  int64_t tail = 0;
  if ((reinterpret_cast<uintptr_t>(X) & 15) == 0) {
    const floatx4* X4 = reinterpret_cast<const floatx4*>(X);
#pragma unroll 4
    for (int64_t k = t; k < n / 4; k += nt) {
      const floatx4 v = X4[k];
#pragma unroll
      for (int c = 0; c < 4; ++c) s[c] = fma((double)v[c], (double)v[c], s[c]);
    }
    tail = n & ~(int64_t)3;
  }
  for (int64_t k = tail + t; k < n; k += nt) s[0] = fma((double)X[k], (double)X[k], s[0]);
  double v = (s[0] + s[1]) + (s[2] + s[3]);
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) v += __shfl_xor(v, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) dpart[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = ((red[0] + red[1]) + red[2]) + red[3];
}

// Fixed-order FP64 sums of the partials and of the (small) B(n), strided per
// thread, then a tree.
__global__ __launch_bounds__(256) void k_loss_finish(const double* __restrict__ dpart, int n_sse,
                                                     const double* __restrict__ rpart, int n_a, SumsqArgs B, int N,
                                                     double nnz, double lam_a, double lam_b,
                                                     double* __restrict__ out4) {
  __shared__ double red[3][4];
  const int t = threadIdx.x;
  double v[3] = {0.0, 0.0, 0.0};
#pragma unroll 8
  for (int k = t; k < n_sse; k += 256) v[0] += dpart[k];
#pragma unroll 4
  for (int k = t; k < n_a; k += 256) v[1] += rpart[k];
  for (int m = 0; m < N; ++m)
#pragma unroll 4
    for (int k = t; k < (int)B.n[m]; k += 256) v[2] = fma((double)B.X[m][k], (double)B.X[m][k], v[2]);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) v[c] += __shfl_xor(v[c], off);
    if ((t & 63) == 0) red[c][t >> 6] = v[c];
  }
  __syncthreads();
  if (t == 0) {
    double f[3];
    for (int c = 0; c < 3; ++c) f[c] = ((red[c][0] + red[c][1]) + red[c][2]) + red[c][3];
    out4[0] = f[0];
    out4[1] = nnz > 0 ? sqrt(f[0] / nnz) : 0.0;
    out4[2] = lam_a * f[1];
    out4[3] = lam_b * f[2];
  }
}

// Predictions for query coordinates (structure of arrays [N][q]).  A wavefront
// takes 64 queries: lane l loads the coordinates of query l (64 distinct
// addresses per load), then the R / V lanes of each slot gather 16-byte slices
// of its rows, 64 V / R queries at a time, with the indices handed over by
// cross-lane permutes.  What bounds it is the rate at which a CU's memory path
// returns the gathered rows, and index loads that repeat an address over the
// lanes of a row take half of its issue slots.  With `bad`, an index outside
// its dimension is replaced by 0 before the gather and marks bad[n] (every
// writer stores the same value).
struct DimArgs {
  int32_t d[FT_MAX_ORDER];
};

template <int N, int R, class T, bool CHECK>
__global__ __launch_bounds__(256) void k_predict(const int32_t* __restrict__ coords, int64_t q, CPtrs<N + 1, T> cp,
                                                 float* __restrict__ out, DimArgs dims, int32_t* __restrict__ bad) {
  constexpr int V = vpl<T>();
  constexpr int QL = R / V;
  constexpr int P = 64 / QL;
  const int lane = threadIdx.x & 63, slot = lane / QL, qq = lane % QL;
  const int64_t x0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64;
  if (x0 >= q) return;
  int32_t ik[N];
#pragma unroll
  for (int n = 0; n < N; ++n) {
    ik[n] = coords[(int64_t)n * q + min(x0 + lane, q - 1)];
    if constexpr (CHECK) {
      const bool off = (uint32_t)ik[n] >= (uint32_t)dims.d[n];
      if (off) bad[n] = 1;
      ik[n] = off ? 0 : ik[n];
    }
  }
  const uint32_t qb = (uint32_t)(16 * qq);
  static_for<0, QL>([&](auto UU) {
    constexpr int u = decltype(UU)::value;
    float w[V];
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int32_t i = QL > 1 ? __shfl(ik[n], u * P + slot) : ik[n];
      float t[V];
      load16(reinterpret_cast<const T*>(reinterpret_cast<const char*>(cp.p[n]) +
                                        ((uint32_t)i * (uint32_t)(R * sizeof(T)) + qb)),
             t);
#pragma unroll
      for (int c = 0; c < V; ++c) w[c] = n == 0 ? t[c] : w[c] * t[c];
    }
    float s = w[0];
#pragma unroll
    for (int c = 1; c < V; ++c) s += w[c];
    s = group_sum<QL>(s);
    const int64_t x = x0 + u * P + slot;
    if (x < q && qq == 0) out[x] = s;
  });
}

__global__ void k_clear(int32_t* __restrict__ p, int n) {
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0;
}

hipError_t reduce_partials(const ft_plan* P, const Scratch& S, int nparts, float* Bm, float* Gout, float lr,
                           float lam, float inv, int update, hipStream_t s) {
  KTimer tm(P, FT_K_REDUCE, s);
  const int JR = P->J * P->R;
  hipLaunchKernelGGL(k_fold_update, dim3(JR / 16), dim3(64 * kFold), 0, s, S.partials, nparts, JR, Bm, Gout, lr, lam,
                     inv, update);
  return hipGetLastError();
}

// workgroups for the work of `waves` wavefronts, at most those resident
int seg_blocks(const void* kernel, int64_t waves) {
  int64_t b = (waves + 3) / 4;
  b = std::min<int64_t>(b, std::min(kPartials, resident_blocks(kernel)));
  if (b < 1) b = 1;
  return (int)b;
}

template <int N, int J, int R, class T>
hipError_t segsum_impl(const ft_plan* P, int m, const ft_params* p, float* partials, int mode, const float* up,
                       float* tseg, hipStream_t s, int* nblocks) {
  const ModeMeta& M = P->meta[m];
  const ModeDev& D = P->dev[m];
  const CPtrs<N, T> cp = others<N, T>(p, m);
  const T* Cm = Store<T>::C(p, m);
  const T* Am = Store<T>::A(p, m);
  // modes 0 and 1 (the core gradient and the gradient of 1/2 sum e^2) launch
  // the same grid, so their sums run in the same order and one is the exact
  // negation of the other
  if constexpr (N >= 3) {
    if (P->run_reuse) {
      const void* kr = mode == 2 ? (const void*)k_segrun<N, J, R, 2, T> : (const void*)k_segrun<N, J, R, 0, T>;
      const int nbr = seg_blocks(kr, M.n_segs);
      *nblocks = nbr;
      KTimer tm(P, FT_K_SEGSUM, s);
      if (mode == 0)
        hipLaunchKernelGGL((k_segrun<N, J, R, 0, T>), dim3(nbr), dim3(256), 0, s, D.segs, M.n_segs, D.idx, P->nnz,
                           D.val, cp, Cm, Am, nullptr, nullptr, partials, tseg, nullptr, nullptr);
      else if (mode == 1)
        hipLaunchKernelGGL((k_segrun<N, J, R, 1, T>), dim3(nbr), dim3(256), 0, s, D.segs, M.n_segs, D.idx, P->nnz,
                           D.val, cp, Cm, Am, nullptr, nullptr, partials, tseg, nullptr, nullptr);
      else
        hipLaunchKernelGGL((k_segrun<N, J, R, 2, T>), dim3(nbr), dim3(256), 0, s, D.segs, M.n_segs, D.idx, P->nnz,
                           D.val, cp, Cm, Am, up, D.perm, partials, tseg, nullptr, nullptr);
      return hipGetLastError();
    }
  }
  const void* kern = mode == 2 ? (const void*)k_segsum<N, J, R, 2, T> : (const void*)k_segsum<N, J, R, 0, T>;
  const void* kshort = mode == 2 ? (const void*)k_segshort<N, J, R, 2, T> : (const void*)k_segshort<N, J, R, 0, T>;
  const int64_t n_short = M.n_segs - M.n_long_segs;
  // the two kernels' partials share the scratch: at most half of it each where both run
  const int most = n_short > 0 ? kPartials / 2 : kPartials;
  const int nb = M.n_long_segs > 0 || n_short == 0 ? std::min(most, seg_blocks(kern, M.n_long_segs)) : 0;
  constexpr int per_wave = 64 * vpl<T>() / R;
  const int nbs = n_short > 0 ? std::min(most, seg_blocks(kshort, (n_short + per_wave - 1) / per_wave)) : 0;
  *nblocks = nb + nbs;
  float* pshort = partials + (int64_t)nb * J * R;
  KTimer tm(P, FT_K_SEGSUM, s);
#define FT_SEGSUM(MODE, UP, PERM)                                                                                     \
  do {                                                                                                                \
    if (nb > 0)                                                                                                       \
      hipLaunchKernelGGL((k_segsum<N, J, R, MODE, T>), dim3(nb), dim3(256), 0, s, D.segs, M.n_long_segs, D.idx,       \
                         P->nnz, D.val, cp, Cm, Am, UP, PERM, partials, tseg);                                        \
    if (nbs > 0)                                                                                                      \
      hipLaunchKernelGGL((k_segshort<N, J, R, MODE, T>), dim3(nbs), dim3(256), 0, s, D.segs, M.n_long_segs, n_short,  \
                         D.idx, P->nnz, D.val, cp, Cm, Am, UP, PERM, pshort, tseg);                                   \
  } while (0)
  if (mode == 0)
    FT_SEGSUM(0, nullptr, nullptr);
  else if (mode == 1)
    FT_SEGSUM(1, nullptr, nullptr);
  else
    FT_SEGSUM(2, up, D.perm);
#undef FT_SEGSUM
  return hipGetLastError();
}

// dpart: kPartials FP64 partials of the loss kernel, then N kSumsqBlocks of
// the A(n).
template <int N, int J, int R, class T>
hipError_t loss_impl(const ft_plan* P, const ft_params* p, double* dpart, double lam_a, double lam_b, double* out4,
                     float* xout, hipStream_t s) {
  // the loss is a sum over all elements: any mode's CSR serves (P->loss_mode)
  const int lm = P->loss_mode;
  const ModeMeta& M = P->meta[lm];
  const ModeDev& D = P->dev[lm];
  const CPtrs<N, T> cp = others<N, T>(p, lm);
  int nb = 0;
  if constexpr (N >= 3) {
    if (P->run_reuse) {
      nb = seg_blocks((const void*)k_segrun<N, J, R, 3, T>, M.n_segs);
      KTimer tm(P, FT_K_LOSS, s);
      hipLaunchKernelGGL((k_segrun<N, J, R, 3, T>), dim3(nb), dim3(256), 0, s, D.segs, M.n_segs, D.idx, P->nnz,
                         D.val, cp, Store<T>::C(p, lm), nullptr, nullptr, D.perm, nullptr, nullptr,
                         out4 ? dpart : nullptr, xout);
    }
  }
  if (nb == 0) {
    nb = seg_blocks((const void*)k_loss<N, R, T>, M.n_segs);
    KTimer tm(P, FT_K_LOSS, s);
    hipLaunchKernelGGL((k_loss<N, R, T>), dim3(nb), dim3(256), 0, s, D.segs, M.n_segs, D.idx, P->nnz, D.val, cp,
                       Store<T>::C(p, lm), out4 ? dpart : nullptr, D.perm, xout);
  }
  if (!out4) return hipGetLastError();
  // the regularisers of Eq. (6) are taken on the FP32 masters
  KTimer tm(P, FT_K_REDUCE, s);
  double* rpart = dpart + kPartials;
  SumsqArgs a{}, bm{};
  int64_t most = 0;
  for (int n = 0; n < N; ++n) {
    a.X[n] = p->A[n];
    a.n[n] = P->desc.dims[n] * J;
    most = std::max(most, a.n[n]);
    bm.X[n] = p->B[n];
    bm.n[n] = (int64_t)J * R;
  }
  // a thread adds at least 16 values; the grid is the largest matrix's for all
  const int nx = (int)std::min<int64_t>(kSumsqBlocks, std::max<int64_t>(1, most / (256 * 16)));
  hipLaunchKernelGGL(k_sumsq, dim3(nx, N), dim3(256), 0, s, a, rpart);
  hipLaunchKernelGGL(k_loss_finish, dim3(1), dim3(256), 0, s, dpart, nb, rpart, nx * N, bm, N, (double)P->nnz, lam_a,
                     lam_b, out4);
  return hipGetLastError();
}

template <int N, int R, class T>
hipError_t predict_impl(const ft_plan* P, const ft_params* p, const int32_t* coords, int64_t q, float* out,
                        int32_t* bad, hipStream_t s) {
  CPtrs<N + 1, T> cp{};
  DimArgs dims{};
  for (int n = 0; n < N; ++n) {
    cp.p[n] = Store<T>::C(p, n);
    dims.d[n] = (int32_t)P->desc.dims[n];
  }
  const unsigned nb = (unsigned)((q + 255) / 256);
  if (bad) {
    hipLaunchKernelGGL(k_clear, dim3(1), dim3(64), 0, s, bad, N);
    hipLaunchKernelGGL((k_predict<N, R, T, true>), dim3(nb), dim3(256), 0, s, coords, q, cp, out, dims, bad);
  } else {
    hipLaunchKernelGGL((k_predict<N, R, T, false>), dim3(nb), dim3(256), 0, s, coords, q, cp, out, dims, bad);
  }
  return hipGetLastError();
}

template <int J, int R, class T>
hipError_t grad_rows_impl(const ft_plan* P, int m, const ft_params* p, const float* tseg, float* gA, hipStream_t s) {
  const int64_t I = P->desc.dims[m];
  const unsigned gb = (unsigned)((I + 63) / 64);
  if (gb > 0)
    hipLaunchKernelGGL((k_grad_rows<J, R, T>), dim3(gb), dim3(256), 0, s, P->dev[m].seg_first, P->dev[m].row_ptr, tseg,
                       Store<T>::B(p, m), gA, I, P->seg_len);
  return hipGetLastError();
}

}  // namespace

static hipError_t segsum(const ft_plan* P, int m, const ft_params* p, float* partials, int mode, const float* up,
                         float* tseg, hipStream_t s, int* nb) {
#define X(n, j, r)                                                                             \
  case key(n, j, r):                                                                           \
    return bf16(p) ? segsum_impl<n, j, r, uint16_t>(P, m, p, partials, mode, up, tseg, s, nb) \
                   : segsum_impl<n, j, r, float>(P, m, p, partials, mode, up, tseg, s, nb);
  FT_DISPATCH()
#undef X
}

// core gradient partials without the C cache (N = 3, J = R = 16, FP32 only)
static hipError_t core_nc(const ft_plan* P, int m, const ft_params* p, float* partials, hipStream_t s, int* nb) {
  if (P->N != 3 || P->J != 16 || P->R != 16 || bf16(p)) return hipErrorInvalidValue;
  const ModeMeta& M = P->meta[m];
  const ModeDev& D = P->dev[m];
  NoC<3> nc{};
  for (int k = 0; k < 2; ++k) {
    nc.A[k] = p->A[(m + 1 + k) % 3];
    nc.B[k] = p->B[(m + 1 + k) % 3];
  }
  int64_t b = (M.n_segs + 15) / 16;
  b = std::max<int64_t>(1, std::min<int64_t>(b, std::min(kPartials, resident_blocks((const void*)k_core_nc<3>))));
  *nb = (int)b;
  KTimer tm(P, FT_K_SEGSUM, s);
  hipLaunchKernelGGL(k_core_nc<3>, dim3((unsigned)b), dim3(256), 0, s, D.segs, M.n_segs, D.idx, P->nnz, D.val, nc,
                     p->A[m], p->B[m], partials);
  return hipGetLastError();
}

hipError_t launch_core_grad(const ft_plan* P, int m, const ft_params* p, const Scratch& S, float* G_out,
                            hipStream_t s) {
  int nb = 0;
  hipError_t e = P->no_c_cache ? core_nc(P, m, p, S.partials, s, &nb)
                               : segsum(P, m, p, S.partials, 0, nullptr, nullptr, s, &nb);
  if (e != hipSuccess) return e;
  return reduce_partials(P, S, nb, nullptr, G_out, 0.f, 0.f, 0.f, 0, s);
}

hipError_t launch_core_update(const ft_plan* P, int m, const ft_params* p, const Scratch& S, double lr, double lam,
                              hipStream_t s) {
  int nb = 0;
  hipError_t e = P->no_c_cache ? core_nc(P, m, p, S.partials, s, &nb)
                               : segsum(P, m, p, S.partials, 0, nullptr, nullptr, s, &nb);
  if (e != hipSuccess) return e;
  const float inv = P->nnz > 0 ? (float)(1.0 / (double)P->nnz) : 0.f;
  return reduce_partials(P, S, nb, p->B[m], nullptr, (float)lr, (float)lam, inv, P->nnz > 0 ? 1 : 0, s);
}

hipError_t launch_loss(const ft_plan* P, const ft_params* p, const Scratch& S, double lam_a, double lam_b,
                       double* out4, hipStream_t s) {
#define X(n, j, r)                                                                             \
  case key(n, j, r):                                                                           \
    return bf16(p) ? loss_impl<n, j, r, uint16_t>(P, p, S.dpartials, lam_a, lam_b, out4, nullptr, s) \
                   : loss_impl<n, j, r, float>(P, p, S.dpartials, lam_a, lam_b, out4, nullptr, s);
  FT_DISPATCH()
#undef X
}

// forward writes no partials (the loss kernel stores xhat only)
hipError_t launch_forward(const ft_plan* P, const ft_params* p, const Scratch&, float* out, hipStream_t s) {
#define X(n, j, r)                                                                             \
  case key(n, j, r):                                                                           \
    return bf16(p) ? loss_impl<n, j, r, uint16_t>(P, p, nullptr, 0.0, 0.0, nullptr, out, s)   \
                   : loss_impl<n, j, r, float>(P, p, nullptr, 0.0, 0.0, nullptr, out, s);
  FT_DISPATCH()
#undef X
}

hipError_t launch_predict(const ft_plan* P, const ft_params* p, const int32_t* coords, int64_t q, float* out,
                          int32_t* bad, hipStream_t s) {
#define X(n, j, r)                                                                             \
  case key(n, j, r):                                                                           \
    return bf16(p) ? predict_impl<n, r, uint16_t>(P, p, coords, q, out, bad, s)               \
                   : predict_impl<n, r, float>(P, p, coords, q, out, bad, s);
  FT_DISPATCH()
#undef X
}

hipError_t launch_grad(const ft_plan* P, const ft_params* p, const Scratch& S, const float* up, float* const* gA,
                       float* const* gB, hipStream_t s) {
  for (int m = 0; m < P->N; ++m) {
    int nb = 0;
    hipError_t e = segsum(P, m, p, S.partials, up ? 2 : 1, up, S.tseg, s, &nb);
    if (e != hipSuccess) return e;
    switch (P->J * 64 + P->R) {
#define X(n_, j, r)                                                                                        \
  case j * 64 + r:                                                                                         \
    e = bf16(p) ? grad_rows_impl<j, r, uint16_t>(P, m, p, S.tseg, gA[m], s)                               \
                : grad_rows_impl<j, r, float>(P, m, p, S.tseg, gA[m], s);                                 \
    break;
      X(0, 8, 8) X(0, 16, 16) X(0, 32, 32) X(0, 8, 16)
#undef X
      default: return hipErrorInvalidValue;
    }
    if (e != hipSuccess) return e;
    e = reduce_partials(P, S, nb, nullptr, gB[m], 0.f, 0.f, 0.f, 0, s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Scratch of ft_loss_noalloc: the FP64 partials of the loss kernel (at most
// kPartials workgroups) followed by those of the sums of squares of A(n)
// (N kSumsqBlocks), in a device array that the library holds on every GPU
// it runs on until the process ends.  Host code uses the address looked up
// per device below, never the array's name.
constexpr size_t kNoAllocDoubles = (size_t)kPartials + FT_MAX_ORDER * kSumsqBlocks;
static __device__ __align__(256) double scratch[kNoAllocDoubles];

size_t noalloc_loss_capacity() { return sizeof(double) * kNoAllocDoubles; }

size_t noalloc_loss_need(const ft_plan* P) {
  return sizeof(double) * ((size_t)kPartials + (size_t)P->N * kSumsqBlocks);
}

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_noalloc_mu;
double* g_noalloc_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device: looked up on the first
// call on each device (with that device current) and kept.
hipError_t noalloc_scratch(double** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_noalloc_mu);
  if (!g_noalloc_ptr[dev]) {
    void* addr = nullptr;
    e = hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!addr) return hipErrorInvalidSymbol;
    g_noalloc_ptr[dev] = static_cast<double*>(addr);
  }
  *out = g_noalloc_ptr[dev];
  return hipSuccess;
}
}  // namespace

hipError_t launch_loss_noalloc(const ft_plan* P, const ft_params* p, double lam_a, double lam_b, double* out4,
                               hipStream_t s) {
  double* d = nullptr;
  hipError_t e = noalloc_scratch(&d);
  if (e != hipSuccess) return e;
  Scratch S{};
  S.dpartials = d;
  // kernel timing creates events; this path creates nothing
  const UntimedScope untimed;
  return launch_loss(P, p, S, lam_a, lam_b, out4, s);
}

}  // namespace ft
