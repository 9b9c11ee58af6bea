// HIP kernels of the R3MG-C hot path for gfx950 (CDNA4, wave64).
//
// Level operators (paper Section 4: inherited operators A_i = P_i^T A P_i) are applied by one fused kernel
// that also performs the Chebyshev-accelerated Jacobi update of the smoother (Section 5 Remark on the
// smoother, Section 6): t = A u; rho -= t; x += u; d = c1 u + c2 D^{-1} rho.  The fine level is CSR; the
// agglomerated levels store dense B x B blocks (B = (p'+1)^d) with one column index per block, laid out so
// that every row's values are contiguous ("block rows": row (K,q) holds blocks j = 0..nb-1, columns c).
// Transfers (Section 4 construction of P_{M-1} and P~) evaluate the box basis on the fly from per-point
// local coordinates; they never store P.
//
// All reductions are deterministic: fixed per-thread order, fixed shuffle trees, fixed LDS trees, and
// per-block partials summed in index order by a single block.  No floating-point atomics.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstdio>
#include <algorithm>
#include <stdexcept>
#include <string>

#include "hip_util.h"
#include "kernels.h"

namespace r3mg {

namespace {

using hiputil::check_launch;
using hiputil::xcd_block;
using hiputil::xcd_grid;

typedef double v4d __attribute__((ext_vector_type(4)));

template <typename T>
struct Basis1D {
  T t[4];
  T w[4];
  int k;
};

template <typename T>
Basis1D<T> make_basis(int pc) {
  double t[4] = {0, 0, 0, 0};
  switch (pc) {
    case 0: t[0] = 0.5; break;
    case 1: t[0] = 0.0; t[1] = 1.0; break;
    case 2: t[0] = 0.0; t[1] = 0.5; t[2] = 1.0; break;
    default: {
      double s = 1.0 / std::sqrt(5.0);
      t[0] = 0.0; t[1] = 0.5 * (1.0 - s); t[2] = 0.5 * (1.0 + s); t[3] = 1.0;
    }
  }
  Basis1D<T> b;
  b.k = pc + 1;
  for (int j = 0; j < 4; ++j) {
    double w = 1.0;
    for (int m = 0; m < b.k; ++m)
      if (m != j && j < b.k) w /= (t[j] - t[m]);
    b.t[j] = (T)t[j];
    b.w[j] = (T)w;
  }
  return b;
}

// l_j(s) = w_j prod_{m != j} (s - t_m) for KB nodes
template <typename T, int KB>
__device__ inline void lag1d_k(const Basis1D<T>& bs, T s, T* l) {
#pragma unroll
  for (int j = 0; j < KB; ++j) {
    T v = bs.w[j];
#pragma unroll
    for (int m = 0; m < KB; ++m)
      if (m != j) v *= (s - bs.t[m]);
    l[j] = v;
  }
}
// calls f(q, phi_q) for q = 0 .. KB^D - 1 in ascending order
template <typename T, int D, int KB, typename F>
__device__ inline void for_each_phi(const T (*l)[4], F&& f) {
  int q = 0;
#pragma unroll
  for (int q2 = 0; q2 < (D == 3 ? KB : 1); ++q2)
#pragma unroll
    for (int q1 = 0; q1 < KB; ++q1)
#pragma unroll
      for (int q0 = 0; q0 < KB; ++q0) {
        T v = l[0][q0] * l[1][q1];
        if (D == 3) v *= l[2][q2];
        f(q++, v);
      }
}

// phi_q of multi-index q = q0 + k q1 + k^2 q2 from 1D tables l[a][.]
template <typename T>
__device__ inline T phi_q(const T (*l)[4], int d, int k, int q) {
  T v = l[0][q % k];
  q /= k;
  v *= l[1][q % k];
  if (d == 3) {
    q /= k;
    v *= l[2][q % k];
  }
  return v;
}

template <typename T>
__device__ inline T wave_sum(T v, int width) {
  for (int off = width >> 1; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Sums of S values over the 64 lanes of a wave (S a power of two, at most 64) by a transposing butterfly: each step
// halves the values a lane carries.  Returns the sum of value `slot` (every S-th lane group holds the same slots), in
// an order that does not depend on the lane.
template <typename T, int S, int H = S / 2, int OFF = 32>
__device__ __forceinline__ T wave_sum_slots(T (&v)[S], int lane, int& slot) {
  if constexpr (H >= 1) {
    const bool up = lane & OFF;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      const T keep = up ? v[i + H] : v[i], send = up ? v[i] : v[i + H];
      v[i] = keep + __shfl_xor(send, OFF, 64);
    }
    slot += up ? H : 0;
    return wave_sum_slots<T, S, H / 2, OFF / 2>(v, lane, slot);
  } else {
#pragma unroll
    for (int off = OFF; off >= 1; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
    return v[0];
  }
}
constexpr int pow2_at_least(int b) { return b <= 1 ? 1 : 2 * pow2_at_least((b + 1) / 2); }

// deterministic block sum (blockDim.x = 256): returns the total in thread 0
__device__ inline double block_sum256(double v, double* sh) {
  v = wave_sum(v, 64);
  int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double r = 0;
  if (threadIdx.x == 0) r = (sh[0] + sh[1]) + (sh[2] + sh[3]);
  __syncthreads();
  return r;
}

}  // namespace

// =============================================================================================
// Fused level kernel: t = A u (CSR or block rows), then the smoother update epilogue.
// G lanes per row (power of two), 256 threads per block, NR right-hand sides interleaved.
// =============================================================================================
template <typename T, int NR, bool BLOCKED>
__device__ inline void row_product(int row, int lane, int G, int blk, const int* __restrict__ ptr,
                                   const int* __restrict__ idx, const T* __restrict__ val,
                                   const T* __restrict__ u, T* acc) {
  if (!BLOCKED) {
    // UNR steps per batch: their column, value and u loads are all in flight before the products (each lane
    // still accumulates its entries in ascending order)
    constexpr int UNR = NR >= 16 ? 2 : 32 / NR;
    const int s = ptr[row], e = ptr[row + 1];
    for (int p0 = s + lane; p0 < e; p0 += UNR * G) {
      T a[UNR];
      int64_t c[UNR];
#pragma unroll
      for (int m = 0; m < UNR; ++m) {
        const int p = p0 + m * G;
        a[m] = p < e ? val[p] : (T)0;
        c[m] = p < e ? (int64_t)idx[p] * NR : 0;
      }
      T uv[UNR][NR];
      constexpr int VW = 16 / (int)sizeof(T);  // entries per 16-byte load (u rows are NR-aligned)
      if constexpr (NR % VW == 0) {
        typedef T V16 __attribute__((ext_vector_type(VW)));
#pragma unroll
        for (int m = 0; m < UNR; ++m)
#pragma unroll
          for (int k = 0; k < NR; k += VW) {
            const V16 t = *reinterpret_cast<const V16*>(u + c[m] + k);
#pragma unroll
            for (int w = 0; w < VW; ++w) uv[m][k + w] = t[w];
          }
      } else {
#pragma unroll
        for (int m = 0; m < UNR; ++m)
#pragma unroll
          for (int k = 0; k < NR; ++k) uv[m][k] = u[c[m] + k];
      }
#pragma unroll
      for (int m = 0; m < UNR; ++m)
#pragma unroll
        for (int k = 0; k < NR; ++k) acc[k] += a[m] * uv[m][k];
    }
  } else {
    const int K = row / blk;
    const int q = row - K * blk;
    const int j0 = ptr[K];
    const int nb = ptr[K + 1] - j0;
    const int64_t vbase = (int64_t)blk * blk * j0 + (int64_t)q * nb * blk;
    const int len = nb * blk;
    int j = lane / blk, c = lane - j * blk;
    const int sj = G / blk, sc = G - sj * blk;
    for (int p = lane; p < len; p += G) {
      const int64_t cc = ((int64_t)idx[j0 + j] * blk + c) * NR;
      const T a = val[vbase + p];
#pragma unroll
      for (int k = 0; k < NR; ++k) acc[k] += a * u[cc + k];
      j += sj;
      c += sc;
      if (c >= blk) { c -= blk; ++j; }
    }
  }
}

template <typename T, int NR, bool BLOCKED>
__global__ __launch_bounds__(256) void k_level(int n, int G, int blk, const int* __restrict__ ptr,
                                               const int* __restrict__ idx, const T* __restrict__ val,
                                               const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                               const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                               const int* __restrict__ skip, int nlog) {
  if (skip && *skip) return;
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  const int rpb = 256 / G;
  const int lane = threadIdx.x & (G - 1);
  const int row = lb * rpb + threadIdx.x / G;
  const bool active = row < n;
  T acc[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) acc[k] = 0;
  if (active) row_product<T, NR, BLOCKED>(row, lane, G, blk, ptr, idx, val, u, acc);
#pragma unroll
  for (int k = 0; k < NR; ++k) acc[k] = wave_sum(acc[k], G);
  if (!active) return;
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    if ((k & (G - 1)) != lane) continue;
    const int64_t i = (int64_t)row * NR + k;
    const T t = acc[k];
    if (flags & F_PLAIN) {
      rho[i] = t;
      continue;
    }
    const T r = ((flags & F_RHO_FROM_B) ? b[i] : rho[i]) - t;
    if (flags & F_RHO_STORE) rho[i] = r;
    const T ui = u[i];
    if (flags & F_X_ASSIGN)
      x[i] = ui;
    else if (flags & F_X_ADD)
      x[i] += ui;
    if (flags & F_D_OUT) dout[i] = c1 * ui + c2 * dinv[row] * r;
  }
}

template <typename T, int NR>
static void launch_level_nr(const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x, T* dout, double c1,
                            double c2, int flags, const int* skip, hipStream_t s) {
  const int G = op.lanes;
  const int rpb = 256 / G;
  const int nlog = (op.n + rpb - 1) / rpb;
  if (nlog == 0) return;
  if (op.blk == 1)
    hipLaunchKernelGGL((k_level<T, NR, false>), dim3(xcd_grid(nlog)), dim3(256), 0, s, op.n, G, 1, op.ptr, op.idx,
                       op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip, nlog);
  else
    hipLaunchKernelGGL((k_level<T, NR, true>), dim3(xcd_grid(nlog)), dim3(256), 0, s, op.n, G, op.blk, op.ptr,
                       op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip, nlog);
  check_launch("k_level");
}

template <typename T>
void launch_level(const LevelOp<T>& op, int nr, const T* u, const T* b, T* rho, T* x, T* dout, double c1,
                  double c2, int flags, const int* skip, hipStream_t s) {
  switch (nr) {
    case 1: launch_level_nr<T, 1>(op, u, b, rho, x, dout, c1, c2, flags, skip, s); break;
    case 2: launch_level_nr<T, 2>(op, u, b, rho, x, dout, c1, c2, flags, skip, s); break;
    case 4: launch_level_nr<T, 4>(op, u, b, rho, x, dout, c1, c2, flags, skip, s); break;
    case 8: launch_level_nr<T, 8>(op, u, b, rho, x, dout, c1, c2, flags, skip, s); break;
    case 16: launch_level_nr<T, 16>(op, u, b, rho, x, dout, c1, c2, flags, skip, s); break;
    default: throw std::runtime_error("unsupported nrhs block");
  }
}
template void launch_level<float>(const LevelOp<float>&, int, const float*, const float*, float*, float*, float*,
                                  double, double, int, const int*, hipStream_t);
template void launch_level<double>(const LevelOp<double>&, int, const double*, const double*, double*, double*,
                                   double*, double, double, int, const int*, hipStream_t);

// ==== fine-level row-block kernels ====

// Matrix load of the fused level kernels: ordinary with KEEP (the level's matrix fits the caches and is applied
// again right away), nontemporal otherwise.  A compile-time choice: a run-time select between the two would be
// folded into one ordinary load.
template <bool KEEP, typename P>
__device__ inline P ld_matrix(const P* ptr) {
  if constexpr (KEEP)
    return *ptr;
  else
    return __builtin_nontemporal_load(ptr);
}

// Row sums of the row-block kernels, in one canonical order that is the same for every shape.  A row's products are
// taken in chunks of four from its first entry: c_j = (p_4j + p_4j+2) + (p_4j+1 + p_4j+3), missing entries of the
// last chunk being +0; a_v = c_v + c_v+4 + ... (v = 0..3, in increasing position); row sum = (a_0 + a_2) + (a_1 + a_3).
// The products are rounded before they are added (no fused multiply-add), so that it does not matter whether a
// kernel adds them in registers or from LDS.

// the sum over a row's chunk sums cs(0..nc) by TPR consecutive lanes (4, 2 or 1); lane sub = 0 holds the result
template <typename T, int TPR, typename F>
__device__ inline T row_sum_chunks(int nc, int sub, F&& cs) {
  static_assert(TPR == 4 || TPR == 2 || TPR == 1, "lanes per row");
  if constexpr (TPR == 4) {
    T a = 0;
    for (int j = sub; j < nc; j += 4) a += cs(j);
    a += __shfl_xor(a, 2, 64);
    a += __shfl_xor(a, 1, 64);
    return a;
  } else if constexpr (TPR == 2) {
    T a = 0, c = 0;
    int j = sub;
    for (; j + 2 < nc; j += 4) {
      a += cs(j);
      c += cs(j + 2);
    }
    if (j < nc) a += cs(j);
    T t = a + c;
    t += __shfl_xor(t, 1, 64);
    return t;
  } else {
    T a[4] = {0, 0, 0, 0};
    int j = 0;
    for (; j + 3 < nc; j += 4) {
#pragma unroll
      for (int v = 0; v < 4; ++v) a[v] += cs(j + v);
    }
#pragma unroll
    for (int v = 0; v < 3; ++v)
      if (j + v < nc) a[v] += cs(j + v);
    return (a[0] + a[2]) + (a[1] + a[3]);
  }
}

// the same over the products prod[s..e) themselves, staged in LDS
template <typename T, int TPR>
__device__ inline T row_sum_canonical(const T* prod, int s, int e, int sub) {
  return row_sum_chunks<T, TPR>((e - s + 3) >> 2, sub, [&](int j) {
    const int k = s + 4 * j;
    const T p1 = k + 1 < e ? prod[k + 1] : (T)0, p2 = k + 2 < e ? prod[k + 2] : (T)0;
    const T p3 = k + 3 < e ? prod[k + 3] : (T)0;
    return (prod[k] + p2) + (p1 + p3);
  });
}

// Row-block ("stream") variant of the fused kernel for the CSR fine level, one right-hand side.  Each
// workgroup owns a host-computed block of <= RPB consecutive rows holding <= CAP - 3 nonzeros: phase 1 streams
// the block's values and column indices with fully coalesced loads (all issued before any gather) and stages
// val * u[col] in LDS, phase 2 sums each row with 256/RPB lanes and applies the same epilogue as k_level.  A row
// longer than CAP forms a block of its own and is summed by the whole workgroup.  With DOT the block also writes
// the partial sum of u_i (A u)_i (PCG's <p, A p>).  The (CAP, RPB) shape and the kernel form are chosen per
// matrix by timing.
template <typename T, bool DOT, int CAP, int RPB>
__global__ __launch_bounds__(256) void k_level_stream(int nrb, const int* __restrict__ rb, const int* __restrict__ ptr,
                                                      const int* __restrict__ idx, const T* __restrict__ val,
                                                      const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                                      const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                      const int* __restrict__ skip, double* partials) {
  constexpr int TPR = 256 / RPB;   // lanes per row in phase 2
  constexpr int EPT = CAP / 256;   // elements per thread in phase 1
  if (skip && *skip) return;
  const int lb = xcd_block(nrb);
  if (lb < 0) return;
  __shared__ T prod[CAP];
  __shared__ double sh[4];
  const int r0 = rb[lb], r1 = rb[lb + 1];
  const int e0 = ptr[r0], e1 = ptr[r1];
  const int nz = e1 - e0;
  // epilogue operands of the row this thread may finalise, fetched before the matrix stream
  const int prow = r0 + (threadIdx.x / TPR);
  const bool pre = (threadIdx.x % TPR) == 0 && prow < r1 && nz <= CAP && !(flags & F_PLAIN);
  T p_old = 0, p_x = 0, p_u = 0, p_di = 0;
  if (pre) {
    p_old = (flags & F_RHO_FROM_B) ? b[prow] : rho[prow];
    p_u = u[prow];
    if (flags & F_X_ADD) p_x = x[prow];
    if (flags & F_D_OUT) p_di = dinv[prow];
  }
  T t = 0;
  int row = -1;
  if (nz <= CAP) {
    // the matrix is streamed once per application: non-temporal loads keep u resident in the caches
    int ci[EPT];
    T vv[EPT];
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
      const int e = threadIdx.x + m * 256;
      if (e < nz) {
        ci[m] = __builtin_nontemporal_load(idx + e0 + e);
        vv[m] = __builtin_nontemporal_load(val + e0 + e);
      }
    }
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
      const int e = threadIdx.x + m * 256;
      if (e < nz) prod[e] = vv[m] * u[ci[m]];
    }
    __syncthreads();
    const int rl = threadIdx.x / TPR, sub = threadIdx.x % TPR;
    int s = 0, e = 0;
    if (r0 + rl < r1) {
      s = ptr[r0 + rl] - e0;
      e = ptr[r0 + rl + 1] - e0;
    }
    const T acc = row_sum_canonical<T, TPR>(prod, s, e, sub);
    if (sub == 0 && r0 + rl < r1) {
      row = r0 + rl;
      t = acc;
    }
  } else {  // one long row
    T acc = 0;
    for (int e = e0 + threadIdx.x; e < e1; e += 256) acc += val[e] * u[idx[e]];
    acc = wave_sum(acc, 64);
    __shared__ T shr[4];
    if ((threadIdx.x & 63) == 0) shr[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      row = r0;
      t = (shr[0] + shr[1]) + (shr[2] + shr[3]);
    }
  }
  double contrib = 0.0;
  if (row >= 0) {
    if (flags & F_PLAIN) {
      rho[row] = t;
      if (DOT) contrib = (double)t * (double)u[row];
    } else {
      if (!pre) {  // the long-row path did not prefetch
        p_old = (flags & F_RHO_FROM_B) ? b[row] : rho[row];
        p_u = u[row];
        if (flags & F_X_ADD) p_x = x[row];
        if (flags & F_D_OUT) p_di = dinv[row];
      }
      const T r = p_old - t;
      if (flags & F_RHO_STORE) rho[row] = r;
      if (flags & F_X_ASSIGN)
        x[row] = p_u;
      else if (flags & F_X_ADD)
        x[row] = p_x + p_u;
      if (flags & F_D_OUT) dout[row] = c1 * p_u + c2 * p_di * r;
    }
  }
  if (DOT) {
    const double s = block_sum256(contrib, sh);
    if (threadIdx.x == 0) partials[lb] = s;
  }
}

// Persistent, software-pipelined row-block kernel with 16-byte matrix loads.  Workgroup w owns the contiguous
// row blocks [w nrb / nwg, (w + 1) nrb / nwg) and, while it sums block i, has the matrix stream of block i + 1 in
// flight: per block the gathers of u and the per-row operands are issued before the next block's stream, so
// waiting for them (memory counters retire in order) never waits for the prefetch.  Products are staged in two
// alternating LDS buffers, so one barrier per block suffices.  (i) Each thread streams four consecutive entries per step, starting from the
// block's first entry rounded down to a multiple of four (entries outside the block are masked; the column and
// value arrays carry four padding entries at the end), and stages the four products with one aligned LDS write
// at their offset from that rounded start; (ii) each wave loads the row pointers of its rows once and spreads
// them with lane shuffles; (iii) the row sums go to LDS and the epilogue of a block runs one iteration later in
// wave 0, one row per lane with coalesced loads and stores (its operands are fetched before the next stream).
// Same summation order as the other row-block kernels.
template <typename T>
struct Vec4 {
  typedef T type __attribute__((ext_vector_type(4)));
};
typedef int i4v __attribute__((ext_vector_type(4)));

template <typename T, bool DOT, int CAP, int RPB>
__global__ __launch_bounds__(256) void k_level_stream_pv(int nrb, int nwg, const int* __restrict__ rb,
                                                         const int* __restrict__ ptr, const int* __restrict__ idx,
                                                         const T* __restrict__ val, const T* __restrict__ u,
                                                         const T* __restrict__ b, T* rho, T* x,
                                                         const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                         const int* __restrict__ skip, double* partials) {
  using V4 = typename Vec4<T>::type;
  constexpr int TPR = 256 / RPB;  // lanes per row
  constexpr int RPW = 64 / TPR;   // rows per wave
  constexpr int NCH = CAP / 1024; // four-entry chunks per thread
  constexpr int EPL = RPB / 64;   // epilogue rows per lane of wave 0
  static_assert(RPB % 64 == 0 && CAP % 1024 == 0, "row-block shape");
  if (skip && *skip) return;
  const int w = xcd_block(nwg);
  if (w < 0) return;
  const int lbA = (int)((int64_t)w * nrb / nwg), lbB = (int)((int64_t)(w + 1) * nrb / nwg);
  __shared__ __align__(32) T prod[2][CAP];
  __shared__ T rsum[2][RPB];
  __shared__ T shr[2][4];
  __shared__ double sh[4];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int rl = threadIdx.x / TPR, sub = threadIdx.x % TPR;
  double contrib = 0.0;
  int r0 = 0, r1 = 0, e0 = 0, e1 = 0;
  i4v ci[NCH];
  V4 vv[NCH];
  if (lbA < lbB) {
    r0 = rb[lbA];
    r1 = rb[lbA + 1];
    e0 = ptr[r0];
    e1 = ptr[r1];
    const int a0 = e0 & ~3;
    if (e1 - a0 <= CAP) {
#pragma unroll
      for (int m = 0; m < NCH; ++m) {
        const int e = a0 + 4 * (threadIdx.x + m * 256);
        if (e < e1) {
          ci[m] = __builtin_nontemporal_load(reinterpret_cast<const i4v*>(idx + e));
          vv[m] = __builtin_nontemporal_load(reinterpret_cast<const V4*>(val + e));
        }
      }
    }
  }
  int pr0 = 0, pr1 = 0;  // rows of the block whose epilogue is pending
  int it = 0;
  for (int lb = lbA; lb < lbB; ++lb, it ^= 1) {
    const int a0 = e0 & ~3;
    const bool staged = e1 - a0 <= CAP;
    // (a) everything this block and the pending epilogue still read
    V4 g[NCH];
    if (staged) {
#pragma unroll
      for (int m = 0; m < NCH; ++m) {
        const int e = a0 + 4 * (threadIdx.x + m * 256);
#pragma unroll
        for (int q = 0; q < 4; ++q) g[m][q] = (e + q >= e0 && e + q < e1) ? u[ci[m][q]] : (T)0;
      }
    }
    int rp = e1;
    if (lane <= RPW) {
      const int rr = r0 + wv * RPW + lane;
      rp = ptr[rr < r1 ? rr : r1];
    }
    T eo[EPL], eu[EPL], ex[EPL], ed[EPL];
#pragma unroll
    for (int q = 0; q < EPL; ++q) {
      eo[q] = eu[q] = ex[q] = ed[q] = 0;
      const int row = pr0 + lane + 64 * q;
      if (wv == 0 && row < pr1) {
        eu[q] = u[row];
        if (!(flags & F_PLAIN)) {
          eo[q] = (flags & F_RHO_FROM_B) ? b[row] : rho[row];
          if (flags & F_X_ADD) ex[q] = x[row];
          if (flags & F_D_OUT) ed[q] = dinv[row];
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // (b) the next block's matrix stream
    int nr0 = 0, nr1 = 0, ne0 = 0, ne1 = 0;
    i4v nci[NCH];
    V4 nvv[NCH];
    if (lb + 1 < lbB) {
      nr0 = r1;
      nr1 = rb[lb + 2];
      ne0 = e1;
      ne1 = ptr[nr1];
      const int na0 = ne0 & ~3;
      if (ne1 - na0 <= CAP) {
#pragma unroll
        for (int m = 0; m < NCH; ++m) {
          const int e = na0 + 4 * (threadIdx.x + m * 256);
          if (e < ne1) {
            nci[m] = __builtin_nontemporal_load(reinterpret_cast<const i4v*>(idx + e));
            nvv[m] = __builtin_nontemporal_load(reinterpret_cast<const V4*>(val + e));
          }
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    // (c) row sums of this block into rsum[it]
    if (staged) {
#pragma unroll
      for (int m = 0; m < NCH; ++m) {
        const int e = a0 + 4 * (threadIdx.x + m * 256);
        if (e < e1) *reinterpret_cast<V4*>(&prod[it][e - a0]) = vv[m] * g[m];
      }
      const int rs = __shfl(rp, lane / TPR, 64), re = __shfl(rp, lane / TPR + 1, 64);
      __syncthreads();
      const T acc = row_sum_canonical<T, TPR>(prod[it], rs - a0, re - a0, sub);
      if (sub == 0) rsum[it][rl] = acc;
    } else {  // one long row
      T acc = 0;
      for (int e = e0 + threadIdx.x; e < e1; e += 256) acc += val[e] * u[idx[e]];
      acc = wave_sum(acc, 64);
      if (lane == 0) shr[it][wv] = acc;
      __syncthreads();
      if (threadIdx.x == 0) rsum[it][0] = (shr[it][0] + shr[it][1]) + (shr[it][2] + shr[it][3]);
    }
    // (d) epilogue of the previous block (its row sums were published by the barrier above)
    if (wv == 0) {
#pragma unroll
      for (int q = 0; q < EPL; ++q) {
        const int row = pr0 + lane + 64 * q;
        if (row < pr1) {
          const T t = rsum[it ^ 1][lane + 64 * q];
          if (flags & F_PLAIN) {
            rho[row] = t;
            if (DOT) contrib += (double)t * (double)eu[q];
          } else {
            const T r = eo[q] - t;
            if (flags & F_RHO_STORE) rho[row] = r;
            if (flags & F_X_ASSIGN)
              x[row] = eu[q];
            else if (flags & F_X_ADD)
              x[row] = ex[q] + eu[q];
            if (flags & F_D_OUT) dout[row] = c1 * eu[q] + c2 * ed[q] * r;
          }
        }
      }
    }
    pr0 = r0;
    pr1 = r1;
    r0 = nr0;
    r1 = nr1;
    e0 = ne0;
    e1 = ne1;
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      ci[m] = nci[m];
      vv[m] = nvv[m];
    }
  }
  // epilogue of the last block
  __syncthreads();
  if (wv == 0) {
#pragma unroll
    for (int q = 0; q < EPL; ++q) {
      const int row = pr0 + lane + 64 * q;
      if (row < pr1) {
        const T t = rsum[it ^ 1][lane + 64 * q];
        const T uu = u[row];
        if (flags & F_PLAIN) {
          rho[row] = t;
          if (DOT) contrib += (double)t * (double)uu;
        } else {
          const T r = ((flags & F_RHO_FROM_B) ? b[row] : rho[row]) - t;
          if (flags & F_RHO_STORE) rho[row] = r;
          if (flags & F_X_ASSIGN)
            x[row] = uu;
          else if (flags & F_X_ADD)
            x[row] = x[row] + uu;
          if (flags & F_D_OUT) dout[row] = c1 * uu + c2 * dinv[row] * r;
        }
      }
    }
  }
  if (DOT) {
    const double s = block_sum256(contrib, sh);
    if (threadIdx.x == 0) partials[w] = s;
  }
}

// Local-column row-block kernel (one workgroup per block).  The block's distinct columns are gathered once into
// LDS (us); the matrix stream then carries the values and 1- or 2-byte positions into that list instead of 4-byte
// column indices, and each product reads its u entry from LDS.  Phase 2 and the epilogue are those of
// k_level_stream, with the same summation order.  A block with more than UCAP distinct columns is a single row,
// summed by the whole workgroup through the CSR columns.
template <typename T, typename IX, bool DOT, int CAP, int RPB, int UCAP>
__global__ __launch_bounds__(256) void k_level_local(int nrb, const int* __restrict__ rb, const int* __restrict__ ubp,
                                                     const int* __restrict__ ucol, const IX* __restrict__ lidx,
                                                     const int* __restrict__ ptr, const int* __restrict__ idx,
                                                     const T* __restrict__ val, const T* __restrict__ u,
                                                     const T* __restrict__ b, T* rho, T* x,
                                                     const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                     const int* __restrict__ skip, double* partials) {
  constexpr int TPR = 256 / RPB;
  constexpr int EPT = CAP / 256;
  constexpr int UPT = (UCAP + 255) / 256;
  if (skip && *skip) return;
  const int lb = xcd_block(nrb);
  if (lb < 0) return;
  __shared__ T us[UCAP];
  __shared__ T prod[CAP];
  __shared__ double sh[4];
  const int r0 = rb[lb], r1 = rb[lb + 1];
  const int e0 = ptr[r0], e1 = ptr[r1];
  const int nz = e1 - e0;
  const int u0 = ubp[lb], nu = ubp[lb + 1] - u0;
  const bool staged = nu <= UCAP;
  const int prow = r0 + (threadIdx.x / TPR);
  const bool pre = (threadIdx.x % TPR) == 0 && prow < r1 && staged && !(flags & F_PLAIN);
  T p_old = 0, p_x = 0, p_u = 0, p_di = 0;
  if (pre) {
    p_old = (flags & F_RHO_FROM_B) ? b[prow] : rho[prow];
    p_u = u[prow];
    if (flags & F_X_ADD) p_x = x[prow];
    if (flags & F_D_OUT) p_di = dinv[prow];
  }
  T t = 0;
  int row = -1;
  if (staged) {
    T ug[UPT];
#pragma unroll
    for (int m = 0; m < UPT; ++m) {
      const int c = threadIdx.x + m * 256;
      if (c < nu) ug[m] = u[ucol[u0 + c]];
    }
    IX li[EPT];
    T vv[EPT];
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
      const int e = threadIdx.x + m * 256;
      if (e < nz) {
        li[m] = __builtin_nontemporal_load(lidx + e0 + e);
        vv[m] = __builtin_nontemporal_load(val + e0 + e);
      }
    }
#pragma unroll
    for (int m = 0; m < UPT; ++m) {
      const int c = threadIdx.x + m * 256;
      if (c < nu) us[c] = ug[m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < EPT; ++m) {
      const int e = threadIdx.x + m * 256;
      if (e < nz) prod[e] = vv[m] * us[li[m]];
    }
    __syncthreads();
    const int rl = threadIdx.x / TPR, sub = threadIdx.x % TPR;
    int s = 0, e = 0;
    if (r0 + rl < r1) {
      s = ptr[r0 + rl] - e0;
      e = ptr[r0 + rl + 1] - e0;
    }
    const T acc = row_sum_canonical<T, TPR>(prod, s, e, sub);
    if (sub == 0 && r0 + rl < r1) {
      row = r0 + rl;
      t = acc;
    }
  } else {  // one long row
    T acc = 0;
    for (int e = e0 + threadIdx.x; e < e1; e += 256) acc += val[e] * u[idx[e]];
    acc = wave_sum(acc, 64);
    __shared__ T shr[4];
    if ((threadIdx.x & 63) == 0) shr[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
      row = r0;
      t = (shr[0] + shr[1]) + (shr[2] + shr[3]);
    }
  }
  double contrib = 0.0;
  if (row >= 0) {
    if (flags & F_PLAIN) {
      rho[row] = t;
      if (DOT) contrib = (double)t * (double)u[row];
    } else {
      if (!pre) {
        p_old = (flags & F_RHO_FROM_B) ? b[row] : rho[row];
        p_u = u[row];
        if (flags & F_X_ADD) p_x = x[row];
        if (flags & F_D_OUT) p_di = dinv[row];
      }
      const T r = p_old - t;
      if (flags & F_RHO_STORE) rho[row] = r;
      if (flags & F_X_ASSIGN)
        x[row] = p_u;
      else if (flags & F_X_ADD)
        x[row] = p_x + p_u;
      if (flags & F_D_OUT) dout[row] = c1 * p_u + c2 * p_di * r;
    }
  }
  if (DOT) {
    const double s = block_sum256(contrib, sh);
    if (threadIdx.x == 0) partials[lb] = s;
  }
}

// Local-column kernel with vector loads (1-byte column positions, one workgroup per block).  As k_level_local,
// but each thread streams four consecutive entries per step (16-byte value loads, 4-byte loads of four packed
// positions) from the block's first entry rounded down to a multiple of four (outside entries masked; values and
// positions carry kFinePad padding entries), stages the four products with one aligned LDS write, and each wave
// loads its rows' row pointers once and spreads them with lane shuffles.
template <typename T, int CAP, int RPB, int UCAP, bool KEEP>
__global__ __launch_bounds__(256) void k_level_local_vec(int nrb, const int4* __restrict__ meta,
                                                         const int* __restrict__ ucol,
                                                         const uint8_t* __restrict__ lidx, const int* __restrict__ ptr,
                                                         const int* __restrict__ idx, const T* __restrict__ val,
                                                         const T* __restrict__ u, const T* __restrict__ b, T* rho,
                                                         T* x, const T* __restrict__ dinv, T* dout, T c1, T c2,
                                                         int flags, const int* __restrict__ skip) {
  using V4 = typename Vec4<T>::type;
  constexpr int TPR = 256 / RPB;
  constexpr int RPW = 64 / TPR;
  constexpr int NCH = CAP / 1024;
  constexpr int UPT = UCAP / 256;
  static_assert(CAP % 1024 == 0 && UCAP % 256 == 0, "local block shape");
  if (skip && *skip) return;
  const int lb = xcd_block(nrb);
  if (lb < 0) return;
  __shared__ T us[UCAP];
  __shared__ __align__(32) T prod[CAP];
  __shared__ T shr[4];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // first row, first nonzero and first distinct column of this block and of the next (one round trip)
  const int4 m0 = meta[lb], m1 = meta[lb + 1];
  const int r0 = m0.x, r1 = m1.x;
  const int e0 = m0.y, e1 = m1.y;
  const int u0 = m0.z, nu = m1.z - u0;
  const bool staged = nu <= UCAP;
  const int rl = threadIdx.x / TPR, sub = threadIdx.x % TPR;
  const int prow = r0 + rl;
  // The loads below are unconditional per thread (clamped addresses; out-of-range values are never used): loads
  // under lane-dependent branches are waited for at the branch's end, which put the block's value stream behind
  // its column list.  Here the column list, values, positions and row pointers are in flight together, and only
  // the gather of u waits for the column list.
  const int prc = min(prow, r1 - 1);  // blocks hold at least one row
  T p_old = 0, p_x = 0, p_u = 0, p_di = 0;
  if (!(flags & F_PLAIN)) {
    p_old = (flags & F_RHO_FROM_B) ? b[prc] : rho[prc];
    p_u = u[prc];
    if (flags & F_X_ADD) p_x = x[prc];
    if (flags & F_D_OUT) p_di = dinv[prc];
  }
  T t = 0;
  if (staged) {
    int uc[UPT];
#pragma unroll
    for (int m = 0; m < UPT; ++m) uc[m] = ucol[u0 + min((int)threadIdx.x + m * 256, nu - 1)];  // nu >= 1
    const int a0 = e0 & ~3;
    uint32_t li[NCH];
    V4 vv[NCH];
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      const int e = a0 + 4 * (threadIdx.x + m * 256);
      const int ec = e < e1 ? e : a0;
      li[m] = ld_matrix<KEEP>(reinterpret_cast<const uint32_t*>(lidx + ec));
      vv[m] = ld_matrix<KEEP>(reinterpret_cast<const V4*>(val + ec));
    }
    const int rp = ptr[min(r0 + wv * RPW + min(lane, RPW), r1)];  // lanes 0..RPW: this wave's row pointers
    // slots nu .. UCAP-1 take copies and are never read (positions are below nu); no branch lets the gather sink
#pragma unroll
    for (int m = 0; m < UPT; ++m) us[threadIdx.x + m * 256] = u[uc[m]];
    // keep the streamed entries ahead of the barrier (the compiler would otherwise sink some loads past it)
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      asm volatile("" ::"v"(li[m]));
#pragma unroll
      for (int q = 0; q < 4; ++q) asm volatile("" ::"v"(vv[m][q]));
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      const int e = a0 + 4 * (threadIdx.x + m * 256);
      if (e < e1) {
        V4 g;
#pragma unroll
        for (int q = 0; q < 4; ++q) g[q] = (e + q >= e0 && e + q < e1) ? us[(li[m] >> (8 * q)) & 0xff] : (T)0;
        *reinterpret_cast<V4*>(&prod[e - a0]) = vv[m] * g;
      }
    }
    const int rs = __shfl(rp, lane / TPR, 64), re = __shfl(rp, lane / TPR + 1, 64);
    __syncthreads();
    t = row_sum_canonical<T, TPR>(prod, rs - a0, re - a0, sub);
  } else {  // one long row
    T acc = 0;
    for (int e = e0 + threadIdx.x; e < e1; e += 256) acc += val[e] * u[idx[e]];
    acc = wave_sum(acc, 64);
    if (lane == 0) shr[wv] = acc;
    __syncthreads();
    t = (shr[0] + shr[1]) + (shr[2] + shr[3]);
  }
  if (sub == 0 && prow < r1 && (staged || rl == 0)) {
    const int row = prow;
    if (flags & F_PLAIN) {
      rho[row] = t;
    } else {
      const T r = p_old - t;
      if (flags & F_RHO_STORE) rho[row] = r;
      if (flags & F_X_ASSIGN)
        x[row] = p_u;
      else if (flags & F_X_ADD)
        x[row] = p_x + p_u;
      if (flags & F_D_OUT) dout[row] = c1 * p_u + c2 * p_di * r;
    }
  }
}

// The same over pairs of blocks: a workgroup takes NB = 2 consecutive blocks and issues the loads of both before
// the first barrier, so that two blocks' streams are in flight per workgroup; each block is summed exactly as by
// k_level_local_vec.
template <typename T, int CAP, int RPB, int UCAP, bool KEEP, int NB>
__global__ __launch_bounds__(256) void k_level_local_vec_nb(int nrb, const int4* __restrict__ meta,
                                                         const int* __restrict__ ucol,
                                                         const uint8_t* __restrict__ lidx, const int* __restrict__ ptr,
                                                         const int* __restrict__ idx, const T* __restrict__ val,
                                                         const T* __restrict__ u, const T* __restrict__ b, T* rho,
                                                         T* x, const T* __restrict__ dinv, T* dout, T c1, T c2,
                                                         int flags, const int* __restrict__ skip) {
  using V4 = typename Vec4<T>::type;
  constexpr int TPR = 256 / RPB;
  constexpr int RPW = 64 / TPR;
  constexpr int NCH = CAP / 1024;
  constexpr int UPT = UCAP / 256;
  static_assert(CAP % 1024 == 0 && UCAP % 256 == 0 && (NB == 1 || NB == 2), "local block shape");
  if (skip && *skip) return;
  const int lg = xcd_block((nrb + NB - 1) / NB);
  if (lg < 0) return;
  __shared__ T us[NB][UCAP];
  __shared__ __align__(32) T prod[NB][CAP];
  __shared__ T shr[NB][4];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int rl = threadIdx.x / TPR, sub = threadIdx.x % TPR;
  // per block: first row, first nonzero and first distinct column of it and of the next (one round trip); a
  // missing second block (odd nrb) repeats the last one and stores nothing
  int r0[NB], r1[NB], e0[NB], e1[NB], u0[NB], nu[NB];
  bool live[NB];
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    live[h] = lg * NB + h < nrb;
    const int lb = min(lg * NB + h, nrb - 1);
    const int4 m0 = meta[lb], m1 = meta[lb + 1];
    r0[h] = m0.x;
    r1[h] = m1.x;
    e0[h] = m0.y;
    e1[h] = m1.y;
    u0[h] = m0.z;
    nu[h] = m1.z - m0.z;
  }
  // The loads below are unconditional per thread (clamped addresses; out-of-range values are never used): loads
  // under lane-dependent branches are waited for at the branch's end, which put the block's value stream behind
  // its column list.  Here the column list, values, positions and row pointers are in flight together, and only
  // the gather of u waits for the column list.
  T p_old[NB], p_x[NB], p_u[NB], p_di[NB];
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    const int prc = min(r0[h] + rl, r1[h] - 1);  // blocks hold at least one row
    p_old[h] = p_x[h] = p_u[h] = p_di[h] = 0;
    if (!(flags & F_PLAIN)) {
      p_old[h] = (flags & F_RHO_FROM_B) ? b[prc] : rho[prc];
      p_u[h] = u[prc];
      if (flags & F_X_ADD) p_x[h] = x[prc];
      if (flags & F_D_OUT) p_di[h] = dinv[prc];
    }
  }
  int uc[NB][UPT];
  uint32_t li[NB][NCH];
  V4 vv[NB][NCH];
  int rp[NB];
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    if (nu[h] > UCAP) continue;  // one long row, summed below (uniform over the workgroup)
#pragma unroll
    for (int m = 0; m < UPT; ++m) uc[h][m] = ucol[u0[h] + min((int)threadIdx.x + m * 256, nu[h] - 1)];  // nu >= 1
    const int a0 = e0[h] & ~3;
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      const int e = a0 + 4 * (threadIdx.x + m * 256);
      const int ec = e < e1[h] ? e : a0;
      li[h][m] = ld_matrix<KEEP>(reinterpret_cast<const uint32_t*>(lidx + ec));
      vv[h][m] = ld_matrix<KEEP>(reinterpret_cast<const V4*>(val + ec));
    }
    rp[h] = ptr[min(r0[h] + wv * RPW + min(lane, RPW), r1[h])];  // lanes 0..RPW: this wave's row pointers
  }
  // slots nu .. UCAP-1 take copies and are never read (positions are below nu); no branch lets the gather sink
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    if (nu[h] > UCAP) continue;
#pragma unroll
    for (int m = 0; m < UPT; ++m) us[h][threadIdx.x + m * 256] = u[uc[h][m]];
  }
  // keep the streamed entries ahead of the barrier (the compiler would otherwise sink some loads past it)
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    if (nu[h] > UCAP) continue;
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      asm volatile("" ::"v"(li[h][m]));
#pragma unroll
      for (int q = 0; q < 4; ++q) asm volatile("" ::"v"(vv[h][m][q]));
    }
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    if (nu[h] > UCAP) continue;
    const int a0 = e0[h] & ~3;
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      const int e = a0 + 4 * (threadIdx.x + m * 256);
      if (e < e1[h]) {
        V4 g;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          g[q] = (e + q >= e0[h] && e + q < e1[h]) ? us[h][(li[h][m] >> (8 * q)) & 0xff] : (T)0;
        *reinterpret_cast<V4*>(&prod[h][e - a0]) = vv[h][m] * g;
      }
    }
  }
  __syncthreads();
  T t[NB];
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    if (nu[h] <= UCAP) {
      const int a0 = e0[h] & ~3;
      const int rs = __shfl(rp[h], lane / TPR, 64), re = __shfl(rp[h], lane / TPR + 1, 64);
      t[h] = row_sum_canonical<T, TPR>(prod[h], rs - a0, re - a0, sub);
    } else {  // one long row
      T acc = 0;
      for (int e = e0[h] + threadIdx.x; e < e1[h]; e += 256) acc += val[e] * u[idx[e]];
      acc = wave_sum(acc, 64);
      if (lane == 0) shr[h][wv] = acc;
      __syncthreads();
      t[h] = (shr[h][0] + shr[h][1]) + (shr[h][2] + shr[h][3]);
    }
  }
#pragma unroll
  for (int h = 0; h < NB; ++h) {
    const bool staged = nu[h] <= UCAP;
    const int row = r0[h] + rl;
    if (!live[h] || sub != 0 || row >= r1[h] || !(staged || rl == 0)) continue;
    if (flags & F_PLAIN) {
      rho[row] = t[h];
    } else {
      const T r = p_old[h] - t[h];
      if (flags & F_RHO_STORE) rho[row] = r;
      if (flags & F_X_ASSIGN)
        x[row] = p_u[h];
      else if (flags & F_X_ADD)
        x[row] = p_x[h] + p_u[h];
      if (flags & F_D_OUT) dout[row] = c1 * p_u[h] + c2 * p_di[h] * r;
    }
  }
}

// Chunk kernel of the fine level (shape kChunkShape).  The matrix is held in chunks of four consecutive entries of one
// row (rows padded with zero values to whole chunks), so a thread adds the four products of a 16- or 32-byte value
// load in registers and stages one sum per chunk in LDS.  The kernels above stage every product: four times the LDS
// traffic, and in 3D half their slots stay empty, because 256 columns (1-byte positions) are reached after about
// 1,000 of 2,048 entries.  Here the positions have 9 bits (8 in a 4-byte word per chunk, the bits above in a byte per
// chunk), the blocks are full, and a block of 3,072 entries needs half as many distinct columns per entry.  Padding
// entries have the position nu, whose slot holds zero, so that they add +0 whatever u holds.
// Bound by memory: the matrix at 5.25 bytes (float32) per entry, the distinct columns and 7 vector streams.  One
// application back to back, best of the kernels above -> this one: 3D Q2 48^3 (912,673 rows) float32 81.1 -> 61.1 us
// (340 MB: 5.6 TB/s, a copy of that size runs at 5.4), float64 y = A p 121.7 -> 109.3; 3D Q2 29^3 float64 27.8 -> 19.3;
// 3D Q2 24^3 float32 12.0 -> 8.2; 3D Q3 16^3 float32 26.8 -> 13.4; 2D Q3 256^2 float32 17.8 -> 16.4 (6.3 TB/s from the
// caches), float64 y = A p 22.8 -> 22.4; 2D Q3 101^2 float64 6.4 -> 4.9; 2D Q2 16^2 (1,089 rows) 3.6 -> 3.4.
template <typename T, int CAPC, int RPB, int UCAP, bool KEEP>
__global__ __launch_bounds__(256) void k_level_chunk(int nrb, const int4* __restrict__ meta,
                                                     const int* __restrict__ ucol, const uint32_t* __restrict__ clo,
                                                     const uint8_t* __restrict__ chi, const int* __restrict__ cptr,
                                                     const T* __restrict__ cval, const int* __restrict__ ptr,
                                                     const int* __restrict__ idx, const T* __restrict__ val,
                                                     const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                                     const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                     const int* __restrict__ skip) {
  using V4 = typename Vec4<T>::type;
  constexpr int TPR = 256 / RPB;
  constexpr int NCH = CAPC / 256;
  constexpr int UPT = UCAP / 256;
  static_assert(CAPC % 256 == 0 && UCAP % 256 == 0 && UCAP <= 1024, "chunk block shape");
  if (skip && *skip) return;
  const int lb = xcd_block(nrb);
  if (lb < 0) return;
  __shared__ T us[UCAP];
  __shared__ T cs[CAPC];
  __shared__ T shr[4];
  const int4 m0 = meta[lb], m1 = meta[lb + 1];
  const int r0 = m0.x, r1 = m1.x;
  const int k0 = m0.y, k1 = m1.y;
  const int u0 = m0.z, nu = m1.z - u0;
  const bool staged = nu < UCAP && k1 - k0 <= CAPC;
  const int rl = threadIdx.x / TPR, sub = threadIdx.x % TPR;
  const int prow = r0 + rl;
  // unconditional loads from clamped addresses, as in k_level_local_vec
  const int prc = min(prow, r1 - 1);  // blocks hold at least one row
  T p_old = 0, p_x = 0, p_u = 0, p_di = 0;
  T t = 0;
  if (staged) {
    int uc[UPT];
#pragma unroll
    for (int m = 0; m < UPT; ++m) uc[m] = ucol[u0 + min((int)threadIdx.x + m * 256, nu - 1)];  // nu >= 1
    uint32_t lo[NCH], hi[NCH];
    V4 vv[NCH];
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      const int k = min(k0 + (int)threadIdx.x + m * 256, k1 - 1);
      lo[m] = ld_matrix<KEEP>(clo + k);
      hi[m] = ld_matrix<KEEP>(chi + k);
      vv[m] = ld_matrix<KEEP>(reinterpret_cast<const V4*>(cval) + k);
    }
    const int rs = cptr[min(prow, r1)] - k0, re = cptr[min(prow + 1, r1)] - k0;
    if (!(flags & F_PLAIN)) {
      p_old = (flags & F_RHO_FROM_B) ? b[prc] : rho[prc];
      p_u = u[prc];
      if (flags & F_X_ADD) p_x = x[prc];
      if (flags & F_D_OUT) p_di = dinv[prc];
    }
#pragma unroll
    for (int m = 0; m < UPT; ++m) {
      const T g = u[uc[m]];
      us[threadIdx.x + m * 256] = (int)threadIdx.x + m * 256 < nu ? g : (T)0;
    }
    // keep the streamed entries ahead of the barrier (the compiler would otherwise sink some loads past it)
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      asm volatile("" ::"v"(lo[m]), "v"(hi[m]));
#pragma unroll
      for (int q = 0; q < 4; ++q) asm volatile("" ::"v"(vv[m][q]));
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
#pragma clang fp contract(off)
      V4 p;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        p[q] = vv[m][q] * us[((lo[m] >> (8 * q)) & 0xff) | (((hi[m] >> (2 * q)) & 3) << 8)];
      cs[threadIdx.x + m * 256] = (p[0] + p[2]) + (p[1] + p[3]);  // past the block: never read
    }
    __syncthreads();
    t = row_sum_chunks<T, TPR>(re - rs, sub, [&](int j) { return cs[rs + j]; });
  } else {  // one long row
    if (!(flags & F_PLAIN)) {
      p_old = (flags & F_RHO_FROM_B) ? b[prc] : rho[prc];
      p_u = u[prc];
      if (flags & F_X_ADD) p_x = x[prc];
      if (flags & F_D_OUT) p_di = dinv[prc];
    }
    const int lane = threadIdx.x & 63;
    T acc = 0;
    for (int e = ptr[r0] + threadIdx.x; e < ptr[r0 + 1]; e += 256) acc += val[e] * u[idx[e]];
    acc = wave_sum(acc, 64);
    if (lane == 0) shr[threadIdx.x >> 6] = acc;
    __syncthreads();
    t = (shr[0] + shr[1]) + (shr[2] + shr[3]);
  }
  if (sub == 0 && prow < r1 && (staged || rl == 0)) {
    const int row = prow;
    if (flags & F_PLAIN) {
      rho[row] = t;
    } else {
      const T r = p_old - t;
      if (flags & F_RHO_STORE) rho[row] = r;
      if (flags & F_X_ASSIGN)
        x[row] = p_u;
      else if (flags & F_X_ADD)
        x[row] = p_x + p_u;
      if (flags & F_D_OUT) dout[row] = c1 * p_u + c2 * p_di * r;
    }
  }
}

template <typename T>
__global__ __launch_bounds__(256) void k_chunk_values(int n, const int* __restrict__ ptr, const int* __restrict__ cptr,
                                                      const T* __restrict__ val, T* cval) {
  const int row = blockIdx.x * 16 + (threadIdx.x >> 4), lane = threadIdx.x & 15;
  if (row >= n) return;
  const int s = ptr[row], len = ptr[row + 1] - s;
  const int k = cptr[row], w = 4 * (cptr[row + 1] - k);
  for (int j = lane; j < w; j += 16) cval[4 * (int64_t)k + j] = j < len ? val[s + j] : (T)0;
}

template <typename T>
void launch_chunk_values(int n, const int* ptr, const int* cptr, const T* val, T* cval, hipStream_t s) {
  hipLaunchKernelGGL((k_chunk_values<T>), dim3((n + 15) / 16), dim3(256), 0, s, n, ptr, cptr, val, cval);
  check_launch("k_chunk_values");
}
template void launch_chunk_values<float>(int, const int*, const int*, const float*, float*, hipStream_t);
template void launch_chunk_values<double>(int, const int*, const int*, const double*, double*, hipStream_t);

template <typename T, int CAP, int RPB>
static int launch_stream_block(const FineBlocks& fb, const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x,
                               T* dout, double c1, double c2, int flags, const int* skip, double* partials,
                               hipStream_t s) {
  const int nrb = fb.nrb;
  if (partials)
    hipLaunchKernelGGL((k_level_stream<T, true, CAP, RPB>), dim3(xcd_grid(nrb)), dim3(256), 0, s, nrb, fb.rb, op.ptr,
                       op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip, partials);
  else
    hipLaunchKernelGGL((k_level_stream<T, false, CAP, RPB>), dim3(xcd_grid(nrb)), dim3(256), 0, s, nrb, fb.rb, op.ptr,
                       op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip, partials);
  return nrb;
}

// workgroups of a persistent kernel: as many as are resident at once on the device (capped by the work)
template <typename K>
static int resident_groups(K kernel) {
  int per_cu = 0, dev = 0, cus = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0) != hipSuccess ||
      hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
    throw std::runtime_error("occupancy query of the pipelined row-block kernel failed");
  return std::max(1, per_cu) * std::max(1, cus);
}

template <typename T, bool DOT, int CAP, int RPB>
static int pipe_groups(int nrb) {
  static const int g = resident_groups(k_level_stream_pv<T, DOT, CAP, RPB>);
  return std::min(nrb, g);
}

template <typename T, int CAP, int RPB>
static int launch_stream_pipe(const FineBlocks& fb, const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x,
                              T* dout, double c1, double c2, int flags, const int* skip, double* partials,
                              hipStream_t s) {
  const int nrb = fb.nrb;
  const int nwg = partials ? pipe_groups<T, true, CAP, RPB>(nrb) : pipe_groups<T, false, CAP, RPB>(nrb);
  const dim3 grid(xcd_grid(nwg));
  if (partials)
    hipLaunchKernelGGL((k_level_stream_pv<T, true, CAP, RPB>), grid, dim3(256), 0, s, nrb, nwg, fb.rb, op.ptr, op.idx,
                       op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip, partials);
  else
    hipLaunchKernelGGL((k_level_stream_pv<T, false, CAP, RPB>), grid, dim3(256), 0, s, nrb, nwg, fb.rb, op.ptr,
                       op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip, partials);
  return nwg;
}

template <typename T, typename IX, int CAP, int RPB, int UCAP>
static int launch_stream_local(const FineBlocks& fb, const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x,
                               T* dout, double c1, double c2, int flags, const int* skip, double* partials,
                               hipStream_t s) {
  const int nrb = fb.nrb;
  const IX* li = static_cast<const IX*>(fb.lidx);
  if (partials)
    hipLaunchKernelGGL((k_level_local<T, IX, true, CAP, RPB, UCAP>), dim3(xcd_grid(nrb)), dim3(256), 0, s, nrb, fb.rb,
                       fb.ubp, fb.ucol, li, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags,
                       skip, partials);
  else
    hipLaunchKernelGGL((k_level_local<T, IX, false, CAP, RPB, UCAP>), dim3(xcd_grid(nrb)), dim3(256), 0, s, nrb,
                       fb.rb, fb.ubp, fb.ucol, li, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2,
                       flags, skip, partials);
  return nrb;
}

template <typename T, int CAP, int RPB, int UCAP, int NB>
static int launch_stream_local_vec(const FineBlocks& fb, const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x,
                                   T* dout, double c1, double c2, int flags, const int* skip, double* partials,
                                   hipStream_t s) {
  if (partials) throw std::runtime_error("local-column vector kernel: no partial sums");
  const int nrb = fb.nrb;
  if (!fb.meta) throw std::runtime_error("local-column vector kernel: block records missing");
  const int4* meta = reinterpret_cast<const int4*>(fb.meta);
  const uint8_t* lidx = static_cast<const uint8_t*>(fb.lidx);
  if constexpr (NB == 1) {
    if (flags & F_KEEP)
      hipLaunchKernelGGL((k_level_local_vec<T, CAP, RPB, UCAP, true>), dim3(xcd_grid(nrb)), dim3(256), 0, s, nrb, meta,
                         fb.ucol, lidx, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip);
    else
      hipLaunchKernelGGL((k_level_local_vec<T, CAP, RPB, UCAP, false>), dim3(xcd_grid(nrb)), dim3(256), 0, s, nrb,
                         meta, fb.ucol, lidx, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags,
                         skip);
  } else {
    const dim3 grid(xcd_grid((nrb + NB - 1) / NB));
    if (flags & F_KEEP)
      hipLaunchKernelGGL((k_level_local_vec_nb<T, CAP, RPB, UCAP, true, NB>), grid, dim3(256), 0, s, nrb, meta, fb.ucol,
                         lidx, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip);
    else
      hipLaunchKernelGGL((k_level_local_vec_nb<T, CAP, RPB, UCAP, false, NB>), grid, dim3(256), 0, s, nrb, meta,
                         fb.ucol, lidx, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip);
  }
  return nrb;
}

template <typename T>
static int launch_chunk(const FineBlocks& fb, const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x, T* dout,
                        double c1, double c2, int flags, const int* skip, double* partials, hipStream_t s) {
  if (partials) throw std::runtime_error("chunk kernel: no partial sums");
  if (!fb.meta || !fb.cptr || !op.cval) throw std::runtime_error("chunk kernel: chunked matrix missing");
  const int4* meta = reinterpret_cast<const int4*>(fb.meta);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(xcd_grid(fb.nrb)), dim3(256), 0, s, fb.nrb, meta, fb.ucol, fb.clo, fb.chi, fb.cptr,
                       op.cval, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip);
  };
  if (flags & F_KEEP)
    go(k_level_chunk<T, kChunkCap, kChunkRows, kChunkUcap, true>);
  else
    go(k_level_chunk<T, kChunkCap, kChunkRows, kChunkUcap, false>);
  return fb.nrb;
}

template <typename T>
int launch_level_stream(int shape, const FineBlocks& fb, const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x,
                        T* dout, double c1, double c2, int flags, const int* skip, double* partials, hipStream_t s) {
  if (fb.nrb == 0) return 0;
  int np = 0;
#define R3MG_ARGS fb, op, u, b, rho, x, dout, c1, c2, flags, skip, partials, s
  switch (shape) {
    case 0: np = launch_stream_block<T, 2048, 64>(R3MG_ARGS); break;
    case 1: np = launch_stream_block<T, 4096, 128>(R3MG_ARGS); break;
    case 2: np = launch_stream_block<T, 4096, 64>(R3MG_ARGS); break;
    case 3: np = launch_stream_pipe<T, 2048, 64>(R3MG_ARGS); break;
    case 4: np = launch_stream_pipe<T, 4096, 128>(R3MG_ARGS); break;
    case 5: np = launch_stream_pipe<T, 4096, 64>(R3MG_ARGS); break;
    case 6: np = launch_stream_local<T, uint8_t, 2048, 64, 256>(R3MG_ARGS); break;
    case 7: np = launch_stream_local<T, uint16_t, 4096, 64, 1024>(R3MG_ARGS); break;
    case 8: np = launch_stream_local<T, uint16_t, 4096, 128, 1024>(R3MG_ARGS); break;
    case 9: np = launch_stream_local_vec<T, 2048, 64, 256, 1>(R3MG_ARGS); break;
    case 10: np = launch_stream_local_vec<T, 3072, 128, 256, 1>(R3MG_ARGS); break;
    case 11: np = launch_stream_local_vec<T, 2048, 64, 256, 2>(R3MG_ARGS); break;
    case 12: np = launch_stream_local_vec<T, 3072, 128, 256, 2>(R3MG_ARGS); break;
    case 13: np = launch_stream_local_vec<T, 3072, 64, 256, 1>(R3MG_ARGS); break;
    case kChunkShape: np = launch_chunk<T>(R3MG_ARGS); break;
    default: throw std::runtime_error("unknown row-block shape");
  }
#undef R3MG_ARGS
  check_launch("k_level_stream");
  return np;
}
template int launch_level_stream<float>(int, const FineBlocks&, const LevelOp<float>&, const float*, const float*,
                                        float*, float*, float*, double, double, int, const int*, double*, hipStream_t);
template int launch_level_stream<double>(int, const FineBlocks&, const LevelOp<double>&, const double*,
                                         const double*, double*, double*, double*, double, double, int, const int*,
                                         double*, hipStream_t);
// ==== end of fine-level row-block kernels ====

// Multi-right-hand-side CSR kernel with the columns split over lanes (NR columns, interleaved n x NR vectors).
// G lanes per row (G a power of two, NG <= G <= 64, NG = NR / GW, GW = 16 / sizeof(T)): lane (j, s) owns the
// column group j (GW consecutive columns, one 16-byte load per nonzero) and the row's entries s, s + G/NG, ...;
// so the NG lanes of one nonzero read its u row as consecutive 16-byte pieces.  The G/NG entry lanes of a group
// are combined by a butterfly and lane s = 0 applies the epilogue of k_level to its GW columns.
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_level_split(int n, int G, const int* __restrict__ ptr,
                                                     const int* __restrict__ idx, const T* __restrict__ val,
                                                     const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                                     const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                     const int* __restrict__ skip, int nlog) {
  constexpr int GW = 16 / (int)sizeof(T);
  constexpr int NG = NR / GW;
  constexpr int UNR = 4;
  static_assert(NR % GW == 0, "column groups");
  typedef T VG __attribute__((ext_vector_type(GW)));
  if (skip && *skip) return;
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  const int rpb = 256 / G;
  const int li = threadIdx.x % G;
  const int j = li % NG, sv = li / NG, S = G / NG;
  const int row = lb * rpb + threadIdx.x / G;
  VG acc = (VG)0;
  if (row < n) {
    const int s = ptr[row], e = ptr[row + 1];
    for (int p0 = s + sv; p0 < e; p0 += UNR * S) {
      T a[UNR];
      int64_t c[UNR];
#pragma unroll
      for (int m = 0; m < UNR; ++m) {
        const int p = p0 + m * S;
        a[m] = p < e ? val[p] : (T)0;
        c[m] = p < e ? (int64_t)idx[p] * NR + j * GW : j * GW;
      }
      VG uv[UNR];
#pragma unroll
      for (int m = 0; m < UNR; ++m) uv[m] = *reinterpret_cast<const VG*>(u + c[m]);
#pragma unroll
      for (int m = 0; m < UNR; ++m) acc += a[m] * uv[m];
    }
  }
  for (int off = NG; off < G; off <<= 1)
#pragma unroll
    for (int w = 0; w < GW; ++w) acc[w] += __shfl_xor(acc[w], off, 64);
  if (sv == 0 && row < n) {
    const int64_t o = (int64_t)row * NR + j * GW;
    if (flags & F_PLAIN) {
      *reinterpret_cast<VG*>(rho + o) = acc;
    } else {
      const VG old = (flags & F_RHO_FROM_B) ? *reinterpret_cast<const VG*>(b + o) : *reinterpret_cast<VG*>(rho + o);
      const VG r = old - acc;
      if (flags & F_RHO_STORE) *reinterpret_cast<VG*>(rho + o) = r;
      const VG ui = *reinterpret_cast<const VG*>(u + o);
      if (flags & F_X_ASSIGN)
        *reinterpret_cast<VG*>(x + o) = ui;
      else if (flags & F_X_ADD)
        *reinterpret_cast<VG*>(x + o) = *reinterpret_cast<VG*>(x + o) + ui;
      if (flags & F_D_OUT) *reinterpret_cast<VG*>(dout + o) = c1 * ui + (c2 * dinv[row]) * r;
    }
  }
}

// The same product with each nonzero's value and column read once: the G lanes of a row load G consecutive
// entries of the row at a time (one value and one column each, coalesced), then NG steps follow in which lane
// (s, j) takes entry t S + s of that chunk from its owner lane by a shuffle and reads column group j of the
// entry's u row (16 bytes).  Per G entries a lane issues 2 + NG loads instead of 3 per entry it owns, which
// halves the address work of the gathers' texture-address unit.  Same epilogue as k_level_split.
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_level_split2(int n, int G, const int* __restrict__ ptr,
                                                      const int* __restrict__ idx, const T* __restrict__ val,
                                                      const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                                      const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                      const int* __restrict__ skip, int nlog) {
  constexpr int GW = 16 / (int)sizeof(T);
  constexpr int NG = NR / GW;
  static_assert(NR % GW == 0, "column groups");
  typedef T VG __attribute__((ext_vector_type(GW)));
  if (skip && *skip) return;
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  const int rpb = 256 / G;
  const int li = threadIdx.x % G;
  const int gbase = (int)(threadIdx.x & 63) - li;  // the row group's first lane in the wave
  const int j = li % NG, sv = li / NG, S = G / NG;
  const int row = lb * rpb + threadIdx.x / G;
  VG acc = (VG)0;
  int s = 0, e = 0;
  if (row < n) {
    s = ptr[row];
    e = ptr[row + 1];
  }
  // every lane of a row group runs the same chunks, so a shuffle only ever reads an active lane of its group
  for (int c0 = s; c0 < e; c0 += G) {
    const int p = c0 + li;
    const T a_l = p < e ? val[p] : (T)0;
    const int i_l = p < e ? idx[p] : 0;
#pragma unroll
    for (int t = 0; t < NG; ++t) {
      const int src = gbase + t * S + sv;
      const T a = __shfl(a_l, src, 64);
      const int64_t ci = (int64_t)__shfl(i_l, src, 64);
      const VG uv = *reinterpret_cast<const VG*>(u + ci * NR + j * GW);
      acc += a * uv;
    }
  }
  for (int off = NG; off < G; off <<= 1)
#pragma unroll
    for (int w = 0; w < GW; ++w) acc[w] += __shfl_xor(acc[w], off, 64);
  if (sv == 0 && row < n) {
    const int64_t o = (int64_t)row * NR + j * GW;
    if (flags & F_PLAIN) {
      *reinterpret_cast<VG*>(rho + o) = acc;
    } else {
      const VG old = (flags & F_RHO_FROM_B) ? *reinterpret_cast<const VG*>(b + o) : *reinterpret_cast<VG*>(rho + o);
      const VG r = old - acc;
      if (flags & F_RHO_STORE) *reinterpret_cast<VG*>(rho + o) = r;
      const VG ui = *reinterpret_cast<const VG*>(u + o);
      if (flags & F_X_ASSIGN)
        *reinterpret_cast<VG*>(x + o) = ui;
      else if (flags & F_X_ADD)
        *reinterpret_cast<VG*>(x + o) = *reinterpret_cast<VG*>(x + o) + ui;
      if (flags & F_D_OUT) *reinterpret_cast<VG*>(dout + o) = c1 * ui + (c2 * dinv[row]) * r;
    }
  }
}

template <typename T>
bool launch_level_split2(const LevelOp<T>& op, int nr, int G, const T* u, const T* b, T* rho, T* x, T* dout,
                         double c1, double c2, int flags, const int* skip, hipStream_t s) {
  constexpr int GW = 16 / (int)sizeof(T);
  if (nr % GW != 0 || G < nr / GW || G > 64 || (G & (G - 1)) != 0 || op.blk != 1) return false;
  const int rpb = 256 / G;
  const int nlog = (op.n + rpb - 1) / rpb;
  if (nlog == 0) return true;
#define R3MG_SPLIT2(NRV)                                                                                          \
  hipLaunchKernelGGL((k_level_split2<T, NRV>), dim3(xcd_grid(nlog)), dim3(256), 0, s, op.n, G, op.ptr, op.idx,   \
                     op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip, nlog)
  switch (nr) {
    case 4: R3MG_SPLIT2(4); break;
    case 8: R3MG_SPLIT2(8); break;
    case 16: R3MG_SPLIT2(16); break;
    default: return false;
  }
#undef R3MG_SPLIT2
  check_launch("k_level_split2");
  return true;
}
template bool launch_level_split2<float>(const LevelOp<float>&, int, int, const float*, const float*, float*, float*,
                                         float*, double, double, int, const int*, hipStream_t);
template bool launch_level_split2<double>(const LevelOp<double>&, int, int, const double*, const double*, double*,
                                          double*, double*, double, double, int, const int*, hipStream_t);

template <typename T>
bool launch_level_split(const LevelOp<T>& op, int nr, int G, const T* u, const T* b, T* rho, T* x, T* dout, double c1,
                        double c2, int flags, const int* skip, hipStream_t s) {
  constexpr int GW = 16 / (int)sizeof(T);
  if (nr % GW != 0 || G < nr / GW || G > 64 || (G & (G - 1)) != 0 || op.blk != 1) return false;
  const int rpb = 256 / G;
  const int nlog = (op.n + rpb - 1) / rpb;
  if (nlog == 0) return true;
#define R3MG_SPLIT(NRV)                                                                                             \
  hipLaunchKernelGGL((k_level_split<T, (NRV < GW ? GW : NRV)>), dim3(xcd_grid(nlog)), dim3(256), 0, s, op.n, G, op.ptr, \
                     op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip, nlog)
  switch (nr) {
    case 2: R3MG_SPLIT(2); break;
    case 4: R3MG_SPLIT(4); break;
    case 8: R3MG_SPLIT(8); break;
    case 16: R3MG_SPLIT(16); break;
    default: return false;
  }
#undef R3MG_SPLIT
  check_launch("k_level_split");
  return true;
}
template bool launch_level_split<float>(const LevelOp<float>&, int, int, const float*, const float*, float*, float*,
                                        float*, double, double, int, const int*, hipStream_t);
template bool launch_level_split<double>(const LevelOp<double>&, int, int, const double*, const double*, double*,
                                         double*, double*, double, double, int, const int*, hipStream_t);

// Sum over the entries [k, z) of one row from LDS: values svs[k], column positions sps[k] into the staged u rows
// usq[p * CH] (16-byte chunks).  Single entries up to a multiple of 4 from vb (the block's aligned start); then
// groups of 8 (two aligned LDS words of 4 values and of 4 positions each), the next group's values and positions
// read together with the current group's u rows, so that one LDS round trip serves 8 entries; then 4-entry groups
// and single entries.  The entries are added in ascending order.
template <typename T, typename VT, int CH>
__device__ __forceinline__ VT lmr_row_sum(const T* svs, const uint16_t* sps, const VT* usq, int vb, int k, int z) {
  typedef T T4 __attribute__((ext_vector_type(4)));
  typedef unsigned short S4 __attribute__((ext_vector_type(4)));
  VT t = (VT)0;
  for (; k < z && ((k - vb) & 3); ++k) t += svs[k] * usq[sps[k] * CH];
  if (k + 8 <= z) {
    T4 a0 = *reinterpret_cast<const T4*>(svs + k), a1 = *reinterpret_cast<const T4*>(svs + k + 4);
    S4 p0 = *reinterpret_cast<const S4*>(sps + k), p1 = *reinterpret_cast<const S4*>(sps + k + 4);
    for (;;) {
      const VT w0 = usq[p0.x * CH], w1 = usq[p0.y * CH], w2 = usq[p0.z * CH], w3 = usq[p0.w * CH];
      const VT w4 = usq[p1.x * CH], w5 = usq[p1.y * CH], w6 = usq[p1.z * CH], w7 = usq[p1.w * CH];
      const T4 c0 = a0, c1 = a1;
      k += 8;
      const bool more = k + 8 <= z;
      if (more) {
        a0 = *reinterpret_cast<const T4*>(svs + k);
        a1 = *reinterpret_cast<const T4*>(svs + k + 4);
        p0 = *reinterpret_cast<const S4*>(sps + k);
        p1 = *reinterpret_cast<const S4*>(sps + k + 4);
      }
      t += c0.x * w0;
      t += c0.y * w1;
      t += c0.z * w2;
      t += c0.w * w3;
      t += c1.x * w4;
      t += c1.y * w5;
      t += c1.z * w6;
      t += c1.w * w7;
      if (!more) break;
    }
  }
  for (; k + 4 <= z; k += 4) {
    const T4 a = *reinterpret_cast<const T4*>(svs + k);
    const S4 p = *reinterpret_cast<const S4*>(sps + k);
    const VT w0 = usq[p.x * CH], w1 = usq[p.y * CH], w2 = usq[p.z * CH], w3 = usq[p.w * CH];
    t += a.x * w0;
    t += a.y * w1;
    t += a.z * w2;
    t += a.w * w3;
  }
  for (; k < z; ++k) t += svs[k] * usq[sps[k] * CH];
  return t;
}

// j-th of the SPLIT cut points of a row's entries [ka, kz) (j = 0: ka, j = SPLIT: kz): the j / SPLIT point rounded
// down to a multiple of 4 entries from vb, so that every part but the first starts aligned
template <int SPLIT>
__device__ __forceinline__ int lmr_cut(int vb, int ka, int kz, int j) {
  if (j <= 0) return ka;
  if (j >= SPLIT) return kz;
  const int c = ka + (int)((int64_t)(kz - ka) * j / SPLIT);
  return min(max(vb + ((c - vb) & ~3), ka), kz);
}

// Epilogue of the fused level kernel for one 16-byte chunk (offset o) of one row, in two parts: the operands it
// reads (loaded before the row sum, so that their latency overlaps it), then, from the row sum t, the values it
// writes: rn (-> rho), xn (-> x), dn (-> dout).
template <typename T, typename VT>
__device__ __forceinline__ void lmr_epi_load(int row, int64_t o, const T* __restrict__ u, const T* __restrict__ b,
                                             const T* rho, const T* x, const T* __restrict__ dinv, int flags, VT& old,
                                             VT& ui, VT& xo, T& di) {
  if (flags & F_PLAIN) return;
  // no branch around the loads (a load under one is waited for at its end, and with it every older load, such as
  // the next block's staging): x and dinv are read whether or not the flags use them
  const T* ob = (flags & F_RHO_FROM_B) ? b : rho;
  old = *reinterpret_cast<const VT*>(ob + o);
  ui = *reinterpret_cast<const VT*>(u + o);
  xo = *reinterpret_cast<const VT*>(x + o);
  di = dinv[row];
}
template <typename T, typename VT>
__device__ __forceinline__ void lmr_epi_store(int64_t o, VT t, VT old, VT ui, VT xo, T di, T c1, T c2, T* rho, T* x,
                                              T* dout, int flags) {
  if (flags & F_PLAIN) {
    *reinterpret_cast<VT*>(rho + o) = t;
    return;
  }
  const VT r = old - t;
  if (flags & F_RHO_STORE) *reinterpret_cast<VT*>(rho + o) = r;
  if (flags & F_X_ASSIGN)
    *reinterpret_cast<VT*>(x + o) = ui;
  else if (flags & F_X_ADD)
    *reinterpret_cast<VT*>(x + o) = xo + ui;
  if (flags & F_D_OUT) *reinterpret_cast<VT*>(dout + o) = c1 * ui + (c2 * di) * r;
}

// Multi-right-hand-side fine-level kernel with LDS staging (NR columns, interleaved n x NR vectors).  One
// workgroup of TPB = 512 threads per block of consecutive rows (MrBlocks); with at most 80 KiB of LDS, two share
// a compute unit (16 waves).  The block's values and 2-byte column positions and u at its distinct columns
// (CH = NR sizeof(T) / 16 chunks of 16 bytes per column) are staged in LDS with 16-byte loads (nontemporal for the
// matrix), all issued before the first LDS store, so that a workgroup keeps ~60 KB of loads in flight; the column
// list carries one padding entry after its last (read by a block without columns).  Thread t then owns chunk
// q = t % CH of half h = (t / CH) % 2 of row slot t / (2 CH): half 0 sums the row's entries below an aligned
// midpoint, half 1 the rest (each in ascending order, from LDS), the two half sums are added across lanes, and
// half 0 applies the epilogue of k_level to its chunk.  With ord, rows take the slots in order of decreasing
// length, so that the rows of a wave have similar lengths.  A block beyond the staging capacity holds one row,
// which the workgroup sums from global memory: phase j takes the entries j, j + TPB / CH, ..., and the phase sums
// are added in phase order.
template <typename T, int NR, int CAP, int UCAP>
__global__ __launch_bounds__(512) void k_level_lmr(int nrb, const int4* __restrict__ meta,
                                                   const int* __restrict__ ucol, const uint16_t* __restrict__ lidx,
                                                   const int* __restrict__ ord, const int* __restrict__ ptr,
                                                   const int* __restrict__ idx, const T* __restrict__ val,
                                                   const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                                   const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                   const int* __restrict__ skip) {
  constexpr int TPB = 512;
  constexpr int VW = 16 / (int)sizeof(T);  // elements per 16-byte chunk
  constexpr int CH = NR / VW;              // chunks per column
  constexpr int RMAX = 256 / CH;           // row slots
  constexpr int NPH = TPB / CH;            // phases of the single-row path
  constexpr int NVC = CAP / VW + 2;        // value chunks of CAP entries from a 16-byte aligned start
  constexpr int NPC = CAP / 8 + 2;         // position chunks (8 per 16 bytes)
  constexpr int NV = (NVC + TPB - 1) / TPB, NP = (NPC + TPB - 1) / TPB, NU = (UCAP * CH + TPB - 1) / TPB;
  static_assert(NR % VW == 0 && 64 % (2 * CH) == 0 && CAP % 8 == 0 && UCAP * CH >= TPB, "staging geometry");
  typedef T VT __attribute__((ext_vector_type(VW)));
  typedef unsigned int U4 __attribute__((ext_vector_type(4)));
  if (skip && *skip) return;
  const int lb = xcd_block(nrb);
  if (lb < 0) return;
  __shared__ VT sv[NVC + 1];  // the last entry of each array takes the stores of threads beyond the block
  __shared__ U4 sp[NPC + 1];
  __shared__ VT us[UCAP * CH + 1];
  const int tid = threadIdx.x;
  const int q = tid % CH, h = (tid / CH) & 1, slot = tid / (2 * CH);
  // first row, first nonzero and first distinct column of this block and of the next: one round trip, after
  // which the value and position streams can be issued
  const int4 m0 = meta[lb], m1 = meta[lb + 1];
  const int r0 = m0.x, r1 = m1.x;
  const int e0 = m0.y, e1 = m1.y;
  const int u0 = m0.z, nu = m1.z - u0;
  const int vb = e0 & ~(VW - 1), pb = e0 & ~7;
  const int nvc = (e1 - vb + VW - 1) / VW, npc = (e1 - pb + 7) / 8;
  VT t = (VT)0;
  int row = -1;
  VT eold = (VT)0, eui = (VT)0, exo = (VT)0;
  T edi = 0;
  if (nu <= UCAP && nvc <= NVC && npc <= NPC) {  // uniform over the workgroup
    // the row of this thread's slot, its entry range and the epilogue's operands, loaded first so that they
    // overlap the staging
    const int nrow = r1 - r0;
    const int rr = ord ? ord[r0 + min(slot, nrow - 1)] : r0 + min(slot, nrow - 1);
    const int ka = ptr[rr], kz = ptr[rr + 1];
    lmr_epi_load<T, VT>(rr, (int64_t)rr * NR + q * VW, u, b, rho, x, dinv, flags, eold, eui, exo, edi);
    // every thread issues all its loads before the first LDS store, with no divergent branch around them (a load
    // under one is waited for at the branch's end): indices beyond the block are clamped to its last chunk, and
    // threads beyond it store into a spare LDS entry
    VT vv[NV];
    U4 pv[NP];
    int uc[NU];
    VT uv[NU];
    const int vlast = max(nvc - 1, 0), plast = max(npc - 1, 0), ulast = max(nu * CH - 1, 0);
#pragma unroll
    for (int m = 0; m < NV; ++m)
      vv[m] = __builtin_nontemporal_load(reinterpret_cast<const VT*>(val + vb) + min(tid + TPB * m, vlast));
#pragma unroll
    for (int m = 0; m < NP; ++m)
      pv[m] = __builtin_nontemporal_load(reinterpret_cast<const U4*>(lidx + pb) + min(tid + TPB * m, plast));
#pragma unroll
    for (int m = 0; m < NU; ++m) uc[m] = ucol[u0 + min(tid + TPB * m, ulast) / CH];
#pragma unroll
    for (int m = 0; m < NU; ++m) {
      const int i = min(tid + TPB * m, ulast);
      uv[m] = *reinterpret_cast<const VT*>(u + (int64_t)uc[m] * NR + (i % CH) * VW);
    }
#pragma unroll
    for (int m = 0; m < NV; ++m) {
      const int i = tid + TPB * m;
      sv[i < nvc ? i : NVC] = vv[m];
    }
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      const int i = tid + TPB * m;
      sp[i < npc ? i : NPC] = pv[m];
    }
#pragma unroll
    for (int m = 0; m < NU; ++m) {
      const int i = tid + TPB * m;
      us[i < nu * CH ? i : UCAP * CH] = uv[m];
    }
    if (slot < nrow) row = rr;
    asm volatile("" ::"v"(ka), "v"(kz));  // keeps the entry-range loads ahead of the barrier
    __syncthreads();
    if (row >= 0) {
      t = lmr_row_sum<T, VT, CH>(reinterpret_cast<const T*>(sv) - vb, reinterpret_cast<const uint16_t*>(sp) - pb,
                                 us + q, vb, lmr_cut<2>(vb, ka, kz, h), lmr_cut<2>(vb, ka, kz, h + 1));
    }
#pragma unroll
    for (int w = 0; w < VW; ++w) t[w] += __shfl_xor(t[w], CH, 64);  // half sums of the row (same on both halves)
  } else {  // one row beyond the staging capacity (r1 == r0 + 1)
    const int ph = tid / CH;
    VT acc = (VT)0;
    for (int e = e0 + ph; e < e1; e += NPH)
      acc += val[e] * *reinterpret_cast<const VT*>(u + (int64_t)idx[e] * NR + q * VW);
    us[tid] = acc;
    __syncthreads();
    if (ph == 0) {
      for (int j = 0; j < NPH; ++j) t += us[j * CH + q];
      row = r0;
      lmr_epi_load<T, VT>(row, (int64_t)row * NR + q * VW, u, b, rho, x, dinv, flags, eold, eui, exo, edi);
    }
  }
  if (row >= 0 && h == 0)
    lmr_epi_store<T, VT>((int64_t)row * NR + q * VW, t, eold, eui, exo, edi, c1, c2, rho, x, dout, flags);
}

// Pipelined form of k_level_lmr: one persistent workgroup of 1024 threads per compute unit walks a contiguous run of blocks (runs
// of neighbouring blocks stay on one XCD, whose L2 then serves the columns they share) with two LDS stages.  While
// block i is summed from one stage, block i+1's values, positions, row-pointer and row-order slices and u at its
// distinct columns arrive in the other by direct global-to-LDS loads (no registers held; the loads of a wave fill
// 64 consecutive 16-byte or 4-byte LDS slots), so the HBM stream never waits for the sums.  Block records
// (first row, first nonzero, first distinct column) are read two blocks ahead and the distinct-column indices one
// block ahead.  The two stages alternate in a loop unrolled by two, so that each LDS access names a fixed stage.
// Row order and epilogue are those of k_level_lmr; each row is summed in four aligned parts (16 waves per compute
// unit), added across lanes.  A block's epilogue operands are loaded before its row sums, and its stores are
// issued at the start of the next step.
template <typename T, int NR, int CAP, int UCAP>
struct LmrStage {
  static constexpr int VW = 16 / (int)sizeof(T), CH = NR / VW, RMAX = 256 / CH;
  static constexpr int NVC = CAP / VW + 2, NPC = CAP / 8 + 2, NUC = UCAP * CH;
  typedef T VT __attribute__((ext_vector_type(VW)));
  typedef unsigned int U4 __attribute__((ext_vector_type(4)));
  VT sv[NVC];
  U4 sp[NPC];
  VT us[NUC];
  int rp[RMAX + 1];
  int ord[RMAX];
};

__device__ __forceinline__ void lds_dma16(const void* g, void* l) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 16, 0, 0);
}
__device__ __forceinline__ void lds_dma4(const void* g, void* l) {
  __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                   (__attribute__((address_space(3))) void*)l, 4, 0, 0);
}

template <typename T, int NR, int CAP, int UCAP>
__global__ __launch_bounds__(1024) void k_level_lmr_pipe(int nrb, int nwg, const int4* __restrict__ meta,
                                                         const int* __restrict__ ucol, const uint16_t* __restrict__ lidx,
                                                         const int* __restrict__ ord, const int* __restrict__ ptr,
                                                         const int* __restrict__ idx, const T* __restrict__ val,
                                                         const T* __restrict__ u, const T* __restrict__ b, T* rho,
                                                         T* x, const T* __restrict__ dinv, T* dout, T c1, T c2,
                                                         int flags, const int* __restrict__ skip) {
  typedef LmrStage<T, NR, CAP, UCAP> S;
  typedef typename S::VT VT;
  constexpr int TPB = 1024, SPLIT = 4;
  constexpr int VW = S::VW, CH = S::CH, RMAX = S::RMAX, NVC = S::NVC, NPC = S::NPC, NUC = S::NUC;
  constexpr int NU = (NUC + TPB - 1) / TPB, NPH = TPB / CH;
  static_assert(RMAX <= 64 && RMAX * CH * SPLIT == TPB && NUC >= TPB, "stage geometry");
  if (skip && *skip) return;
  const int lw = xcd_block(nwg);
  if (lw < 0) return;
  const int bb = (int)((int64_t)lw * nrb / nwg), be = (int)((int64_t)(lw + 1) * nrb / nwg);
  if (bb >= be) return;
  // two LDS objects (not one array), so that the compiler sees that the loads into one stage never write the other
  __shared__ S st0, st1;
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const int q = tid % CH, h = (tid / CH) % SPLIT, slot = tid / (CH * SPLIT);
  // float: epilogue operands loaded before the row sums and stores issued one step later (double: both after the
  // row sums; its registers allow neither)
  constexpr bool DEFER = sizeof(T) == 4;
  VT eold = (VT)0, eui = (VT)0, exo = (VT)0, et = (VT)0;
  T edi = 0;
  int prow = -1;  // DEFER: row of the stores still to issue (-1: none)

  auto staged = [&](int4 m0, int4 m1) {
    const int vb = m0.y & ~(VW - 1), pb = m0.y & ~7;
    return m1.z - m0.z <= UCAP && (m1.y - vb + VW - 1) / VW <= NVC && (m1.y - pb + 7) / 8 <= NPC;
  };
  auto load_uc = [&](int4 m0, int4 m1, int* uc) {
    const int last = max((m1.z - m0.z) * CH - 1, 0);
#pragma unroll
    for (int m = 0; m < NU; ++m) uc[m] = ucol[m0.z + min(tid + TPB * m, last) / CH];
  };
  // direct loads of block (m0, m1) into stage D
  auto issue = [&](S& D, int4 m0, int4 m1, const int* uc) {
    if (!staged(m0, m1)) return;
    const int vb = m0.y & ~(VW - 1), pb = m0.y & ~7;
    const int nvc = (m1.y - vb + VW - 1) / VW, npc = (m1.y - pb + 7) / 8, nuc = (m1.z - m0.z) * CH;
    const int nrow = m1.x - m0.x;
    for (int base = wv * 64; base < nvc; base += TPB)
      if (base + ln < nvc) lds_dma16(val + vb + (int64_t)(base + ln) * VW, &D.sv[base]);
    for (int base = wv * 64; base < npc; base += TPB)
      if (base + ln < npc) lds_dma16(lidx + pb + (int64_t)(base + ln) * 8, &D.sp[base]);
#pragma unroll
    for (int m = 0; m < NU; ++m) {
      const int base = m * TPB + wv * 64;
      if (base < nuc && base + ln < nuc)
        lds_dma16(u + (int64_t)uc[m] * NR + ((base + ln) % CH) * VW, &D.us[base]);
    }
    if (wv < 2 && wv * 64 + ln <= nrow) lds_dma4(ptr + m0.x + wv * 64 + ln, &D.rp[wv * 64]);
    if (ord && wv == 2 && ln < nrow) lds_dma4(ord + m0.x + ln, &D.ord[0]);
  };
  // row sums of block (m0, m1) from stage D (part h of SPLIT per thread, parts added across lanes), then the
  // epilogue
  auto compute = [&](S& D, int4 m0, int4 m1) {
    VT t = (VT)0;
    if (staged(m0, m1)) {
      const int nrow = m1.x - m0.x;
      int row = -1;
      if (slot < nrow) {
        const int lr = ord ? D.ord[slot] - m0.x : slot;
        row = m0.x + lr;
        if (DEFER && h == 0)
          lmr_epi_load<T, VT>(row, (int64_t)row * NR + q * VW, u, b, rho, x, dinv, flags, eold, eui, exo, edi);
        const int vb = m0.y & ~(VW - 1), pb = m0.y & ~7;
        const int ka = D.rp[lr], kz = D.rp[lr + 1];
        t = lmr_row_sum<T, VT, CH>(reinterpret_cast<const T*>(D.sv) - vb,
                                   reinterpret_cast<const uint16_t*>(D.sp) - pb, D.us + q, vb,
                                   lmr_cut<SPLIT>(vb, ka, kz, h), lmr_cut<SPLIT>(vb, ka, kz, h + 1));
      }
#pragma unroll
      for (int w = 0; w < VW; ++w) {
        t[w] += __shfl_xor(t[w], CH, 64);
        t[w] += __shfl_xor(t[w], 2 * CH, 64);
      }
      if (row >= 0 && h == 0) {
        if (DEFER) {
          prow = row;
          et = t;
        } else {
          VT lo = (VT)0, lu = (VT)0, lx = (VT)0;
          T ld = 0;
          lmr_epi_load<T, VT>(row, (int64_t)row * NR + q * VW, u, b, rho, x, dinv, flags, lo, lu, lx, ld);
          lmr_epi_store<T, VT>((int64_t)row * NR + q * VW, t, lo, lu, lx, ld, c1, c2, rho, x, dout, flags);
        }
      }
    } else {  // one row beyond the stage capacity: summed from global memory, phase sums added in phase order, and
              // its epilogue applied at once (no load of this path is left in flight)
      const int ph = tid / CH;
      VT acc = (VT)0;
      for (int e = m0.y + ph; e < m1.y; e += NPH)
        acc += val[e] * *reinterpret_cast<const VT*>(u + (int64_t)idx[e] * NR + q * VW);
      D.us[tid] = acc;
      __syncthreads();
      if (ph == 0) {  // the next step's barrier precedes any reuse of the stage
        for (int j = 0; j < NPH; ++j) t += D.us[j * CH + q];
        const int row = m0.x;
        VT lo = (VT)0, lu = (VT)0, lx = (VT)0;
        T ld = 0;
        lmr_epi_load<T, VT>(row, (int64_t)row * NR + q * VW, u, b, rho, x, dinv, flags, lo, lu, lx, ld);
        lmr_epi_store<T, VT>((int64_t)row * NR + q * VW, t, lo, lu, lx, ld, c1, c2, rho, x, dout, flags);
      }
    }
  };
  // DEFER: the stores of the previous block's rows, issued at the start of the next step (their operands are then
  // known to be loaded), so that they are acknowledged while a block is summed rather than at the next wait
  auto flush = [&] {
    if (DEFER && prow >= 0)
      lmr_epi_store<T, VT>((int64_t)prow * NR + q * VW, et, eold, eui, exo, edi, c1, c2, rho, x, dout, flags);
    prow = -1;
  };

  int uc[NU];
  int4 m0 = meta[bb], m1 = meta[bb + 1];
  load_uc(m0, m1, uc);
  issue(st0, m0, m1, uc);
  int4 m2 = bb + 2 <= nrb ? meta[bb + 2] : m1;
  if (bb + 1 < be) load_uc(m1, m2, uc);
  // block bi in stage A: wait for its loads, start block bi + 1's into stage B, prefetch for bi + 2, sum bi
  // (the stages come in as restrict pointers: the compiler then knows that the loads into B never write A and does
  // not wait for them before reading A)
  auto step = [&](S* __restrict__ A, S* __restrict__ B, int bi) {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0) (expcnt, lgkmcnt unconstrained), visible to the compiler
    __syncthreads();
    flush();
    if (bi + 1 < be) issue(*B, m1, m2, uc);
    const int4 m3 = bi + 3 <= nrb ? meta[bi + 3] : m2;
    if (bi + 2 < be) load_uc(m2, m3, uc);
    compute(*A, m0, m1);
    m0 = m1;
    m1 = m2;
    m2 = m3;
  };
  for (int bi = bb; bi < be; bi += 2) {
    step(&st0, &st1, bi);
    if (bi + 1 < be) step(&st1, &st0, bi + 1);
  }
  flush();
}

template <typename T, int NR, int CLS>
static void launch_lmr_t(const MrBlocks& mb, const LevelOp<T>& op, const int* ord, const T* u, const T* b, T* rho,
                         T* x, T* dout, double c1, double c2, int flags, const int* skip, hipStream_t s) {
  if (!mb.meta) throw std::runtime_error("LDS-staged multi-RHS kernel: block records missing");
  hipLaunchKernelGGL((k_level_lmr<T, NR, kMrCap[CLS], kMrUcap[CLS]>), dim3(xcd_grid(mb.nrb)), dim3(512), 0, s, mb.nrb,
                     reinterpret_cast<const int4*>(mb.meta), mb.ucol, mb.lidx, ord, op.ptr, op.idx, op.val, u, b,
                     rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip);
}

template <typename T, int NR, int CLS>
static void launch_lmr_pipe_t(const MrBlocks& mb, const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x,
                              T* dout, double c1, double c2, int flags, const int* skip, hipStream_t s) {
  static const int cus = [] {
    int d = 0, v = 0;
    if (hipGetDevice(&d) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, d) != hipSuccess)
      v = 256;
    return std::max(v, 1);
  }();
  const int nwg = std::min(mb.nrb, cus);
  hipLaunchKernelGGL((k_level_lmr_pipe<T, NR, kMrCap[CLS], kMrUcap[CLS]>), dim3(xcd_grid(nwg)), dim3(1024), 0, s,
                     mb.nrb, nwg, reinterpret_cast<const int4*>(mb.meta), mb.ucol, mb.lidx, mb.ord, op.ptr, op.idx,
                     op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip);
}

template <typename T>
bool launch_level_lmr(const MrBlocks& mb, const LevelOp<T>& op, int nr, bool pipelined, const T* u, const T* b,
                      T* rho, T* x, T* dout, double c1, double c2, int flags, const int* skip, hipStream_t s) {
  const int cls = mr_class(nr, (int)sizeof(T));
  if (cls < 0 || mb.cls != cls || mb.nrb <= 0 || op.blk != 1) return false;
  if constexpr (sizeof(T) == 4) {
    if (pipelined)
      launch_lmr_pipe_t<float, 16, 0>(mb, op, u, b, rho, x, dout, c1, c2, flags, skip, s);
    else
      launch_lmr_t<float, 16, 0>(mb, op, mb.ord, u, b, rho, x, dout, c1, c2, flags, skip, s);
  } else {
    if (cls == 1) {
      if (pipelined)
        launch_lmr_pipe_t<double, 16, 1>(mb, op, u, b, rho, x, dout, c1, c2, flags, skip, s);
      else
        launch_lmr_t<double, 16, 1>(mb, op, mb.ord, u, b, rho, x, dout, c1, c2, flags, skip, s);
    } else {
      if (pipelined)
        launch_lmr_pipe_t<double, 8, 2>(mb, op, u, b, rho, x, dout, c1, c2, flags, skip, s);
      else
        launch_lmr_t<double, 8, 2>(mb, op, mb.ord, u, b, rho, x, dout, c1, c2, flags, skip, s);
    }
  }
  check_launch(pipelined ? "k_level_lmr_pipe" : "k_level_lmr");
  return true;
}
template bool launch_level_lmr<float>(const MrBlocks&, const LevelOp<float>&, int, bool, const float*, const float*,
                                      float*, float*, float*, double, double, int, const int*, hipStream_t);
template bool launch_level_lmr<double>(const MrBlocks&, const LevelOp<double>&, int, bool, const double*,
                                       const double*, double*, double*, double*, double, double, int, const int*,
                                       hipStream_t);



// Block-row variant of the fused kernel for the agglomerated levels, one right-hand side.  One wave per box K,
// L = floor(64 / B) lanes per row: lane (q, s) owns the columns p = s, s + L, ... of row (K, q) (w = nb*B values,
// one contiguous run per row).  Every memory access of the box is put in flight at once: the row's first KMAX
// values per lane (registers), the epilogue operands, and the w entries of u the block row touches (nb stored
// blocks of B consecutive columns, staged in LDS once and shared by the B rows).  Each lane then sums its
// columns in ascending order, the L lane sums of a row are added in lane order through LDS, and lane q applies
// the epilogue of row (K, q).  Dynamic LDS: 4 waves x (maxw + 64) entries, maxw = max_K nb_K * B.
template <typename T, int KMAX, bool KEEP>
__global__ __launch_bounds__(256) void k_level_blockrow(int nbox, int blk, int maxw, const int* __restrict__ bptr,
                                                        const int* __restrict__ bcol, const T* __restrict__ val,
                                                        const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                                        const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                        int nlog) {
  extern __shared__ unsigned char smem_raw[];
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int K = lb * 4 + wv;
  if (K >= nbox) return;  // whole wave leaves; no block-wide barrier follows
  T* xs = reinterpret_cast<T*>(smem_raw) + (size_t)wv * (maxw + 64);
  T* part = xs + maxw;
  const int L = 64 / blk;
  const int q = lane / L, sv = lane - q * L;
  const bool active = q < blk;
  const int j0 = bptr[K], nb = bptr[K + 1] - j0;
  const int w = nb * blk;
  const T* vrow = val + (int64_t)blk * blk * j0 + (int64_t)q * w;
  T v[KMAX];
#pragma unroll
  for (int m = 0; m < KMAX; ++m) {
    const int p = sv + L * m;
    v[m] = (active && p < w) ? ld_matrix<KEEP>(vrow + p) : (T)0;
  }
  const int row = K * blk + lane;
  T p_old = 0, p_u = 0, p_x = 0, p_di = 0;
  if (lane < blk && !(flags & F_PLAIN)) {
    p_old = (flags & F_RHO_FROM_B) ? b[row] : rho[row];
    p_u = u[row];
    if (flags & F_X_ADD) p_x = x[row];
    if (flags & F_D_OUT) p_di = dinv[row];
  }
  for (int p = lane; p < w; p += 64) {
    const int j = p / blk, c = p - j * blk;
    xs[p] = u[(int64_t)bcol[j0 + j] * blk + c];
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  T acc = 0;
  if (active) {
#pragma unroll
    for (int m = 0; m < KMAX; ++m) {
      const int p = sv + L * m;
      if (p < w) acc += v[m] * xs[p];
    }
    for (int p = sv + L * KMAX; p < w; p += L) acc += vrow[p] * xs[p];  // rows longer than L * KMAX
  }
  part[lane] = acc;
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  if (lane < blk) {
    T t = 0;
    for (int s2 = 0; s2 < L; ++s2) t += part[lane * L + s2];
    if (flags & F_PLAIN) {
      rho[row] = t;
    } else {
      const T r = p_old - t;
      if (flags & F_RHO_STORE) rho[row] = r;
      if (flags & F_X_ASSIGN)
        x[row] = p_u;
      else if (flags & F_X_ADD)
        x[row] = p_x + p_u;
      if (flags & F_D_OUT) dout[row] = c1 * p_u + c2 * p_di * r;
    }
  }
}

// LDS bytes of k_level_blockrow for block rows of at most maxw entries
size_t blockrow_lds_bytes(int blk, int maxw, size_t esz) {
  (void)blk;
  return esz * (size_t)4 * (maxw + 64);
}

template <typename T>
void launch_level_blockrow(const LevelOp<T>& op, int maxnb, const T* u, const T* b, T* rho, T* x, T* dout, double c1,
                           double c2, int flags, hipStream_t s) {
  const int nbox = op.n / op.blk;
  const int nlog = (nbox + 3) / 4;
  if (nlog == 0) return;
  const int maxw = maxnb * op.blk;
  const size_t shm = blockrow_lds_bytes(op.blk, maxw, sizeof(T));
  if (shm > 65536) throw std::runtime_error("block-row kernel: block row too wide for LDS");
  if (op.blk > 64) throw std::runtime_error("block-row kernel: more than 64 rows per box");
  if (flags & F_KEEP)
    hipLaunchKernelGGL((k_level_blockrow<T, 16, true>), dim3(xcd_grid(nlog)), dim3(256), shm, s, nbox, op.blk, maxw,
                       op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, nlog);
  else
    hipLaunchKernelGGL((k_level_blockrow<T, 16, false>), dim3(xcd_grid(nlog)), dim3(256), shm, s, nbox, op.blk, maxw,
                       op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, nlog);
  check_launch("k_level_blockrow");
}
template void launch_level_blockrow<float>(const LevelOp<float>&, int, const float*, const float*, float*, float*,
                                           float*, double, double, int, hipStream_t);
template void launch_level_blockrow<double>(const LevelOp<double>&, int, const double*, const double*, double*,
                                            double*, double*, double, double, int, hipStream_t);

// Residual staging of the fused restriction: wave w's rows at [w BLK, (w + 1) BLK) of one LDS array.
template <typename T, int BLK>
__device__ inline T* rsh_data() {
  __shared__ T rsh[4 * BLK];
  return rsh;
}
template <typename T, int BLK>
__device__ inline void rsh_store(int wv, int row, T r) {
  rsh_data<T, BLK>()[wv * BLK + row] = r;
}

// Box-row kernel (2D agglomerated levels: boxes of BLK = 4, 9 or 16 rows): one wave per box K.  Lane p owns the
// positions p + 64 m (m < NP) of the box's block row (w = nb BLK entries; position j BLK + c is column
// bcol[j0 + j] BLK + c): it gathers u there once and multiplies it with that position's value in each of the
// BLK rows, so every value load is a coalesced 256-byte row segment and no column list or LDS staging is
// needed.  The BLK row sums over the 64 lanes come out of a transposing butterfly over 16 slots (each step halves
// the rows a lane keeps and doubles the lanes summed), in a fixed order; lane l then holds row
// 8 b5 + 4 b4 + 2 b3 + b2 (b = bits of l) and the lanes with l % 4 == 0 apply the epilogue of k_level.
// With RESTRICT (nbox a multiple of 4, workgroup G = the four children of parent box G) the workgroup then
// restricts its residuals into the parent's entries of the next level (BoxRestrict).
template <typename T, int BLK, int NP, bool KEEP, bool RESTRICT>
__global__ __launch_bounds__(256) void k_level_boxrow(int nbox, const int* __restrict__ bptr,
                                                      const int* __restrict__ bcol, const T* __restrict__ val,
                                                      const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                                      const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                      int nlog, BoxRestrict<T> rs) {
  static_assert(BLK <= 16, "rows per box");
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  // the wave index is uniform: the box's block-row record then comes through scalar loads
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int K = lb * 4 + wv;
  if (K >= nbox) return;  // whole wave leaves; no barrier follows
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8, b2 = lane & 4;
  const int myrow = (b5 ? 8 : 0) + (b4 ? 4 : 0) + (b3 ? 2 : 0) + (b2 ? 1 : 0);
  const bool owner = (lane & 3) == 0 && myrow < BLK;
  const int row = K * BLK + min(myrow, BLK - 1);  // clamped: every lane loads, only owners use the values
  // All loads below are unconditional per lane (clamped addresses, masked values): a load under a lane-dependent
  // branch would be waited for at the branch's end, which serialised the box's round trips.
  T p_old = 0, p_u = 0, p_x = 0, p_di = 0;
  if (!(flags & F_PLAIN)) {
    p_old = (flags & F_RHO_FROM_B) ? b[row] : rho[row];
    p_u = u[row];
    if (flags & F_X_ADD) p_x = x[row];
    if (flags & F_D_OUT) p_di = dinv[row];
  }
  const int j0 = bptr[K], w = (bptr[K + 1] - j0) * BLK;  // w >= BLK: every box holds its diagonal block
  const T* vb = val + (int64_t)BLK * BLK * j0;  // row q of the box at vb + q w
  T acc[16];
#pragma unroll
  for (int q = 0; q < 16; ++q) acc[q] = 0;
  int pc[NP];
  int cj[NP];
#pragma unroll
  for (int m = 0; m < NP; ++m) {
    pc[m] = min(lane + 64 * m, w - 1);
    cj[m] = bcol[j0 + pc[m] / BLK];
  }
  T v[NP][BLK];
#pragma unroll
  for (int m = 0; m < NP; ++m)
#pragma unroll
    for (int q = 0; q < BLK; ++q) v[m][q] = ld_matrix<KEEP>(vb + (int64_t)q * w + pc[m]);
#pragma unroll
  for (int m = 0; m < NP; ++m) {
    const int c = pc[m] - (pc[m] / BLK) * BLK;
    const T ug = u[(int64_t)cj[m] * BLK + c];
    const T uv = lane + 64 * m < w ? ug : (T)0;
#pragma unroll
    for (int q = 0; q < BLK; ++q) acc[q] += v[m][q] * uv;
  }
  T h8[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) h8[q] = (b5 ? acc[8 + q] : acc[q]) + __shfl_xor(b5 ? acc[q] : acc[8 + q], 32, 64);
  T h4[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) h4[q] = (b4 ? h8[4 + q] : h8[q]) + __shfl_xor(b4 ? h8[q] : h8[4 + q], 16, 64);
  T h2[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) h2[q] = (b3 ? h4[2 + q] : h4[q]) + __shfl_xor(b3 ? h4[q] : h4[2 + q], 8, 64);
  T t = (b2 ? h2[1] : h2[0]) + __shfl_xor(b2 ? h2[0] : h2[1], 4, 64);
  t += __shfl_xor(t, 2, 64);
  t += __shfl_xor(t, 1, 64);
  if (owner) {
    if (flags & F_PLAIN) {
      rho[row] = t;
    } else {
      const T r = p_old - t;
      if (flags & F_RHO_STORE) rho[row] = r;
      if (flags & F_X_ASSIGN)
        x[row] = p_u;
      else if (flags & F_X_ADD)
        x[row] = p_x + p_u;
      if (flags & F_D_OUT) dout[row] = c1 * p_u + c2 * p_di * r;
      if constexpr (RESTRICT) rsh_store<T, BLK>(wv, myrow, r);
    }
  }
  if constexpr (RESTRICT) {
    __syncthreads();  // every wave is present: nbox is a multiple of 4
    if (wv == 0 && lane < BLK) {
      constexpr int k = BLK == 4 ? 2 : BLK == 9 ? 3 : 4, kk = k * k;
      const int q0 = lane % k, q1 = lane / k;
      const T* src = rsh_data<T, BLK>();
      T sum = 0;
      for (int C = 0; C < 4; ++C) {
        const T* m = rs.pt + (int64_t)(lb * 4 + C) * 2 * kk;
        const T* sc = src + C * BLK;
        int qc = 0;
        for (int a1 = 0; a1 < k; ++a1)
          for (int a0 = 0; a0 < k; ++a0, ++qc) sum += (m[a0 * k + q0] * m[kk + a1 * k + q1]) * sc[qc];
      }
      const int64_t tq = (int64_t)lb * BLK + lane;
      rs.bnext[tq] = sum;
      if (rs.dnext) rs.dnext[tq] = rs.dinv_next[tq] * sum * rs.inv_theta_next;
    }
  }
}

bool boxrow_supported(int blk, int maxnb) {
  return (blk == 4 || blk == 9 || blk == 16) && maxnb > 0 && (int64_t)maxnb * blk <= 64 * kBoxRowMaxNP;
}

template <typename T>
void launch_level_boxrow(const LevelOp<T>& op, int maxnb, const T* u, const T* b, T* rho, T* x, T* dout, double c1,
                         double c2, int flags, hipStream_t s, const BoxRestrict<T>* rs) {
  if (!boxrow_supported(op.blk, maxnb)) throw std::runtime_error("box-row kernel: unsupported box shape");
  const int nbox = op.n / op.blk;
  const int nlog = (nbox + 3) / 4;
  if (nlog == 0) return;
  if (rs && (nbox % 4 != 0 || (flags & F_PLAIN) || !rs->pt || !rs->bnext))
    throw std::runtime_error("box-row kernel: fused restriction needs four boxes per parent and a residual");
  const int np = (maxnb * op.blk + 63) / 64;
  const BoxRestrict<T> ra = rs ? *rs : BoxRestrict<T>{};
#define R3_BR(B, N)                                                                                               \
  do {                                                                                                            \
    if (rs) {                                                                                                     \
      if (flags & F_KEEP)                                                                                         \
        hipLaunchKernelGGL((k_level_boxrow<T, B, N, true, true>), dim3(xcd_grid(nlog)), dim3(256), 0, s, nbox,   \
                           op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, nlog,  \
                           ra);                                                                                   \
      else                                                                                                        \
        hipLaunchKernelGGL((k_level_boxrow<T, B, N, false, true>), dim3(xcd_grid(nlog)), dim3(256), 0, s, nbox,  \
                           op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, nlog,  \
                           ra);                                                                                   \
    } else if (flags & F_KEEP) {                                                                                  \
      hipLaunchKernelGGL((k_level_boxrow<T, B, N, true, false>), dim3(xcd_grid(nlog)), dim3(256), 0, s, nbox,    \
                         op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, nlog, ra); \
    } else {                                                                                                      \
      hipLaunchKernelGGL((k_level_boxrow<T, B, N, false, false>), dim3(xcd_grid(nlog)), dim3(256), 0, s, nbox,   \
                         op.ptr, op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, nlog, ra); \
    }                                                                                                             \
  } while (0)
  if (op.blk == 4) {
    if (np == 1) R3_BR(4, 1); else if (np == 2) R3_BR(4, 2); else R3_BR(4, 3);
  } else if (op.blk == 9) {
    if (np == 1) R3_BR(9, 1); else if (np == 2) R3_BR(9, 2); else R3_BR(9, 3);
  } else {
    if (np == 1) R3_BR(16, 1); else if (np == 2) R3_BR(16, 2); else R3_BR(16, 3);
  }
#undef R3_BR
  check_launch("k_level_boxrow");
}
template void launch_level_boxrow<float>(const LevelOp<float>&, int, const float*, const float*, float*, float*,
                                         float*, double, double, int, hipStream_t,
                                         const BoxRestrict<float>*);
template void launch_level_boxrow<double>(const LevelOp<double>&, int, const double*, const double*, double*,
                                          double*, double*, double, double, int, hipStream_t,
                                          const BoxRestrict<double>*);

// Block-row kernel for wide block rows (3D), one right-hand side: a workgroup takes R rows of a box.  A thread owns
// positions tid, tid + 256, ... of the block row in all R rows: it gathers u there once and multiplies it into each row,
// so every value load is a coalesced row segment; the R sums over a wave's lanes come from a transposing butterfly and
// the waves are added in order.  All loads of a batch of NP positions (columns, values, epilogue operands) are issued
// together and only the gather of u waits for the columns.  The earlier kernel staged u in LDS first and read the
// values after that barrier and the epilogue operands after the sums.  3D Q2 48^3 (13,824 rows, 26 MB) float32
// 7.4 -> 5.7 us, 3D Q2 25^3 (3,456 rows) float32 4.9 -> 3.6, 3D Q2 29^3 (3,456 rows) float64 6.4 -> 5.6.
template <typename T, int B, int R, int NP, bool KEEP>
__global__ __launch_bounds__(256) void k_level_blockrow_wg(int nbox, const int* __restrict__ bptr,
                                                           const int* __restrict__ bcol, const T* __restrict__ val,
                                                           const T* __restrict__ u, const T* __restrict__ b, T* rho,
                                                           T* x, const T* __restrict__ dinv, T* dout, T c1, T c2,
                                                           int flags, int nlog) {
  constexpr int CH = (B + R - 1) / R, S = pow2_at_least(R);
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  __shared__ T rs[4][S];
  const int K = lb / CH, q0 = (lb - K * CH) * R;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int j0 = bptr[K], w = (bptr[K + 1] - j0) * B;
  const int nrow = min(R, B - q0);
  const int row = K * B + q0 + min((int)threadIdx.x, nrow - 1);
  T p_old = 0, p_u = 0, p_x = 0, p_di = 0;
  if (!(flags & F_PLAIN)) {
    p_old = (flags & F_RHO_FROM_B) ? b[row] : rho[row];
    p_u = u[row];
    if (flags & F_X_ADD) p_x = x[row];
    if (flags & F_D_OUT) p_di = dinv[row];
  }
  const T* v0 = val + (int64_t)B * B * j0 + (int64_t)q0 * w;
  T acc[S];
#pragma unroll
  for (int r = 0; r < S; ++r) acc[r] = 0;
  for (int p0 = threadIdx.x; p0 < w; p0 += 256 * NP) {
    int cc[NP];
    T vv[NP][R];
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      const int p = min(p0 + 256 * m, w - 1), j = p / B;
      cc[m] = bcol[j0 + j] * B + (p - j * B);
    }
#pragma unroll
    for (int m = 0; m < NP; ++m)
#pragma unroll
      for (int r = 0; r < R; ++r)
        vv[m][r] = ld_matrix<KEEP>(v0 + (int64_t)min(r, nrow - 1) * w + min(p0 + 256 * m, w - 1));
    T uv[NP];
#pragma unroll
    for (int m = 0; m < NP; ++m) uv[m] = u[cc[m]];
#pragma unroll
    for (int m = 0; m < NP; ++m) {
      const bool in = p0 + 256 * m < w;
#pragma unroll
      for (int r = 0; r < R; ++r) acc[r] += in ? vv[m][r] * uv[m] : (T)0;
    }
  }
  int slot = 0;
  const T t = wave_sum_slots<T, S>(acc, lane, slot);
  rs[wv][slot] = t;  // lanes with the same slot store the same value
  __syncthreads();
  if ((int)threadIdx.x < nrow) {
    const T t4 = (rs[0][threadIdx.x] + rs[1][threadIdx.x]) + (rs[2][threadIdx.x] + rs[3][threadIdx.x]);
    if (flags & F_PLAIN) {
      rho[row] = t4;
    } else {
      const T r = p_old - t4;
      if (flags & F_RHO_STORE) rho[row] = r;
      if (flags & F_X_ASSIGN)
        x[row] = p_u;
      else if (flags & F_X_ADD)
        x[row] = p_x + p_u;
      if (flags & F_D_OUT) dout[row] = c1 * p_u + c2 * p_di * r;
    }
  }
}

template <typename T, int B, int R, int NP>
static void launch_blockrow_wg_b(const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x, T* dout, double c1,
                                 double c2, int flags, hipStream_t s) {
  const int nbox = op.n / B;
  const int nlog = nbox * ((B + R - 1) / R);
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(xcd_grid(nlog)), dim3(256), 0, s, nbox, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv,
                       dout, (T)c1, (T)c2, flags, nlog);
  };
  if (flags & F_KEEP)
    go(k_level_blockrow_wg<T, B, R, NP, true>);
  else
    go(k_level_blockrow_wg<T, B, R, NP, false>);
}

template <typename T>
void launch_level_blockrow_wg(const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x, T* dout,
                              double c1, double c2, int flags, hipStream_t s) {
  if (op.n == 0) return;
  // rows of a workgroup: enough workgroups for the smaller levels, and R x NP values of a thread in registers
  switch (op.blk) {
    case 8: launch_blockrow_wg_b<T, 8, 8, 2>(op, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 9: launch_blockrow_wg_b<T, 9, 9, 2>(op, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 16: launch_blockrow_wg_b<T, 16, 8, 2>(op, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 27: launch_blockrow_wg_b<T, 27, 9, 3>(op, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 64: launch_blockrow_wg_b<T, 64, 8, 4>(op, u, b, rho, x, dout, c1, c2, flags, s); break;
    default: throw std::runtime_error("block-row kernel: unsupported box size");
  }
  check_launch("k_level_blockrow_wg");
}
template void launch_level_blockrow_wg<float>(const LevelOp<float>&, const float*, const float*, float*, float*,
                                              float*, double, double, int, hipStream_t);
template void launch_level_blockrow_wg<double>(const LevelOp<double>&, const double*, const double*, double*,
                                               double*, double*, double, double, int, hipStream_t);

// Fine level for several right-hand sides over chunked rows (see k_level_chunk; n x NR interleaved vectors).  A workgroup
// takes a block of at most CAPC chunks, RPB rows and UCAP - 1 distinct columns and stages its values, positions,
// u rows (all NR columns) and row bounds in LDS, every load of the block issued at once; one barrier later each row is
// summed by CL x NG lanes (CL chunks at a time, NG pieces of W columns), a lane reading four values, four positions and
// four W-column pieces of u per step; the CL partial sums are added by a butterfly.  The rows of a block are taken in
// order of decreasing length, so that the rows a wave sums together are about equally long.  Row sums pass through
// LDS to the epilogue, whose operands were fetched first and whose accesses are consecutive.
// One application, best of the other kernels -> this one: float32, 16 columns, 3D Q3 16^3 53.8 -> 41.8 us and 28^3
// 243 -> 213; 8 columns, 2D Q3 200^2 44.3 -> 24.4; float64, 4 columns, 3D Q2 20^3 21.3 -> 14.1.  With 16 float64
// columns the column-split kernel stays ahead (62 against 66 us).  At 16 float32 columns LDS is busy 52% of the time
// (a quarter of that bank conflicts), the vector units 59%, and 16 waves per compute unit wait 55% of theirs: no one
// unit bounds it, and reading two chunks a step ahead changed nothing.
template <typename T, int NR>
struct MrShape {
  static constexpr int W = NR * (int)sizeof(T) >= 16 ? 16 / (int)sizeof(T) : NR;  // columns per lane
  static constexpr int NG = NR / W;                                              // lanes per chunk
  static constexpr int CL = NG >= 8 ? 2 : 4;                                     // chunks of a row at a time
  typedef T vec __attribute__((ext_vector_type(W)));
  // LDS slot of column position p.  A row of u covers 1 / C of the banks.  The entries that CL lanes read together lie
  // four positions apart where a row's columns are consecutive, in the same part of the banks for C <= 4 (and every
  // other one for C = 8), so the parts are rotated from one group of positions to the next.
  static constexpr int C = 256 / (NG * W * (int)sizeof(T));
  static __device__ __forceinline__ int slot(int p) {
    if constexpr (C > 8 || C < 2)
      return p;
    else
      return (p & ~(C - 1)) | ((p + (p >> (C == 8 ? 3 : 2))) & (C - 1));
  }
};
template <typename T, int NR, int NT, int CAPC, int RPB, int UCAP, bool KEEP>
__global__ __launch_bounds__(NT) void k_level_chunk_mr(int nrb, const int4* __restrict__ meta,
                                                       const int* __restrict__ ucol, const uint32_t* __restrict__ clo,
                                                       const uint8_t* __restrict__ chi, const int* __restrict__ cptr,
                                                       const uint8_t* __restrict__ ord, const T* __restrict__ cval,
                                                       const int* __restrict__ ptr, const int* __restrict__ idx,
                                                       const T* __restrict__ val, const T* __restrict__ u,
                                                       const T* __restrict__ b, T* rho, T* x,
                                                       const T* __restrict__ dinv, T* dout, T c1, T c2, int flags,
                                                       const int* __restrict__ skip) {
  using V4 = typename Vec4<T>::type;
  using MS = MrShape<T, NR>;
  using VW = typename MS::vec;
  constexpr int W = MS::W, NG = MS::NG, CL = MS::CL, LPR = CL * NG, RPP = NT / LPR;
  constexpr int NCH = CAPC / NT, UPT = (UCAP * NG + NT - 1) / NT, EP = (RPB * NG + NT - 1) / NT;
  static_assert(CAPC % NT == 0 && NT % LPR == 0, "staging shape");
  if (skip && *skip) return;
  const int lb = xcd_block(nrb);
  if (lb < 0) return;
  __shared__ VW us[UCAP * NG];
  __shared__ V4 sv[CAPC];
  __shared__ uint2 sp[CAPC];  // four 16-bit indices into us (of piece 0)
  __shared__ VW st[RPB * NG];
  __shared__ int sr[RPB + 1];
  __shared__ uint8_t so[RPB];
  const int4 m0 = meta[lb], m1 = meta[lb + 1];
  const int r0 = m0.x, nr = m1.x - r0;
  const int k0 = m0.y, nk = m1.y - k0;
  const int u0 = m0.z, nu = m1.z - u0;
  const bool staged = nu < UCAP && nk <= CAPC;
  const VW* uv = reinterpret_cast<const VW*>(u);
  // epilogue operands: the block's nr x NG pieces are consecutive
  VW p_old[EP], p_u[EP], p_x[EP];
  T p_di[EP];
#pragma unroll
  for (int m = 0; m < EP; ++m) {
    const int e = min((int)threadIdx.x + m * NT, nr * NG - 1);
    const int64_t o = (int64_t)r0 * NG + e;
    p_old[m] = p_u[m] = p_x[m] = VW(0);
    p_di[m] = 0;
    if (!(flags & F_PLAIN)) {
      p_old[m] = reinterpret_cast<const VW*>((flags & F_RHO_FROM_B) ? b : rho)[o];
      p_u[m] = uv[o];
      if (flags & F_X_ADD) p_x[m] = reinterpret_cast<const VW*>(x)[o];
      if (flags & F_D_OUT) p_di[m] = dinv[r0 + e / NG];
    }
  }
  if (staged) {
    int uc[UPT];
#pragma unroll
    for (int m = 0; m < UPT; ++m) uc[m] = ucol[u0 + min(((int)threadIdx.x + m * NT) / NG, nu - 1)];  // nu >= 1
    uint32_t lo[NCH], hi[NCH];
    V4 vv[NCH];
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      const int k = k0 + min((int)threadIdx.x + m * NT, nk - 1);
      lo[m] = ld_matrix<KEEP>(clo + k);
      hi[m] = ld_matrix<KEEP>(chi + k);
      vv[m] = ld_matrix<KEEP>(reinterpret_cast<const V4*>(cval) + k);
    }
    const int rr = min((int)threadIdx.x, RPB);
    const int cp = cptr[r0 + min(rr, nr)] - k0;
    const int od = ord[r0 + min(rr, nr - 1)];
    VW ug[UPT];
#pragma unroll
    for (int m = 0; m < UPT; ++m) ug[m] = uv[(int64_t)uc[m] * NG + threadIdx.x % NG];  // NT is a multiple of NG
    // keep every load ahead of the LDS writes (the compiler would otherwise sink some of them behind others' waits)
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      asm volatile("" ::"v"(lo[m]), "v"(hi[m]));
#pragma unroll
      for (int q = 0; q < 4; ++q) asm volatile("" ::"v"(vv[m][q]));
    }
#pragma unroll
    for (int m = 0; m < NCH; ++m) {
      const int e = threadIdx.x + m * NT;
      sv[e] = vv[m];
      uint32_t q[4];
#pragma unroll
      for (int v = 0; v < 4; ++v)
        q[v] = NG * MS::slot(((lo[m] >> (8 * v)) & 0xff) | (((hi[m] >> (2 * v)) & 3) << 8));
      sp[e] = make_uint2(q[0] | (q[1] << 16), q[2] | (q[3] << 16));
    }
    if (threadIdx.x <= RPB) sr[threadIdx.x] = cp;
    if (threadIdx.x < RPB) so[threadIdx.x] = (uint8_t)od;
#pragma unroll
    for (int m = 0; m < UPT; ++m) {
      const int e = threadIdx.x + m * NT;
      // position nu holds zero: the padding entries' position
      if (e < UCAP * NG) us[MS::slot(e / NG) * NG + e % NG] = e < nu * NG ? ug[m] : VW(0);
    }
    __syncthreads();
    const int g = threadIdx.x % NG, cl = threadIdx.x / NG % CL;
    for (int q = threadIdx.x / LPR; q < nr; q += RPP) {
      const int row = so[q];
      const int ke = sr[row + 1];
      VW acc = VW(0);
#pragma unroll 2
      for (int k = sr[row] + cl; k < ke; k += CL) {
        const V4 a = sv[k];
        const uint2 ps = sp[k];
        acc += a[0] * us[(ps.x & 0xffff) + g];
        acc += a[1] * us[(ps.x >> 16) + g];
        acc += a[2] * us[(ps.y & 0xffff) + g];
        acc += a[3] * us[(ps.y >> 16) + g];
      }
#pragma unroll
      for (int off = NG; off < LPR; off <<= 1)
#pragma unroll
        for (int w = 0; w < W; ++w) acc[w] += __shfl_xor(acc[w], off, 64);
      if (cl == 0) st[row * NG + g] = acc;
    }
  } else {  // one long row, from memory: every NG lanes take an entry, partial sums added in thread order
    VW acc = VW(0);
    for (int e = ptr[r0] + threadIdx.x / NG; e < ptr[r0 + 1]; e += NT / NG)
      acc += val[e] * uv[(int64_t)idx[e] * NG + threadIdx.x % NG];
    static_assert(UCAP * NG >= NT, "staging of the partial sums");
    us[threadIdx.x] = acc;
    __syncthreads();
    if (threadIdx.x < NG) {
      VW t = VW(0);
      for (int q = 0; q < NT / NG; ++q) t += us[q * NG + threadIdx.x];
      st[threadIdx.x] = t;
    }
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < EP; ++m) {
    const int e = threadIdx.x + m * NT;
    if (e >= nr * NG) continue;
    const int64_t o = (int64_t)r0 * NG + e;
    const VW t = st[e];
    if (flags & F_PLAIN) {
      reinterpret_cast<VW*>(rho)[o] = t;
      continue;
    }
    const VW r = p_old[m] - t;
    if (flags & F_RHO_STORE) reinterpret_cast<VW*>(rho)[o] = r;
    if (flags & F_X_ASSIGN)
      reinterpret_cast<VW*>(x)[o] = p_u[m];
    else if (flags & F_X_ADD)
      reinterpret_cast<VW*>(x)[o] = p_x[m] + p_u[m];
    if (flags & F_D_OUT) reinterpret_cast<VW*>(dout)[o] = c1 * p_u[m] + (c2 * p_di[m]) * r;
  }
}

template <typename T, int NR, int G>
static void launch_chunk_mr_t(const ChunkMrBlocks& cb, const LevelOp<T>& op, const T* u, const T* b, T* rho, T* x,
                              T* dout, double c1, double c2, int flags, const int* skip, hipStream_t s) {
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(xcd_grid(cb.nrb)), dim3(kChunkMrThreads[G]), 0, s, cb.nrb,
                       reinterpret_cast<const int4*>(cb.meta), cb.ucol, cb.clo, cb.chi, cb.cptr, cb.ord, op.cval, op.ptr,
                       op.idx, op.val, u, b, rho, x, op.dinv, dout, (T)c1, (T)c2, flags, skip);
  };
  constexpr int NT = kChunkMrThreads[G], C = kChunkCapOf[G], R = kChunkRowsOf[G], U = kChunkUcapOf[G];
  if (flags & F_KEEP)
    go(k_level_chunk_mr<T, NR, NT, C, R, U, true>);
  else
    go(k_level_chunk_mr<T, NR, NT, C, R, U, false>);
}

template <typename T>
void launch_level_chunk_mr(const ChunkMrBlocks& cb, const LevelOp<T>& op, int nr, const T* u, const T* b, T* rho, T* x,
                           T* dout, double c1, double c2, int flags, const int* skip, hipStream_t s) {
  if (cb.nrb == 0 || !op.cval) throw std::runtime_error("multi-RHS chunk kernel: chunked matrix missing");
#define R3MG_CMR(NRV)                                                                                    \
  case NRV:                                                                                              \
    if (cb.geom == 0)                                                                                    \
      launch_chunk_mr_t<T, NRV, 0>(cb, op, u, b, rho, x, dout, c1, c2, flags, skip, s);                  \
    else                                                                                                 \
      launch_chunk_mr_t<T, NRV, 1>(cb, op, u, b, rho, x, dout, c1, c2, flags, skip, s);                  \
    break;
  switch (nr) {
    R3MG_CMR(2)
    R3MG_CMR(4)
    R3MG_CMR(8)
    R3MG_CMR(16)
    default: throw std::runtime_error("multi-RHS chunk kernel: unsupported number of columns");
  }
#undef R3MG_CMR
  check_launch("k_level_chunk_mr");
}
template void launch_level_chunk_mr<float>(const ChunkMrBlocks&, const LevelOp<float>&, int, const float*, const float*,
                                           float*, float*, float*, double, double, int, const int*, hipStream_t);
template void launch_level_chunk_mr<double>(const ChunkMrBlocks&, const LevelOp<double>&, int, const double*,
                                            const double*, double*, double*, double*, double, double, int, const int*,
                                            hipStream_t);

// ---- encoding of the chunk kernels' blocks ----

// LDS table of distinct columns: open addressing, at most half full.  Returns the column's slot and whether this call
// entered it.
template <int H>
__device__ __forceinline__ int col_slot(int* key, int c, bool& entered) {
  int s = (int)((uint32_t)c * 2654435769u % H);
  for (;;) {
    const int old = atomicCAS(key + s, -1, c);
    entered = old == -1;
    if (entered || old == c) return s;
    s = (s + 1) % H;
  }
}
// position of v in the ascending list a[0 .. n): the last one with a[i] <= v
__device__ __forceinline__ int last_at_most(const int* a, int n, int v) {
  int lo = 0, hi = n - 1;
  while (lo < hi) {
    const int m = (lo + hi + 1) >> 1;
    if (a[m] <= v)
      lo = m;
    else
      hi = m - 1;
  }
  return lo;
}

// Step 1, one workgroup per row segment.  Every row that the row and chunk limits let into the next block enters its
// columns into an LDS table that keeps each column's first row; a row's new columns are those that it holds first, and
// the block ends before the row whose running total passes the column limit.  A row beyond the limits by itself is a
// block.  Bound by the chain of a segment's blocks: one round trip each (its columns and row bounds together), then LDS,
// about 5 us a block.  3D Q3 16^3 (117,649 rows, 28 segments of 113 blocks): 0.60 ms, and 0.13 for step 2; on the host both
// took 93 ms on one thread.
template <int CAP, int RPB, int UCAP>
__global__ __launch_bounds__(1024) void k_chunk_cut(int n, int nseg, const int* __restrict__ rowptr,
                                                    const int* __restrict__ cptr, const int* __restrict__ col, int2* blk,
                                                    int2* segn) {
  constexpr int NT = 1024, EPT = 4 * CAP / NT, H = CAP <= 512 ? 4096 : 8192, V = RPB / 64;
  static_assert(4 * CAP % NT == 0 && 8 * CAP <= H && RPB % 64 == 0 && UCAP <= 4 * CAP, "block shape");
  __shared__ int key[H], first[H];
  __shared__ int rp[RPB + 1], cp[RPB + 1], cnt[RPB], res[2];
  const int tid = threadIdx.x;
  const int ra = (int)((int64_t)blockIdx.x * n / nseg), rz = (int)((int64_t)(blockIdx.x + 1) * n / nseg);
  const int last = rowptr[n] - 1;
  int r = ra, eb = rowptr[ra], k = 0, tot = 0;
  while (r < rz) {
    int c[EPT];
#pragma unroll
    for (int m = 0; m < EPT; ++m) c[m] = col[min((int64_t)eb + tid + m * NT, (int64_t)last)];
    if (tid <= RPB) {
      rp[tid] = rowptr[min(r + tid, rz)];
      cp[tid] = cptr[min(r + tid, rz)];
      if (tid < RPB) cnt[tid] = 0;
    }
    for (int i = tid; i < H; i += NT) {
      key[i] = -1;
      first[i] = RPB;
    }
    __syncthreads();
    // rows within the row and chunk limits (the first ones: both grow)
    const int nc = __syncthreads_count(tid < RPB && r + tid < rz && cp[min(tid, RPB - 1) + 1] - cp[0] <= CAP);
    const int len0 = rp[1] - rp[0];
    int nr = 1, nu = len0;
    if (nc > 0 && len0 < UCAP) {
      const int e1 = rp[nc] - eb;  // at most 4 CAP entries
      int row[EPT], slot[EPT];
#pragma unroll
      for (int m = 0; m < EPT; ++m) {
        const int e = tid + m * NT;
        if (e >= e1) continue;
        bool entered;
        row[m] = last_at_most(rp, nc, eb + e);
        slot[m] = col_slot<H>(key, c[m], entered);
        atomicMin(first + slot[m], row[m]);
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < EPT; ++m)
        if (tid + m * NT < e1 && first[slot[m]] == row[m]) atomicAdd(cnt + row[m], 1);
      __syncthreads();
      if (tid < 64) {
        int t[V], sum = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) t[v] = sum += cnt[V * tid + v];
        int run = sum;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
          const int o = __shfl_up(run, off, 64);
          if (tid >= off) run += o;
        }
        int fit = 0;
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const int upto = run - sum + t[v];  // distinct columns of rows 0 .. V tid + v
          const bool ok = V * tid + v < nc && upto < UCAP;
          fit += __popcll(__ballot(ok));
          t[v] = upto;
        }
#pragma unroll
        for (int v = 0; v < V; ++v)
          if (V * tid + v == fit - 1) {
            res[0] = fit;
            res[1] = t[v];
          }
      }
      __syncthreads();
      nr = res[0];
      nu = res[1];
    }
    if (tid == 0) blk[ra + k] = make_int2(r, nu);
    ++k;
    tot += nu;
    r += nr;
    eb = rp[nr];
    __syncthreads();  // rp, res and the table are written again
  }
  if (tid == 0) segn[blockIdx.x] = make_int2(k, tot);
}

// Block records of a segment, one wave: (first row, first chunk, first distinct column, 0), and one past the last block
__global__ __launch_bounds__(64) void k_chunk_meta(int n, int nseg, const int* __restrict__ cptr,
                                                   const int2* __restrict__ blk, const int2* __restrict__ segn,
                                                   int4* __restrict__ meta) {
  const int lane = threadIdx.x, sg = blockIdx.x;
  const int ra = (int)((int64_t)sg * n / nseg);
  int kb = 0, ub = 0;
  for (int j = lane; j < sg; j += 64) {
    kb += segn[j].x;
    ub += segn[j].y;
  }
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    kb += __shfl_xor(kb, off, 64);
    ub += __shfl_xor(ub, off, 64);
  }
  const int nb = segn[sg].x;
  for (int k0 = 0; k0 < nb; k0 += 64) {
    const int k = k0 + lane;
    const int2 b = blk[ra + min(k, nb - 1)];
    const int own = k < nb ? b.y : 0;
    int run = own;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int o = __shfl_up(run, off, 64);
      if (lane >= off) run += o;
    }
    if (k < nb) meta[kb + k] = make_int4(b.x, cptr[b.x], ub + run - own, 0);
    ub += __shfl(run, 63, 64);
  }
  if (sg == nseg - 1 && lane == 0) meta[kb + nb] = make_int4(n, cptr[n], ub, 0);
}

// Step 2, one workgroup per block: its distinct columns in ascending order, the positions of every chunk's columns in that
// list (padding entries: the slot after the last one) and the order of its rows, equal ones in row order.  The lists and
// positions of a block of one row beyond the limits are never read.
template <int CAP, int RPB, int UCAP>
__global__ __launch_bounds__(512) void k_chunk_lists(const int4* __restrict__ meta, const int* __restrict__ rowptr,
                                                     const int* __restrict__ cptr, const int* __restrict__ col, int* ucol,
                                                     uint32_t* clo, uint8_t* chi, uint8_t* ord) {
  constexpr int NT = 512, H = CAP <= 512 ? 4096 : 8192, P = UCAP <= 512 ? 512 : 1024;
  __shared__ int key[H], list[P];
  __shared__ int rp[RPB + 1], cp[RPB + 1], count;
  const int tid = threadIdx.x;
  const int4 m0 = meta[blockIdx.x], m1 = meta[blockIdx.x + 1];
  const int r0 = m0.x, nr = m1.x - r0, k0 = m0.y, nk = m1.y - k0, u0 = m0.z, nu = m1.z - u0;
  if (tid <= nr) {
    rp[tid] = rowptr[r0 + tid];
    cp[tid] = cptr[r0 + tid] - k0;
  }
  for (int i = tid; i < H; i += NT) key[i] = -1;
  for (int i = tid; i < P; i += NT) list[i] = 0x7fffffff;
  if (tid == 0) count = 0;
  __syncthreads();
  if (ord && tid < nr) {
    const int len = cp[tid + 1] - cp[tid];
    int k = 0;
    for (int j = 0; j < nr; ++j) {
      const int lj = cp[j + 1] - cp[j];
      k += lj > len || (lj == len && j < tid);
    }
    ord[r0 + k] = (uint8_t)tid;
  }
  if (nu >= UCAP || nk > CAP) return;
  for (int e = rp[0] + tid; e < rp[nr]; e += NT) {
    bool entered;
    const int c = col[e];
    col_slot<H>(key, c, entered);
    if (entered) list[atomicAdd(&count, 1)] = c;
  }
  for (int w = 2; w <= P; w <<= 1)
    for (int h = w >> 1; h >= 1; h >>= 1) {
      __syncthreads();
      for (int i = tid; i < P / 2; i += NT) {
        const int a = 2 * h * (i / h) + i % h, b = a + h;  // pairs of a bitonic merge
        const bool up = (a & w) == 0;
        const int va = list[a], vb = list[b];
        if ((va > vb) == up) {
          list[a] = vb;
          list[b] = va;
        }
      }
    }
  __syncthreads();
  for (int i = tid; i < nu; i += NT) ucol[u0 + i] = list[i];
  for (int k = tid; k < nk; k += NT) {
    const int row = last_at_most(cp, nr, k);
    const int e0 = rp[row] + 4 * (k - cp[row]), e1 = rp[row + 1];
    uint32_t lo = 0, hi = 0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const uint32_t ps = e0 + m < e1 ? (uint32_t)last_at_most(list, nu, col[e0 + m]) : (uint32_t)nu;
      lo |= (ps & 0xff) << (8 * m);
      hi |= (ps >> 8) << (2 * m);
    }
    clo[k0 + k] = lo;
    chi[k0 + k] = (uint8_t)hi;
  }
}

template <typename F>
static void chunk_geom_dispatch(int g, F&& f) {
  switch (g) {
    case 0: f(std::integral_constant<int, 0>{}); break;
    case 1: f(std::integral_constant<int, 1>{}); break;
    case 2: f(std::integral_constant<int, 2>{}); break;
    default: throw std::runtime_error("chunk blocks: unknown geometry");
  }
}
void launch_chunk_cut(const ChunkLists& c, hipStream_t s) {
  chunk_geom_dispatch(c.geom, [&](auto g) {
    hipLaunchKernelGGL((k_chunk_cut<kChunkCapOf[g.value], kChunkRowsOf[g.value], kChunkUcapOf[g.value]>), dim3(c.nseg),
                       dim3(1024), 0, s, c.n, c.nseg, c.rowptr, c.cptr, c.col, c.blk, c.segn);
  });
  check_launch("k_chunk_cut");
}
void launch_chunk_lists(const ChunkLists& c, hipStream_t s) {
  int4* meta = reinterpret_cast<int4*>(c.meta);
  hipLaunchKernelGGL(k_chunk_meta, dim3(c.nseg), dim3(64), 0, s, c.n, c.nseg, c.cptr, c.blk, c.segn, meta);
  chunk_geom_dispatch(c.geom, [&](auto g) {
    hipLaunchKernelGGL((k_chunk_lists<kChunkCapOf[g.value], kChunkRowsOf[g.value], kChunkUcapOf[g.value]>), dim3(c.nrb),
                       dim3(512), 0, s, meta, c.rowptr, c.cptr, c.col, c.ucol, c.clo, c.chi, c.ord);
  });
  check_launch("k_chunk_lists");
}

// 16 x 16 x 4 matrix instructions.  Lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16]; result element r of lane l is
// C[row(l, r)][l % 16].
template <typename T>
struct Mfma16;
template <>
struct Mfma16<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  typedef float load __attribute__((ext_vector_type(4), aligned(4)));
  static constexpr int KV = 4;
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }  // of result element r
};
template <>
struct Mfma16<double> {
  typedef v4d acc;
  typedef double load __attribute__((ext_vector_type(2), aligned(8)));
  static constexpr int KV = 2;
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lane, int r) { return 4 * r + (lane >> 4); }
};

// Agglomerated levels for several right-hand sides, on the matrix cores: one workgroup per box, the box's B x w block
// row times the w x NR gathered rows of u, as 16 x 16 x 4 products (rows of the box x columns x block-row positions).
// The four waves take every fourth step of 4 KV positions and add their tiles in wave order through LDS; a lane's KV
// consecutive positions (16 bytes of the matrix row) are the four k groups of KV instructions, the same for both
// operands.  Epilogue as in k_level, operands fetched first.
// The lanes kernel gives each lane whole positions and all NR columns, so it is a long chain of loads per lane and a
// butterfly per column at the end; here a step is one 16-byte load, KV gathered words and KV instructions.  One
// application, best lanes count -> this kernel: float64 with 8 columns, 9-row boxes, 9,216 rows 14.1 -> 5.7 us and
// 2,304 rows 10.5 -> 3.9; float32 with 16 columns, 27-row boxes (3D Q3 28^3) 50.5 -> 12.1 us.  Now bound by the three
// dependent round trips (block row, columns, u) and the launch.
template <typename T, int B, int NR>
__global__ __launch_bounds__(256) void k_level_box_mr(int nbox, const int* __restrict__ bptr,
                                                      const int* __restrict__ bcol, const T* __restrict__ val,
                                                      const T* __restrict__ u, const T* __restrict__ b, T* rho, T* x,
                                                      const T* __restrict__ dinv, T* dout, T c1, T c2, int flags) {
  using M = Mfma16<T>;
  constexpr int MT = (B + 15) / 16, KV = M::KV, KS = 4 * KV, UN = 2;
  constexpr int EP = (B * NR + 255) / 256;
  const int K = xcd_block(nbox);
  if (K < 0) return;
  __shared__ T red[4][MT * 16][NR];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, kk = lane >> 4, n = i % NR;
  const int j0 = bptr[K], nb = bptr[K + 1] - j0, w = nb * B;
  const int bc = bcol[j0 + min(lane, nb - 1)];  // lane j: block column j (nb <= 64)
  // epilogue operands: the box's B x NR entries are consecutive
  const int64_t ebase = (int64_t)K * B * NR;
  T p_old[EP], p_u[EP], p_x[EP], p_di[EP];
#pragma unroll
  for (int m = 0; m < EP; ++m) {
    const int e = min((int)threadIdx.x + 256 * m, B * NR - 1);
    p_old[m] = p_u[m] = p_x[m] = p_di[m] = 0;
    if (!(flags & F_PLAIN)) {
      p_old[m] = (flags & F_RHO_FROM_B) ? b[ebase + e] : rho[ebase + e];
      p_u[m] = u[ebase + e];
      if (flags & F_X_ADD) p_x[m] = x[ebase + e];
      if (flags & F_D_OUT) p_di[m] = dinv[(int64_t)K * B + e / NR];
    }
  }
  const T* vrow[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) vrow[t] = val + (int64_t)B * B * j0 + (int64_t)min(16 * t + i, B - 1) * w;
  typename M::acc acc[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = typename M::acc{0, 0, 0, 0};
  const int S = (w + KS - 1) / KS;
  for (int s0 = wv; s0 < S; s0 += 4 * UN) {
    typename M::load av[UN][MT];
    T uv[UN][KV];
#pragma unroll
    for (int h = 0; h < UN; ++h) {
      const int k0 = (s0 + 4 * h) * KS + kk * KV;
      // a load that starts inside the row may run past its end by KV - 1 entries (the values carry kFinePad of them)
#pragma unroll
      for (int t = 0; t < MT; ++t) av[h][t] = *reinterpret_cast<const typename M::load*>(vrow[t] + min(k0, w - 1));
#pragma unroll
      for (int q = 0; q < KV; ++q) {
        const int k = min(k0 + q, w - 1), jb = k / B;
        uv[h][q] = u[((int64_t)__shfl(bc, jb, 64) * B + (k - jb * B)) * NR + n];
      }
    }
#pragma unroll
    for (int h = 0; h < UN; ++h) {
      const int k0 = (s0 + 4 * h) * KS + kk * KV;
#pragma unroll
      for (int q = 0; q < KV; ++q) {
        const bool in = k0 + q < w;  // beyond the row: zero in both operands
        const T uq = in ? uv[h][q] : (T)0;
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t] = M::mma(in ? av[h][t][q] : (T)0, uq, acc[t]);
      }
    }
  }
  if (i < NR) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wv][16 * t + M::row(lane, r)][i] = acc[t][r];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < EP; ++m) {
    const int e = threadIdx.x + 256 * m;
    if (e >= B * NR) continue;
    const int q = e / NR, c = e % NR;
    const T t = (red[0][q][c] + red[1][q][c]) + (red[2][q][c] + red[3][q][c]);
    const int64_t o = ebase + e;
    if (flags & F_PLAIN) {
      rho[o] = t;
      continue;
    }
    const T r = p_old[m] - t;
    if (flags & F_RHO_STORE) rho[o] = r;
    if (flags & F_X_ASSIGN)
      x[o] = p_u[m];
    else if (flags & F_X_ADD)
      x[o] = p_x[m] + p_u[m];
    if (flags & F_D_OUT) dout[o] = c1 * p_u[m] + c2 * p_di[m] * r;
  }
}

bool box_mr_supported(int blk, int maxnb) {
  return maxnb >= 1 && maxnb <= 64 && (blk == 4 || blk == 8 || blk == 9 || blk == 16 || blk == 27 || blk == 64);
}

template <typename T, int B>
static void launch_box_mr_b(const LevelOp<T>& op, int nr, const T* u, const T* b, T* rho, T* x, T* dout, double c1,
                            double c2, int flags, hipStream_t s) {
  const int nbox = op.n / B;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(xcd_grid(nbox)), dim3(256), 0, s, nbox, op.ptr, op.idx, op.val, u, b, rho, x, op.dinv,
                       dout, (T)c1, (T)c2, flags);
  };
  switch (nr) {
    case 2: go(k_level_box_mr<T, B, 2>); break;
    case 4: go(k_level_box_mr<T, B, 4>); break;
    case 8: go(k_level_box_mr<T, B, 8>); break;
    case 16: go(k_level_box_mr<T, B, 16>); break;
    default: throw std::runtime_error("multi-RHS box kernel: unsupported number of columns");
  }
}

template <typename T>
void launch_level_box_mr(const LevelOp<T>& op, int nr, const T* u, const T* b, T* rho, T* x, T* dout, double c1,
                         double c2, int flags, hipStream_t s) {
  if (op.n == 0) return;
  switch (op.blk) {
    case 4: launch_box_mr_b<T, 4>(op, nr, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 8: launch_box_mr_b<T, 8>(op, nr, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 9: launch_box_mr_b<T, 9>(op, nr, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 16: launch_box_mr_b<T, 16>(op, nr, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 27: launch_box_mr_b<T, 27>(op, nr, u, b, rho, x, dout, c1, c2, flags, s); break;
    case 64: launch_box_mr_b<T, 64>(op, nr, u, b, rho, x, dout, c1, c2, flags, s); break;
    default: throw std::runtime_error("multi-RHS box kernel: unsupported box size");
  }
  check_launch("k_level_box_mr");
}
template void launch_level_box_mr<float>(const LevelOp<float>&, int, const float*, const float*, float*, float*, float*,
                                         double, double, int, hipStream_t);
template void launch_level_box_mr<double>(const LevelOp<double>&, int, const double*, const double*, double*, double*,
                                          double*, double, double, int, hipStream_t);

// q = A p with per-block partial sums of p.q (float64 CSR)
template <int NR>
__global__ __launch_bounds__(256) void k_spmv_dot(int n, int G, const int* __restrict__ ptr,
                                                  const int* __restrict__ idx, const double* __restrict__ val,
                                                  const double* __restrict__ p, double* q, double* partials,
                                                  const int* __restrict__ skip, int nlog) {
  if (skip && *skip) return;
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  __shared__ double sh[4 * NR];
  const int rpb = 256 / G;
  const int lane = threadIdx.x & (G - 1);
  const int row = lb * rpb + threadIdx.x / G;
  const bool active = row < n;
  double acc[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) acc[k] = 0;
  if (active) row_product<double, NR, false>(row, lane, G, 1, ptr, idx, val, p, acc);
#pragma unroll
  for (int k = 0; k < NR; ++k) acc[k] = wave_sum(acc[k], G);
  double contrib[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    contrib[k] = 0;
    if (active && lane == 0) {
      const int64_t i = (int64_t)row * NR + k;
      q[i] = acc[k];
      contrib[k] = acc[k] * p[i];
    }
  }
  // block reduction (fixed order)
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    double v = wave_sum(contrib[k], 64);
    if ((threadIdx.x & 63) == 0) sh[(threadIdx.x >> 6) * NR + k] = v;
  }
  __syncthreads();
  if (threadIdx.x < NR) {
    const int k = threadIdx.x;
    partials[(int64_t)lb * NR + k] = (sh[k] + sh[NR + k]) + (sh[2 * NR + k] + sh[3 * NR + k]);
  }
}

int launch_spmv_dot(const LevelOp<double>& op, int nr, const double* p, double* q, double* partials,
                    const int* skip, hipStream_t s) {
  const int G = op.lanes;
  const int rpb = 256 / G;
  const int nlog = (op.n + rpb - 1) / rpb;
  dim3 grid(xcd_grid(nlog));
#define R3_SD(NRV) \
  hipLaunchKernelGGL((k_spmv_dot<NRV>), grid, dim3(256), 0, s, op.n, G, op.ptr, op.idx, op.val, p, q, partials, skip, nlog)
  switch (nr) {
    case 1: R3_SD(1); break;
    case 2: R3_SD(2); break;
    case 4: R3_SD(4); break;
    case 8: R3_SD(8); break;
    case 16: R3_SD(16); break;
    default: throw std::runtime_error("unsupported nrhs block");
  }
#undef R3_SD
  check_launch("k_spmv_dot");
  return nlog;
}

// =============================================================================================
// Transfers
// =============================================================================================
// Several right-hand sides (nr > 1, interleaved: entry i of column c at i * nr + c): the transfer kernels below
// give each thread a chunk of VW = min(nr, 16 bytes / sizeof(T)) adjacent columns, loaded and stored as one
// vector, so the basis functions and transfer entries are formed once per chunk instead of once per column.
// Each column is summed in the same order as the one-column kernel, except k_restrict0_mr (points in index order).
template <typename T, int W>
struct ColVec {
  typedef T type __attribute__((ext_vector_type(W)));
};
template <typename T>
constexpr int col_vw() {
  return 16 / (int)sizeof(T);
}
// the vector path needs 16-byte aligned vectors (always so for the library's buffers)
static inline bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// f(dk) with the dimension and the nodes per axis as the compile-time constants dk.D, dk.K
template <int DD, int KK>
struct BoxShape {
  static constexpr int D = DD, K = KK;
};
template <typename F>
static void box_dispatch(int d, int k, F&& f) {
  switch (d * 8 + k) {
    case 17: f(BoxShape<2, 1>{}); break;
    case 18: f(BoxShape<2, 2>{}); break;
    case 19: f(BoxShape<2, 3>{}); break;
    case 20: f(BoxShape<2, 4>{}); break;
    case 25: f(BoxShape<3, 1>{}); break;
    case 26: f(BoxShape<3, 2>{}); break;
    case 27: f(BoxShape<3, 3>{}); break;
    case 28: f(BoxShape<3, 4>{}); break;
    default: throw std::runtime_error("transfer: unsupported dimension or degree");
  }
}

// Restriction fine -> first agglomerated level, one workgroup of up to eight waves per box K:
// b[K B + q] = sum over the box's free points of phi_q(x_i) src_i.  A thread adds the B products of its points (two at
// a time, loads from clamped addresses, masked afterwards) in registers; the waves' lanes are then added by one
// transposing butterfly and the waves in order through LDS.  dnext = dinv_next b inv_theta_next when it is set.
// Bound by latency (a few hundred boxes, each one chain of loads, products and sums).  The earlier kernel staged every
// product in LDS and summed 64 points of a box at a time: 3D Q2 48^3 float32 (512 boxes of 1,783 points) 11.9 -> 7.2 us,
// 3D Q2 29^3 float64 (128 boxes) 11.6 -> 6.3, 2D Q3 256^2 float32 (8,192 boxes of 72) 6.3 -> 6.1.
template <typename T, int D, int KB>
__global__ __launch_bounds__(512) void k_restrict0(Basis1D<T> bs, int nr, const int* __restrict__ leaf_off,
                                                   const int* __restrict__ owner, const T* __restrict__ xi,
                                                   const T* __restrict__ src, T* bnext, const T* __restrict__ dinv_next,
                                                   T* dnext, T inv_theta_next) {
  constexpr int B = D == 3 ? KB * KB * KB : KB * KB;
  constexpr int S = pow2_at_least(B);
  __shared__ T wt[8][S];
  const int NT = blockDim.x, W = NT >> 6;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int K = blockIdx.x;
  const int i0 = leaf_off[K], i1 = leaf_off[K + 1];
  const int64_t t = (int64_t)K * B + min((int)threadIdx.x, B - 1);
  const T di = dnext ? dinv_next[t] : (T)0;
  for (int c = 0; c < nr; ++c) {
    T acc[S];
#pragma unroll
    for (int q = 0; q < S; ++q) acc[q] = 0;
    for (int base = i0 + threadIdx.x; base < i1; base += 2 * NT) {
      T r[2], x[2][3];
      bool ok[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int i = min(base + h * NT, i1 - 1);
        const int ow = owner[i];
        r[h] = src[(int64_t)i * nr + c];
#pragma unroll
        for (int a = 0; a < D; ++a) x[h][a] = xi[(int64_t)i * D + a];
        ok[h] = ow >= 0 && base + h * NT < i1;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const T rv = ok[h] ? r[h] : (T)0;
        T l[3][4];
#pragma unroll
        for (int a = 0; a < D; ++a) lag1d_k<T, KB>(bs, x[h][a], l[a]);
        for_each_phi<T, D, KB>(l, [&](int q, T ph) { acc[q] += ph * rv; });
      }
    }
    int slot = 0;
    const T w = wave_sum_slots<T, S>(acc, lane, slot);
    wt[wv][slot] = w;  // lanes with the same slot store the same value
    __syncthreads();
    if (threadIdx.x < B) {
      T v = 0;
      for (int u = 0; u < W; ++u) v += wt[u][threadIdx.x];
      bnext[t * nr + c] = v;
      if (dnext) dnext[t * nr + c] = di * v * inv_theta_next;
    }
    __syncthreads();
  }
}

// Restriction fine -> first agglomerated level for NR > 1 columns, one workgroup of up to eight waves per box, on the
// matrix cores: the B x points matrix phi_q(x_i) times the points x NR entries of src, four points an instruction.
// Lane (i, k) evaluates phi_q at point k for q = 16 t + i in every tile t (its weights and nodes per axis are held in
// registers) and supplies column i % NR of src at that point (zero at constrained points and past the box).  The waves
// take the points in turn and their tiles are added in wave order through LDS.
// The earlier kernel staged 32 points' values and entries in LDS per team of lanes and summed point by point: 3D Q3
// 16^3, 16 float32 columns (64 boxes of 1,838 points) 63 us with four teams, 36.5 with eight, now 28.3.
template <typename T, int D, int KB, int NR>
__global__ __launch_bounds__(512) void k_restrict0_mr(Basis1D<T> bs, const int* __restrict__ leaf_off,
                                                      const int* __restrict__ owner, const T* __restrict__ xi,
                                                      const T* __restrict__ src, T* bnext,
                                                      const T* __restrict__ dinv_next, T* dnext, T inv_theta_next) {
  using M = Mfma16<T>;
  constexpr int B = D == 3 ? KB * KB * KB : KB * KB;
  constexpr int MT = (B + 15) / 16, UN = 2;
  __shared__ T red[8][MT * 16][NR];
  const int W = blockDim.x >> 6, wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = lane & 15, kk = lane >> 4, n = i % NR;
  const int K = blockIdx.x;
  const int i0 = leaf_off[K], i1 = leaf_off[K + 1];
  // phi_q = prod over axes of w (s - t_1) .. (s - t_{KB-1}): the weight and the other nodes of this lane's functions
  T wq[MT], tn[MT][D][KB > 1 ? KB - 1 : 1];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    int q = min(16 * t + i, B - 1);
    wq[t] = 1;
#pragma unroll
    for (int a = 0; a < D; ++a) {
      const int j = q % KB;
      q /= KB;
      T w = bs.w[0];
#pragma unroll
      for (int m = 1; m < KB; ++m) w = j == m ? bs.w[m] : w;
      wq[t] *= w;
#pragma unroll
      for (int m = 0; m + 1 < KB; ++m) {
        // the m-th node other than node j
        tn[t][a][m] = j <= m ? bs.t[m + 1] : bs.t[m];
      }
    }
  }
  typename M::acc acc[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) acc[t] = typename M::acc{0, 0, 0, 0};
  for (int p0 = i0 + 4 * wv; p0 < i1; p0 += 4 * W * UN) {
    T x[UN][D], r[UN];
    int ow[UN];
#pragma unroll
    for (int h = 0; h < UN; ++h) {
      const int p = min(p0 + 4 * W * h + kk, i1 - 1);
      ow[h] = owner[p];
      r[h] = src[(int64_t)p * NR + n];
#pragma unroll
      for (int a = 0; a < D; ++a) x[h][a] = xi[(int64_t)p * D + a];
    }
#pragma unroll
    for (int h = 0; h < UN; ++h) {
      const T rv = (ow[h] >= 0 && p0 + 4 * W * h + kk < i1) ? r[h] : (T)0;
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        T ph = wq[t];
#pragma unroll
        for (int a = 0; a < D; ++a)
#pragma unroll
          for (int m = 0; m + 1 < KB; ++m) ph *= x[h][a] - tn[t][a][m];
        acc[t] = M::mma(ph, rv, acc[t]);
      }
    }
  }
  if (i < NR) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wv][16 * t + M::row(lane, r)][i] = acc[t][r];
  }
  __syncthreads();
  for (int e = threadIdx.x; e < B * NR; e += blockDim.x) {
    const int q = e / NR, c = e % NR;
    T v = 0;
    for (int u = 0; u < W; ++u) v += red[u][q][c];
    const int64_t row = (int64_t)K * B + q;
    bnext[row * NR + c] = v;
    if (dnext) dnext[row * NR + c] = dinv_next[row] * v * inv_theta_next;
  }
}

template <typename T>
void launch_restrict0(int nbox, int64_t n_points, int d, int pc, int nr, const int* leaf_off, const int* owner,
                      const T* xi, const T* src, T* bnext, const T* dinv_next, T* dnext, double inv_theta_next,
                      hipStream_t s) {
  const int k = pc + 1;
  if (nbox == 0) return;
  // waves per box: two points a thread in an average box, at most eight waves
  int W = 1;
  while (W < 8 && (int64_t)W * 128 * nbox < n_points) W <<= 1;
  const Basis1D<T> bs = make_basis<T>(pc);
  if (nr == 2 || nr == 4 || nr == 8 || nr == 16) {
    // waves per box: 32 points (eight instructions a tile) each in an average box, at most eight
    int Wm = 1;
    while (Wm < 8 && (int64_t)Wm * 32 * nbox < n_points) Wm <<= 1;
    box_dispatch(d, k, [&](auto dk) {
      auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(nbox), dim3(64 * Wm), 0, s, bs, leaf_off, owner, xi, src, bnext, dinv_next, dnext,
                           (T)inv_theta_next);
      };
      switch (nr) {
        case 2: go(k_restrict0_mr<T, dk.D, dk.K, 2>); break;
        case 4: go(k_restrict0_mr<T, dk.D, dk.K, 4>); break;
        case 8: go(k_restrict0_mr<T, dk.D, dk.K, 8>); break;
        default: go(k_restrict0_mr<T, dk.D, dk.K, 16>); break;
      }
    });
    check_launch("k_restrict0_mr");
    return;
  }
#define R3MG_R0(DD, KK)                                                                                           \
  hipLaunchKernelGGL((k_restrict0<T, DD, KK>), dim3(nbox), dim3(64 * W), 0, s, bs, nr, leaf_off, owner, xi, src, \
                     bnext, dinv_next, dnext, (T)inv_theta_next)
  switch (d * 8 + k) {
    case 17: R3MG_R0(2, 1); break;
    case 18: R3MG_R0(2, 2); break;
    case 19: R3MG_R0(2, 3); break;
    case 20: R3MG_R0(2, 4); break;
    case 25: R3MG_R0(3, 1); break;
    case 26: R3MG_R0(3, 2); break;
    case 27: R3MG_R0(3, 3); break;
    case 28: R3MG_R0(3, 4); break;
    default: throw std::runtime_error("restriction: unsupported dimension or degree");
  }
#undef R3MG_R0
  check_launch("k_restrict0");
}
template void launch_restrict0<float>(int, int64_t, int, int, int, const int*, const int*, const float*,
                                      const float*, float*, const float*, float*, double, hipStream_t);
template void launch_restrict0<double>(int, int64_t, int, int, int, const int*, const int*, const double*,
                                       const double*, double*, const double*, double*, double,
                                       hipStream_t);

// Prolongation from the first agglomerated level: v_i = sum_q phi^K_q(xi_i) (e + epend)[K*B+q] (0 if i is
// constrained).  One thread per fine point.
template <typename T, int D, int KB>
__global__ __launch_bounds__(256) void k_prolong0(int n, Basis1D<T> bs, int nr, const int* __restrict__ owner,
                                                  const T* __restrict__ xi, const T* __restrict__ e,
                                                  const T* __restrict__ epend, T* v,
                                                  int nlog) {
  constexpr int B = D == 3 ? KB * KB * KB : KB * KB;
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  const int i = lb * 256 + threadIdx.x;
  if (i >= n) return;
  const int K = owner[i];
  if (K < 0) {
    for (int c = 0; c < nr; ++c) v[(int64_t)i * nr + c] = 0;
    return;
  }
  T l[3][4];
#pragma unroll
  for (int a = 0; a < D; ++a) lag1d_k<T, KB>(bs, xi[(int64_t)i * D + a], l[a]);
  for (int c = 0; c < nr; ++c) {
    T s = 0;
    for_each_phi<T, D, KB>(l, [&](int q, T ph) {
      const int64_t o = ((int64_t)K * B + q) * nr + c;
      T ev = e[o];
      if (epend) ev += epend[o];
      s += ph * ev;
    });
    v[(int64_t)i * nr + c] = s;
  }
}

// The same for boxes of many points: `per` workgroups per box, the box's coarse entries (e + epend) in LDS and read by
// all threads at once, phi evaluated axis by axis (KB^2 + KB + 1 sums of KB products instead of B products of D + 1).
// 3D Q2 48^3 float32 (512 boxes of 1,783 points): 17.9 -> 6.2 us.
template <typename T, int D, int KB>
__global__ __launch_bounds__(256) void k_prolong0_box(Basis1D<T> bs, int nr, int per, const int* __restrict__ leaf_off,
                                                      const int* __restrict__ owner, const T* __restrict__ xi,
                                                      const T* __restrict__ e, const T* __restrict__ epend, T* v,
                                                      int nlog) {
  constexpr int B = D == 3 ? KB * KB * KB : KB * KB;
  const int lb = xcd_block(nlog);
  if (lb < 0) return;
  __shared__ T es[B];
  const int K = lb / per, part = lb - K * per;
  const int i0 = leaf_off[K], i1 = leaf_off[K + 1];
  for (int c = 0; c < nr; ++c) {
    if (threadIdx.x < B) {
      const int64_t o = ((int64_t)K * B + threadIdx.x) * nr + c;
      T ev = e[o];
      if (epend) ev += epend[o];
      es[threadIdx.x] = ev;
    }
    __syncthreads();
    for (int i = i0 + part * 256 + threadIdx.x; i < i1; i += per * 256) {
      const int ow = owner[i];
      T l[3][4];
#pragma unroll
      for (int a = 0; a < D; ++a) lag1d_k<T, KB>(bs, xi[(int64_t)i * D + a], l[a]);
      T s2 = 0;
#pragma unroll
      for (int q2 = 0; q2 < (D == 3 ? KB : 1); ++q2) {
        T s1 = 0;
#pragma unroll
        for (int q1 = 0; q1 < KB; ++q1) {
          T s0 = 0;
#pragma unroll
          for (int q0 = 0; q0 < KB; ++q0) s0 += l[0][q0] * es[q0 + KB * q1 + KB * KB * q2];
          s1 += l[1][q1] * s0;
        }
        s2 = D == 3 ? s2 + l[2][q2] * s1 : s1;
      }
      v[(int64_t)i * nr + c] = ow >= 0 ? s2 : (T)0;
    }
    __syncthreads();
  }
}

// The same for nr > 1 columns: `per` workgroups per level-1 box K (its points are leaf_off[K] .. leaf_off[K+1] - 1,
// owned by K or constrained).  Each forms the box's B coarse entries of e + epend (all columns) in LDS; thread (i, j) of
// the box then takes fine point i and column chunk j (chunks of one point adjacent), in k_prolong0's order.  Reading the entries from LDS instead of L2 for every point and chunk was what bounded the kernel.
template <typename T, int D, int KB, int VW>
__global__ __launch_bounds__(256) void k_prolong0_mr(Basis1D<T> bs, int nr, int per, const int* __restrict__ leaf_off,
                                                     const int* __restrict__ owner, const T* __restrict__ xi,
                                                     const T* __restrict__ e, const T* __restrict__ epend, T* v) {
  using VT = typename ColVec<T, VW>::type;
  constexpr int B = D == 3 ? KB * KB * KB : KB * KB;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  VT* es = reinterpret_cast<VT*>(smem_raw);  // [B][nch]
  const int nch = nr / VW;
  const int K = blockIdx.x / per, part = blockIdx.x - K * per;
  const int i0 = leaf_off[K], i1 = leaf_off[K + 1];
  for (int t = threadIdx.x; t < B * nch; t += blockDim.x) {
    const int64_t o = (int64_t)K * B * nr + (int64_t)t * VW;  // entry (K B + t / nch), chunk t % nch
    VT ev = *reinterpret_cast<const VT*>(e + o);
    if (epend) ev += *reinterpret_cast<const VT*>(epend + o);
    es[t] = ev;
  }
  __syncthreads();
  const int total = (i1 - i0) * nch;
  for (int idx = part * 256 + threadIdx.x; idx < total; idx += per * 256) {
    const int i = i0 + idx / nch, j = idx - (idx / nch) * nch;
    const int ow = owner[i];  // unconditional loads; a constrained point's value is replaced by zero
    T l[3][4];
#pragma unroll
    for (int a = 0; a < D; ++a) lag1d_k<T, KB>(bs, xi[(int64_t)i * D + a], l[a]);
    VT sum = (VT)0;
    for_each_phi<T, D, KB>(l, [&](int q, T ph) { sum += ph * es[q * nch + j]; });
    *reinterpret_cast<VT*>(v + (int64_t)i * nr + j * VW) = ow < 0 ? (VT)0 : sum;
  }
}

template <typename T>
void launch_prolong0(int n, int nbox, int d, int pc, int nr, const int* leaf_off, const int* owner, const T* xi,
                     const T* e, const T* epend, T* v, hipStream_t s) {
  const Basis1D<T> bs = make_basis<T>(pc);
  constexpr int VW = col_vw<T>();
  if (nr > 1 && nr % std::min(nr, VW) == 0 && aligned16(e) && (!epend || aligned16(epend)) && aligned16(v)) {
    const int vw = std::min(nr, VW), nch = nr / vw;
    const int k = pc + 1, B = (d == 3) ? k * k * k : k * k;
    if (nbox == 0) return;
    const size_t shm = (size_t)16 * B * nch;
    // workgroups per box: two entries a thread in an average box, as long as the chip is not full (a level of 64 boxes
    // on 64 compute units: 3D Q3 16^3, 16 float32 columns 29.8 -> 7.0 us)
    const int per = (int)std::max<int64_t>(1, std::min<int64_t>({((int64_t)n / nbox * nch + 511) / 512, 4096 / nbox, 64}));
#define R3MG_P0M(DD, KK)                                                                                           \
  do {                                                                                                             \
    if (vw == 2)                                                                                                   \
      hipLaunchKernelGGL((k_prolong0_mr<T, DD, KK, 2>), dim3(nbox * per), dim3(256), shm, s, bs, nr, per, leaf_off, owner, xi, \
                         e, epend, v);                                                                         \
    else                                                                                                           \
      hipLaunchKernelGGL((k_prolong0_mr<T, DD, KK, VW>), dim3(nbox * per), dim3(256), shm, s, bs, nr, per, leaf_off, owner, \
                         xi, e, epend, v);                                                                     \
  } while (0)
    switch (d * 8 + pc + 1) {
      case 17: R3MG_P0M(2, 1); break;
      case 18: R3MG_P0M(2, 2); break;
      case 19: R3MG_P0M(2, 3); break;
      case 20: R3MG_P0M(2, 4); break;
      case 25: R3MG_P0M(3, 1); break;
      case 26: R3MG_P0M(3, 2); break;
      case 27: R3MG_P0M(3, 3); break;
      case 28: R3MG_P0M(3, 4); break;
      default: throw std::runtime_error("prolongation: unsupported dimension or degree");
    }
#undef R3MG_P0M
    check_launch("k_prolong0_mr");
    return;
  }
  if (n == 0) return;
  // boxes of at least 192 points (three waves of a workgroup) take the box kernel, smaller ones a thread per point
  const bool boxed = nbox > 0 && (int64_t)n >= (int64_t)192 * nbox;
  const int per = boxed ? (int)((n / nbox + 255) / 256) : 1;
  const int nlog = boxed ? nbox * per : (n + 255) / 256;
#define R3MG_P0(DD, KK)                                                                                              \
  do {                                                                                                               \
    if (boxed)                                                                                                       \
      hipLaunchKernelGGL((k_prolong0_box<T, DD, KK>), dim3(xcd_grid(nlog)), dim3(256), 0, s, bs, nr, per, leaf_off,  \
                         owner, xi, e, epend, v, nlog);                                                        \
    else                                                                                                             \
      hipLaunchKernelGGL((k_prolong0<T, DD, KK>), dim3(xcd_grid(nlog)), dim3(256), 0, s, n, bs, nr, owner, xi, e,    \
                         epend, v, nlog);                                                                      \
  } while (0)
  switch (d * 8 + pc + 1) {
    case 17: R3MG_P0(2, 1); break;
    case 18: R3MG_P0(2, 2); break;
    case 19: R3MG_P0(2, 3); break;
    case 20: R3MG_P0(2, 4); break;
    case 25: R3MG_P0(3, 1); break;
    case 26: R3MG_P0(3, 2); break;
    case 27: R3MG_P0(3, 3); break;
    case 28: R3MG_P0(3, 4); break;
    default: throw std::runtime_error("prolongation: unsupported dimension or degree");
  }
#undef R3MG_P0
  check_launch("k_prolong0");
}
template void launch_prolong0<float>(int, int, int, int, int, const int*, const int*, const float*, const float*,
                                     const float*, float*, hipStream_t);
template void launch_prolong0<double>(int, int, int, int, int, const int*, const int*, const double*,
                                      const double*, const double*, double*, hipStream_t);

// P~ entry [q'][q] of child box c: prod_a M_c[a][q'_a][q_a]
template <typename T>
__device__ inline T pt_entry(const T* __restrict__ pt, int64_t c, int d, int k, int qc, int qp) {
  const T* m = pt + (int64_t)c * d * k * k;
  T v = m[(0 * k + qc % k) * k + qp % k];
  qc /= k;
  qp /= k;
  v *= m[(1 * k + qc % k) * k + qp % k];
  if (d == 3) {
    qc /= k;
    qp /= k;
    v *= m[(2 * k + qc % k) * k + qp % k];
  }
  return v;
}

// Tensor application of a child box's 1D factors m (D x KB x KB, m[x][child node][parent node]) to the KB^D values in
// `a`, by KB^D of the GL lanes of a group (GL divides 64, so the group is in one wave): axis by axis, through `b`.
// restriction (TR): r[q] = sum_a prod_x m[x][a_x][q_x] a[a]; prolongation: r[a] = sum_q prod_x m[x][a_x][q_x] a[q].
__device__ inline void wave_lds_sync() {
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <typename T, int D, int KB, bool TR>
__device__ inline T tensor_apply(T* a, T* b, const T* m, int q, bool active) {
  constexpr int KK = KB * KB;
  const int dg[3] = {q % KB, q / KB % KB, q / KK};
  const int st[3] = {1, KB, KK};
  T r = 0;
#pragma unroll
  for (int x = 0; x < D; ++x) {
    r = 0;
    if (active) {
      const T* in = (x & 1) ? b : a;
      const int base = q - dg[x] * st[x];
#pragma unroll
      for (int y = 0; y < KB; ++y)
        r += (TR ? m[x * KK + y * KB + dg[x]] : m[x * KK + dg[x] * KB + y]) * in[base + y * st[x]];
    }
    if (x + 1 < D) {
      wave_lds_sync();  // the input has been read
      if (active) ((x & 1) ? a : b)[q] = r;
      wave_lds_sync();
    }
  }
  return r;
}
template <int D, int KB>
struct BoxLanes {
  static constexpr int B = D == 3 ? KB * KB * KB : KB * KB;
  static constexpr int GL = B <= 1 ? 1 : pow2_at_least(B);  // lanes of a child box
  static constexpr int NG = 256 / GL;                       // child boxes of a workgroup at a time
  static constexpr int M = D * KB * KB;                     // 1D factors of a child box
};

// Restriction between agglomerated levels, one workgroup per parent box G: a group of lanes per child box C forms
// P~_C^T src_C axis by axis, and the children are added in order.  dnext = dinv_next b inv_theta_next when it is set.
// One lane per parent function used to sum over all children's B functions in turn, which in 3D is a chain of
// 216 products of four factors: 3D Q2 29^3 float64 (16 parents) 26.8 -> 3.8 us.
template <typename T, int D, int KB>
__global__ __launch_bounds__(256) void k_restrict_c(int nbox_next, int nbox, int shift, int nr,
                                                    const T* __restrict__ pt, const T* __restrict__ src, T* bnext,
                                                    const T* __restrict__ dinv_next, T* dnext, T inv_theta_next) {
  using BL = BoxLanes<D, KB>;
  constexpr int B = BL::B, GL = BL::GL, NG = BL::NG, M = BL::M;
  extern __shared__ unsigned char smem_raw[];
  __shared__ T sa[NG][B], sb[NG][B], sm[NG][M];
  T* part = reinterpret_cast<T*>(smem_raw);  // [children][B]
  const int G = blockIdx.x;
  const int g = threadIdx.x / GL, q = threadIdx.x % GL;
  const bool active = q < B;
  const int c0 = G << shift, nc = min(nbox, (G + 1) << shift) - c0;
  const int64_t t = (int64_t)G * B + min((int)threadIdx.x, B - 1);
  const T di = dnext ? dinv_next[t] : (T)0;
  for (int c = 0; c < nr; ++c) {
    for (int C = g; C < nc; C += NG) {
      wave_lds_sync();
      for (int u = q; u < M; u += GL) sm[g][u] = pt[(int64_t)(c0 + C) * M + u];
      if (active) sa[g][q] = src[((int64_t)(c0 + C) * B + q) * nr + c];
      wave_lds_sync();
      const T r = tensor_apply<T, D, KB, true>(sa[g], sb[g], sm[g], q, active);
      if (active) part[C * B + q] = r;
    }
    __syncthreads();
    if (threadIdx.x < B) {
      T v = 0;
      for (int C = 0; C < nc; ++C) v += part[C * B + threadIdx.x];
      bnext[t * nr + c] = v;
      if (dnext) dnext[t * nr + c] = di * v * inv_theta_next;
    }
    __syncthreads();
  }
}

// The same for nr > 1 columns: one workgroup per parent box G, thread (q, j) takes coarse function q and column
// chunk j.  The children's 1D injection factors are staged in LDS once, each child's B x nr entries (contiguous in
// src) one child at a time.
template <typename T, int VW>
__global__ __launch_bounds__(512) void k_restrict_c_mr(int nbox_next, int nbox, int shift, int d, int k, int nr,
                                                       const T* __restrict__ pt, const T* __restrict__ src, T* bnext,
                                                       const T* __restrict__ dinv_next, T* dnext, T inv_theta_next) {
  using VT = typename ColVec<T, VW>::type;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int B = (d == 3) ? k * k * k : k * k;
  const int kk = k * k;
  const int nch = nr / VW;
  VT* srcs = reinterpret_cast<VT*>(smem_raw);  // [B][nch] of the current child
  T* pts = reinterpret_cast<T*>(srcs + B * nch);
  const int G = blockIdx.x;
  const int c0 = G << shift;
  const int nc = min(nbox, (G + 1) << shift) - c0;
  for (int t = threadIdx.x; t < nc * d * kk; t += blockDim.x) pts[t] = pt[(int64_t)c0 * d * kk + t];
  const int q = threadIdx.x / nch, j = threadIdx.x - q * nch;
  const bool active = q < B;
  const int q0 = q % k, q1 = (q / k) % k, q2 = q / kk;
  VT acc = (VT)0;
  for (int C = 0; C < nc; ++C) {
    __syncthreads();
    const VT* sg = reinterpret_cast<const VT*>(src + (int64_t)(c0 + C) * B * nr);
    for (int t = threadIdx.x; t < B * nch; t += blockDim.x) srcs[t] = sg[t];
    __syncthreads();
    if (active) {
      const T* m = pts + C * d * kk;
      int qc = 0;
      for (int a2 = 0; a2 < (d == 3 ? k : 1); ++a2)
        for (int a1 = 0; a1 < k; ++a1)
          for (int a0 = 0; a0 < k; ++a0, ++qc) {
            T w = m[a0 * k + q0] * m[kk + a1 * k + q1];
            if (d == 3) w *= m[2 * kk + a2 * k + q2];
            acc += w * srcs[qc * nch + j];
          }
    }
  }
  if (active) {
    const int64_t row = (int64_t)G * B + q;
    *reinterpret_cast<VT*>(bnext + row * nr + j * VW) = acc;
    if (dnext) *reinterpret_cast<VT*>(dnext + row * nr + j * VW) = (dinv_next[row] * acc) * inv_theta_next;
  }
}

template <typename T>
void launch_restrict_c(int nbox_next, int nbox, int shift, int d, int pc, int nr, const T* pt, const T* src,
                       T* bnext, const T* dinv_next, T* dnext, double inv_theta_next,
                       hipStream_t s) {
  const int k = pc + 1;
  const int B = (d == 3) ? k * k * k : k * k;
  if (nbox_next == 0) return;
  if (B > 64) throw std::runtime_error("restriction: more than 64 coarse functions per box");
  constexpr int VW = col_vw<T>();
  if (nr > 1 && nr % std::min(nr, VW) == 0 && aligned16(src) && aligned16(bnext) && (!dnext || aligned16(dnext))) {
    const int vw = std::min(nr, VW), nch = nr / vw;
    const int thr = (B * nch + 63) / 64 * 64;
    if (thr > 512) throw std::runtime_error("restriction: too many columns");
    const size_t shmm = sizeof(T) * ((size_t)B * nr + (size_t)(1 << shift) * d * k * k);
    if (vw == 2)
      hipLaunchKernelGGL((k_restrict_c_mr<T, 2>), dim3(nbox_next), dim3(thr), shmm, s, nbox_next, nbox, shift, d, k, nr,
                         pt, src, bnext, dinv_next, dnext, (T)inv_theta_next);
    else
      hipLaunchKernelGGL((k_restrict_c_mr<T, VW>), dim3(nbox_next), dim3(thr), shmm, s, nbox_next, nbox, shift, d, k,
                         nr, pt, src, bnext, dinv_next, dnext, (T)inv_theta_next);
    check_launch("k_restrict_c_mr");
    return;
  }
  const size_t shm = sizeof(T) * ((size_t)B << shift);
  box_dispatch(d, k, [&](auto dk) {
    hipLaunchKernelGGL((k_restrict_c<T, dk.D, dk.K>), dim3((unsigned)nbox_next), dim3(256), shm, s, nbox_next, nbox, shift,
                       nr, pt, src, bnext, dinv_next, dnext, (T)inv_theta_next);
  });
  check_launch("k_restrict_c");
}
template void launch_restrict_c<float>(int, int, int, int, int, int, const float*, const float*, float*,
                                       const float*, float*, double, hipStream_t);
template void launch_restrict_c<double>(int, int, int, int, int, int, const double*, const double*, double*,
                                        const double*, double*, double, hipStream_t);

// Prolongation between agglomerated levels: v[C B + a] = sum_q P~_C[a][q] (e + epend)[G B + q], G = C >> shift the
// parent of child box C; a group of lanes per child box, axis by axis.
template <typename T, int D, int KB>
__global__ __launch_bounds__(256) void k_prolong_c(int nbox, int shift, int nr, const T* __restrict__ pt,
                                                   const T* __restrict__ e, const T* __restrict__ epend, T* v) {
  using BL = BoxLanes<D, KB>;
  constexpr int B = BL::B, GL = BL::GL, NG = BL::NG, M = BL::M;
  __shared__ T sa[NG][B], sb[NG][B], sm[NG][M];
  const int g = threadIdx.x / GL, q = threadIdx.x % GL;
  const int C = blockIdx.x * NG + g;
  const bool live = C < nbox, active = q < B && live;
  const int Cc = min(C, nbox - 1), G = Cc >> shift;
  for (int u = q; u < M; u += GL) sm[g][u] = pt[(int64_t)Cc * M + u];
  for (int c = 0; c < nr; ++c) {
    wave_lds_sync();
    if (active) {
      const int64_t o = ((int64_t)G * B + q) * nr + c;
      T ev = e[o];
      if (epend) ev += epend[o];
      sa[g][q] = ev;
    }
    wave_lds_sync();
    const T r = tensor_apply<T, D, KB, false>(sa[g], sb[g], sm[g], q, active);
    if (active) v[((int64_t)C * B + q) * nr + c] = r;
  }
}

// The same for nr > 1 columns: thread (C B + q', j) takes one fine entry and column chunk j.
template <typename T, int VW>
__global__ __launch_bounds__(256) void k_prolong_c_mr(int nbox, int shift, int d, int k, int nr,
                                                      const T* __restrict__ pt, const T* __restrict__ e,
                                                      const T* __restrict__ epend, T* v) {
  using VT = typename ColVec<T, VW>::type;
  const int B = (d == 3) ? k * k * k : k * k;
  const int nch = nr / VW;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)nbox * B * nch) return;
  const int64_t row = t / nch;
  const int j = (int)(t - row * nch);
  const int C = (int)(row / B), qc = (int)(row - (int64_t)C * B);
  const int G = C >> shift;
  VT sum = (VT)0;
  for (int q = 0; q < B; ++q) {
    const int64_t o = ((int64_t)G * B + q) * nr + j * VW;
    VT ev = *reinterpret_cast<const VT*>(e + o);
    if (epend) ev += *reinterpret_cast<const VT*>(epend + o);
    sum += pt_entry(pt, C, d, k, qc, q) * ev;
  }
  *reinterpret_cast<VT*>(v + row * nr + j * VW) = sum;
}

template <typename T>
void launch_prolong_c(int nbox, int shift, int d, int pc, int nr, const T* pt, const T* e, const T* epend, T* v,
                      hipStream_t s) {
  const int k = pc + 1;
  const int B = (d == 3) ? k * k * k : k * k;
  constexpr int VW = col_vw<T>();
  if (nr > 1 && nr % std::min(nr, VW) == 0 && aligned16(e) && (!epend || aligned16(epend)) && aligned16(v)) {
    const int vw = std::min(nr, VW);
    const int64_t totm = (int64_t)nbox * B * (nr / vw);
    if (totm == 0) return;
    if (vw == 2)
      hipLaunchKernelGGL((k_prolong_c_mr<T, 2>), dim3((unsigned)((totm + 255) / 256)), dim3(256), 0, s, nbox, shift, d,
                         k, nr, pt, e, epend, v);
    else
      hipLaunchKernelGGL((k_prolong_c_mr<T, VW>), dim3((unsigned)((totm + 255) / 256)), dim3(256), 0, s, nbox, shift,
                         d, k, nr, pt, e, epend, v);
    check_launch("k_prolong_c_mr");
    return;
  }
  if (nbox == 0) return;
  box_dispatch(d, k, [&](auto dk) {
    constexpr int NG = BoxLanes<dk.D, dk.K>::NG;
    hipLaunchKernelGGL((k_prolong_c<T, dk.D, dk.K>), dim3((unsigned)((nbox + NG - 1) / NG)), dim3(256), 0, s, nbox, shift,
                       nr, pt, e, epend, v);
  });
  check_launch("k_prolong_c");
}
template void launch_prolong_c<float>(int, int, int, int, int, const float*, const float*, const float*, float*,
                                      hipStream_t);
template void launch_prolong_c<double>(int, int, int, int, int, const double*, const double*, const double*,
                                       double*, hipStream_t);

// =============================================================================================
// Elementwise helpers
// =============================================================================================
template <typename T>
__global__ void k_xupdate(int64_t count, T* x, const T* __restrict__ v, int assign) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  x[i] = assign ? v[i] : x[i] + v[i];
}
template <typename T>
void launch_xupdate(int64_t count, T* x, const T* v, int assign, hipStream_t s) {
  if (count == 0) return;
  hipLaunchKernelGGL((k_xupdate<T>), dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, count, x, v, assign);
  check_launch("k_xupdate");
}
template void launch_xupdate<float>(int64_t, float*, const float*, int, hipStream_t);
template void launch_xupdate<double>(int64_t, double*, const double*, int, hipStream_t);

// V-cycle entry: b0[i] = r_user[perm[i]] (column c at r_user + c*ld), d0 = dinv * b0 * inv_theta
template <typename T>
__global__ void k_vc_entry(int n, int nr, const int* __restrict__ perm, const double* __restrict__ r, int64_t ld,
                           T* b0, const T* __restrict__ dinv, T* d0, T inv_theta) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)n * nr) return;
  const int i = (int)(t / nr), c = (int)(t - (int64_t)i * nr);
  const T v = (T)r[(int64_t)c * ld + perm[i]];
  b0[t] = v;
  if (d0) d0[t] = dinv[i] * v * inv_theta;
}
template <typename T>
void launch_vc_entry(int n, int nr, const int* perm, const double* r_user, int64_t ld_user, T* b0, const T* dinv,
                     T* d0, double inv_theta, hipStream_t s) {
  const int64_t tot = (int64_t)n * nr;
  hipLaunchKernelGGL((k_vc_entry<T>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, n, nr, perm, r_user, ld_user,
                     b0, dinv, d0, (T)inv_theta);
  check_launch("k_vc_entry");
}
template void launch_vc_entry<float>(int, int, const int*, const double*, int64_t, float*, const float*, float*,
                                     double, hipStream_t);
template void launch_vc_entry<double>(int, int, const int*, const double*, int64_t, double*, const double*,
                                      double*, double, hipStream_t);

template <typename T>
__global__ void k_vc_exit(int n, int nr, const int* __restrict__ perm, const T* __restrict__ x0,
                          const T* __restrict__ dp, double* z, int64_t ld) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)n * nr) return;
  const int i = (int)(t / nr), c = (int)(t - (int64_t)i * nr);
  T v = x0[t];
  if (dp) v += dp[t];
  z[(int64_t)c * ld + perm[i]] = (double)v;
}
template <typename T>
void launch_vc_exit(int n, int nr, const int* perm, const T* x0, const T* dpend, double* z_user, int64_t ld_user,
                    hipStream_t s) {
  const int64_t tot = (int64_t)n * nr;
  hipLaunchKernelGGL((k_vc_exit<T>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, n, nr, perm, x0, dpend,
                     z_user, ld_user);
  check_launch("k_vc_exit");
}
template void launch_vc_exit<float>(int, int, const int*, const float*, const float*, double*, int64_t, hipStream_t);
template void launch_vc_exit<double>(int, int, const int*, const double*, const double*, double*, int64_t,
                                     hipStream_t);

// Dense coarsest solve x = A_L^{-1} b with the float64 explicit inverse (one wave per row).
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_dense_apply(int nc, const double* __restrict__ cinv, const T* __restrict__ b,
                                                     T* x) {
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= nc) return;
  double acc[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) acc[k] = 0;
  const double* a = cinv + (int64_t)row * nc;
  int c = lane;
  for (; c + 192 < nc; c += 256) {  // four independent loads in flight per lane
    const double m0 = a[c], m1 = a[c + 64], m2 = a[c + 128], m3 = a[c + 192];
#pragma unroll
    for (int k = 0; k < NR; ++k)
      acc[k] += (m0 * (double)b[(int64_t)c * NR + k] + m1 * (double)b[(int64_t)(c + 64) * NR + k]) +
                (m2 * (double)b[(int64_t)(c + 128) * NR + k] + m3 * (double)b[(int64_t)(c + 192) * NR + k]);
  }
  for (; c < nc; c += 64) {
    const double m = a[c];
#pragma unroll
    for (int k = 0; k < NR; ++k) acc[k] += m * (double)b[(int64_t)c * NR + k];
  }
#pragma unroll
  for (int k = 0; k < NR; ++k) {
    acc[k] = wave_sum(acc[k], 64);
    if (lane == k) x[(int64_t)row * NR + k] = (T)acc[k];
  }
}
// The same for nr > 1 columns on the matrix cores: 16 rows and all columns per workgroup, the columns of the inverse dealt
// to 16 waves 16 at a time (lane (i, k) reads four consecutive entries of row i, the k groups of four instructions), and
// the waves' tiles added in wave order through LDS.  A lane of the kernel above holds whole columns of the inverse and
// reads all nr entries of b for each, then does a butterfly per column.  Four steps of a wave are loaded at once.
// Bound by the inverse (24 MB at 1,728 unknowns) and its round trips.  16 float32 columns 21.5 -> 13.7 us (18.9 with two
// steps at once).  Fewer than four unknowns (the last four of a row are read as one vector) keep the kernel above.
template <typename T, int NR>
__global__ __launch_bounds__(1024) void k_dense_apply_mr(int nc, const double* __restrict__ cinv,
                                                         const T* __restrict__ b, T* x) {
  using M = Mfma16<double>;
  constexpr int NW = 16, UN = 4;
  typedef double V4 __attribute__((ext_vector_type(4), aligned(8)));
  __shared__ double red[NW][256];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = lane & 15, kk = lane >> 4;
  const int row0 = blockIdx.x * 16;
  const double* a = cinv + (int64_t)min(row0 + i, nc - 1) * nc;
  M::acc acc = {0.0, 0.0, 0.0, 0.0};
  for (int k0 = 16 * w; k0 < nc; k0 += 16 * NW * UN) {
    V4 av[UN];
    T bv[UN][4];
#pragma unroll
    for (int m = 0; m < UN; ++m) {  // the last four entries where a lane's own pass the end (nc >= 4)
      const int k = min(k0 + 16 * NW * m + 4 * kk, nc - 4);
      av[m] = *reinterpret_cast<const V4*>(a + k);
#pragma unroll
      for (int q = 0; q < 4; ++q) bv[m][q] = b[(int64_t)(k + q) * NR + i % NR];
    }
#pragma unroll
    for (int m = 0; m < UN; ++m) {
      const int k1 = k0 + 16 * NW * m + 4 * kk, k = min(k1, nc - 4);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const bool own = k + q >= k1;  // each entry once, and neither operand otherwise: 0 * inf would be NaN
        acc = M::mma(own ? av[m][q] : 0.0, own ? (double)bv[m][q] : 0.0, acc);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) red[w][M::row(lane, r) * 16 + i] = acc[r];
  __syncthreads();
  if (threadIdx.x < 256) {
    const int r = row0 + (int)threadIdx.x / 16, c = threadIdx.x % 16;
    double t = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) t += red[v][threadIdx.x];
    if (r < nc && c < NR) x[(int64_t)r * NR + c] = (T)t;
  }
}
template <typename T>
void launch_dense_apply(int nc, int nr, const double* cinv, const T* b, T* x, hipStream_t s) {
#define R3_DAP(NRV)                                                                                              \
  case NRV:                                                                                                      \
    if (NRV == 1 || nc < 4)                                                                                      \
      hipLaunchKernelGGL((k_dense_apply<T, NRV>), dim3((nc + 3) / 4), dim3(256), 0, s, nc, cinv, b, x);    \
    else                                                                                                         \
      hipLaunchKernelGGL((k_dense_apply_mr<T, NRV>), dim3((nc + 15) / 16), dim3(1024), 0, s, nc, cinv, b, x); \
    break;
  switch (nr) {
    R3_DAP(1)
    R3_DAP(2)
    R3_DAP(4)
    R3_DAP(8)
    R3_DAP(16)
    default: throw std::runtime_error("unsupported nrhs block");
  }
#undef R3_DAP
  check_launch("k_dense_apply");
}
template void launch_dense_apply<float>(int, int, const double*, const float*, float*, hipStream_t);
template void launch_dense_apply<double>(int, int, const double*, const double*, double*, hipStream_t);

// Symmetric dense coarsest product.  Pass 1: one workgroup per upper tile (I, J); wave w holds the tile's rows
// 16 w .. 16 w + 15 in registers (stored as M = float64, or float32 for the float32 V-cycle, and widened to
// float64 where used: the products and partial sums are float64 either way), lane = column.  The row products
// are summed over the 64 lanes by a transposing butterfly (each step halves the rows a lane keeps and doubles
// the columns summed), which leaves lane l with row 8 b5 + 4 b4 + 2 b3 + b2 of its wave (b = bits of l).  The
// transposed products of an off-diagonal tile take the wave's 16 rows of b from LDS and are summed over the four
// waves in order.
template <typename T, typename M, int NR>
__global__ __launch_bounds__(256) void k_dense_sym_tiles(int nc, int nt, const M* __restrict__ packed,
                                                         const int2* __restrict__ tiles, const T* __restrict__ b,
                                                         double* part) {
  __shared__ double sh[4][64];
  __shared__ T sbr[4][16 * NR];  // wave w's 16 rows of b (0 past the last row), read at use (fewer registers)
  const int t = blockIdx.x;
  const int2 ij = tiles[t];
  const int I = ij.x, J = ij.y;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const M* a = packed + (int64_t)t * (kDenseTile * kDenseTile) + (16 * w) * kDenseTile + lane;
  M m[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) m[k] = a[k * kDenseTile];
  const int cj = J * kDenseTile + lane;
  const int ri = I * kDenseTile + 16 * w;
  // the entries of b are loaded up front from clamped addresses and masked (loads under a lane-dependent
  // condition would each be waited for)
  T bj[NR];
#pragma unroll
  for (int c = 0; c < NR; ++c) bj[c] = b[(int64_t)min(cj, nc - 1) * NR + c];
  if (I != J) {  // uniform over the workgroup
    if (lane < 16) {
      const T* bp = b + (int64_t)min(ri + lane, nc - 1) * NR;
#pragma unroll
      for (int c = 0; c < NR; ++c) sbr[w][lane * NR + c] = ri + lane < nc ? bp[c] : (T)0;
    }
    __syncthreads();
  }
  const bool b5 = lane & 32, b4 = lane & 16, b3 = lane & 8, b2 = lane & 4;
  const int myrow = (b5 ? 8 : 0) + (b4 ? 4 : 0) + (b3 ? 2 : 0) + (b2 ? 1 : 0);
  for (int c = 0; c < NR; ++c) {
    const double xj = cj < nc ? (double)bj[c] : 0.0;
    double h8[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double lo = (double)m[q] * xj, hi = (double)m[8 + q] * xj;
      h8[q] = (b5 ? hi : lo) + __shfl_xor(b5 ? lo : hi, 32, 64);
    }
    double h4[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) h4[q] = (b4 ? h8[4 + q] : h8[q]) + __shfl_xor(b4 ? h8[q] : h8[4 + q], 16, 64);
    double h2[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) h2[q] = (b3 ? h4[2 + q] : h4[q]) + __shfl_xor(b3 ? h4[q] : h4[2 + q], 8, 64);
    double h1 = (b2 ? h2[1] : h2[0]) + __shfl_xor(b2 ? h2[0] : h2[1], 4, 64);
    h1 += __shfl_xor(h1, 2, 64);
    h1 += __shfl_xor(h1, 1, 64);
    if ((lane & 3) == 0)
      part[(((int64_t)I * nt + J) * kDenseTile + 16 * w + myrow) * NR + c] = h1;
    if (I != J) {  // uniform over the workgroup
      double cs = 0;
#pragma unroll
      for (int k = 0; k < 16; ++k) cs += (double)m[k] * (double)sbr[w][k * NR + c];
      sh[w][lane] = cs;
      __syncthreads();
      if (w == 0)
        part[(((int64_t)J * nt + I) * kDenseTile + lane) * NR + c] = (sh[0][lane] + sh[1][lane]) +
                                                                      (sh[2][lane] + sh[3][lane]);
      __syncthreads();
    }
  }
}

// Pass 2: the sum of row `row`'s nt slots, as taken by thread (g, i) of a 16 x 16 group (g = slot group, i =
// row): slot S is taken by group S % 16 in index order, the group sums go to sh[g][i], and sum16 adds the 16 groups
// in order.
__device__ inline double dense_slot_sum(int nt, const double* __restrict__ part, int row, int g, int nr, int c) {
  const int R = row / kDenseTile, i = row - R * kDenseTile;
  double acc = 0;
#pragma unroll 4
  for (int S = g; S < nt; S += 16) acc += part[(((int64_t)R * nt + S) * kDenseTile + i) * nr + c];
  return acc;
}
__device__ inline double dense_sum16(const double (*sh)[17], int i) {
  double t = 0;
#pragma unroll
  for (int k = 0; k < 16; ++k) t += sh[k][i];
  return t;
}

// Pass 2 alone: rows 16 Q .. 16 Q + 15 of row block R = blockIdx.x / 4 (Q = blockIdx.x % 4).
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_dense_sym_reduce(int nc, int nt, const double* __restrict__ part, T* x) {
  __shared__ double sh[16][17];
  const int R = blockIdx.x >> 2, i = 16 * (blockIdx.x & 3) + (threadIdx.x & 15), g = threadIdx.x >> 4;
  const int row = R * kDenseTile + i;
  for (int c = 0; c < NR; ++c) {
    sh[g][threadIdx.x & 15] = dense_slot_sum(nt, part, row, g, NR, c);
    __syncthreads();
    if (g == 0 && row < nc) x[(int64_t)row * NR + c] = (T)dense_sum16(sh, threadIdx.x & 15);
    __syncthreads();
  }
}

// Pass 2 fused with the prolongation to the level above (k_prolong_c with no pending direction): one workgroup
// per parent box G of that level (= box G of the coarsest level, B rows).  Its B rows of x are summed from the
// slots as in k_dense_sym_reduce (16 rows at a time), stored, and kept in LDS; then a group of lanes per child box C of
// G forms v[C B + a] = sum_q P~_C[a][q] x[G B + q] axis by axis, as k_prolong_c does.  The factors of the first
// children are fetched before the sums.  3D Q2 29^3 float64: 10.0 -> 3.8 us.
template <typename T, int D, int KB, int NR>
__global__ __launch_bounds__(256) void k_dense_sym_reduce_prolong(int nbox, int shift, int nt,
                                                                  const double* __restrict__ part, T* x,
                                                                  const T* __restrict__ pt, T* v) {
  using BL = BoxLanes<D, KB>;
  constexpr int B = BL::B, GL = BL::GL, NG = BL::NG, M = BL::M;
  __shared__ double sh[16][17];
  __shared__ T xs[B * NR];
  __shared__ T sa[NG][B], sb[NG][B], sm[NG][M];
  const int G = blockIdx.x;
  const int cg = threadIdx.x / GL, q = threadIdx.x % GL;
  const int c0 = G << shift, nch = min(nbox, (G + 1) << shift) - c0;
  for (int u = q; u < M; u += GL) sm[cg][u] = pt[(int64_t)(c0 + min(cg, nch - 1)) * M + u];
  const int g = threadIdx.x >> 4, i = threadIdx.x & 15;
  for (int r0 = 0; r0 < B; r0 += 16) {
    const int r = r0 + i;
    for (int c = 0; c < NR; ++c) {
      if (r < B) sh[g][i] = dense_slot_sum(nt, part, G * B + r, g, NR, c);
      __syncthreads();
      if (g == 0 && r < B) {
        const T t = (T)dense_sum16(sh, i);
        x[((int64_t)G * B + r) * NR + c] = t;
        xs[r * NR + c] = t;
      }
      __syncthreads();
    }
  }
  for (int C = cg; C < nch; C += NG) {
    if (C != cg) {
      wave_lds_sync();
      for (int u = q; u < M; u += GL) sm[cg][u] = pt[(int64_t)(c0 + C) * M + u];
    }
    for (int c = 0; c < NR; ++c) {
      wave_lds_sync();
      if (q < B) sa[cg][q] = xs[q * NR + c];
      wave_lds_sync();
      const T r = tensor_apply<T, D, KB, false>(sa[cg], sb[cg], sm[cg], q, q < B);
      if (q < B) v[((int64_t)(c0 + C) * B + q) * NR + c] = r;
    }
  }
}

template <typename M>
__global__ __launch_bounds__(256) void k_dense_pack_sym(int nc, const double* __restrict__ full,
                                                        const int2* __restrict__ tiles, M* packed) {
  const int t = blockIdx.x;
  const int2 ij = tiles[t];
  for (int e = threadIdx.x; e < kDenseTile * kDenseTile; e += 256) {
    const int i = ij.x * kDenseTile + e / kDenseTile, j = ij.y * kDenseTile + e % kDenseTile;
    packed[(int64_t)t * (kDenseTile * kDenseTile) + e] = (i < nc && j < nc) ? (M)full[(int64_t)i * nc + j] : (M)0;
  }
}
template <typename M>
void launch_dense_pack_sym(int nc, int ntiles, const double* full, const int* tiles, M* packed, hipStream_t s) {
  hipLaunchKernelGGL((k_dense_pack_sym<M>), dim3(ntiles), dim3(256), 0, s, nc, full,
                     reinterpret_cast<const int2*>(tiles), packed);
  check_launch("k_dense_pack_sym");
}
template void launch_dense_pack_sym<double>(int, int, const double*, const int*, double*, hipStream_t);
template void launch_dense_pack_sym<float>(int, int, const double*, const int*, float*, hipStream_t);

template <typename T, typename M>
void launch_dense_apply_sym(int nc, int nt, int nr, const M* packed, const int* tiles, double* part, const T* b,
                            T* x, const DenseProlong<T>* pr, hipStream_t s) {
  const int ntiles = nt * (nt + 1) / 2;
  const int2* tl = reinterpret_cast<const int2*>(tiles);
  int B = 0;
  if (pr) {
    B = pr->d == 3 ? (pr->pc + 1) * (pr->pc + 1) * (pr->pc + 1) : (pr->pc + 1) * (pr->pc + 1);
    if (B > 64 || (int64_t)B * pr->nbox_coarse != nc)
      throw std::runtime_error("dense coarsest product: prolongation boxes do not match the coarsest level");
  }
  switch (nr) {
#define R3_DS(NRV)                                                                                                  \
  hipLaunchKernelGGL((k_dense_sym_tiles<T, M, NRV>), dim3(ntiles), dim3(256), 0, s, nc, nt, packed, tl, b, part);  \
  if (pr)                                                                                                           \
    box_dispatch(pr->d, pr->pc + 1, [&](auto dk) {                                                                   \
      hipLaunchKernelGGL((k_dense_sym_reduce_prolong<T, dk.D, dk.K, NRV>), dim3(pr->nbox_coarse), dim3(256), 0, s,   \
                         pr->nbox, pr->shift, nt, part, x, pr->pt, pr->v);                                     \
    });                                                                                                              \
  else                                                                                                              \
    hipLaunchKernelGGL((k_dense_sym_reduce<T, NRV>), dim3(4 * nt), dim3(256), 0, s, nc, nt, part, x);        \
  break;
    case 1: R3_DS(1)
    case 2: R3_DS(2)
    case 4: R3_DS(4)
#undef R3_DS
    default: throw std::runtime_error("symmetric dense coarsest product: unsupported nrhs block");
  }
  check_launch("k_dense_sym");
}
template void launch_dense_apply_sym<float, float>(int, int, int, const float*, const int*, double*, const float*,
                                                   float*, const DenseProlong<float>*, hipStream_t);
template void launch_dense_apply_sym<float, double>(int, int, int, const double*, const int*, double*,
                                                    const float*, float*, const DenseProlong<float>*,
                                                    hipStream_t);
template void launch_dense_apply_sym<double, double>(int, int, int, const double*, const int*, double*,
                                                     const double*, double*, const DenseProlong<double>*, hipStream_t);

__global__ void k_gather_cols(int n, int nr, int nuser, const int* __restrict__ perm,
                              const double* __restrict__ user, int64_t ld, double* out) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)n * nr) return;
  const int i = (int)(t / nr), c = (int)(t - (int64_t)i * nr);
  out[t] = c < nuser ? user[(int64_t)c * ld + perm[i]] : 0.0;
}
void launch_gather_cols(int n, int nr, int nuser, const int* perm, const double* user, int64_t ld_user,
                        double* out, hipStream_t s) {
  const int64_t tot = (int64_t)n * nr;
  hipLaunchKernelGGL(k_gather_cols, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, n, nr, nuser, perm, user,
                     ld_user, out);
  check_launch("k_gather_cols");
}
__global__ void k_scatter_cols(int n, int nr, int nuser, const int* __restrict__ perm,
                               const double* __restrict__ in, double* user, int64_t ld) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)n * nr) return;
  const int i = (int)(t / nr), c = (int)(t - (int64_t)i * nr);
  if (c < nuser) user[(int64_t)c * ld + perm[i]] = in[t];
}
void launch_scatter_cols(int n, int nr, int nuser, const int* perm, const double* in, double* user,
                         int64_t ld_user, hipStream_t s) {
  const int64_t tot = (int64_t)n * nr;
  hipLaunchKernelGGL(k_scatter_cols, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, n, nr, nuser, perm, in,
                     user, ld_user);
  check_launch("k_scatter_cols");
}

__global__ void k_cast_d2f(int64_t count, const double* __restrict__ a, float* b) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < count; i += (int64_t)gridDim.x * 256) b[i] = (float)a[i];
}
void launch_cast_d2f(int64_t count, const double* a, float* b, hipStream_t s) {
  if (count == 0) return;
  int64_t g = (count + 255) / 256;
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(k_cast_d2f, dim3((unsigned)g), dim3(256), 0, s, count, a, b);
  check_launch("k_cast_d2f");
}

__global__ void k_gather_vals(int64_t nnz, const int64_t* __restrict__ src, const double* __restrict__ uv,
                              double* out) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nnz; i += (int64_t)gridDim.x * 256) out[i] = uv[src[i]];
}
void launch_gather_vals(int64_t nnz, const int64_t* src, const double* user_vals, double* out, hipStream_t s) {
  if (nnz == 0) return;
  int64_t g = (nnz + 255) / 256;
  if (g > 65536) g = 65536;
  hipLaunchKernelGGL(k_gather_vals, dim3((unsigned)g), dim3(256), 0, s, nnz, src, user_vals, out);
  check_launch("k_gather_vals");
}

// =============================================================================================
// Set-up kernels
// =============================================================================================
// inverse diagonal of a level operator; *bad = 1 if any diagonal entry is not > 0
__global__ void k_diag_inv(int n, int blk, const int* __restrict__ ptr, const int* __restrict__ idx,
                           const double* __restrict__ val, double* dinv, double* diag, int* bad) {
  const int row = blockIdx.x * 256 + threadIdx.x;
  if (row >= n) return;
  double dv = 0.0;
  if (blk == 1) {
    int lo = ptr[row], hi = ptr[row + 1];
    while (lo < hi) {  // lower bound of `row`
      int mid = (lo + hi) >> 1;
      if (idx[mid] < row) lo = mid + 1; else hi = mid;
    }
    if (lo < ptr[row + 1] && idx[lo] == row) dv = val[lo];
  } else {
    const int K = row / blk, q = row - K * blk;
    const int j0 = ptr[K], nb = ptr[K + 1] - j0;
    int lo = j0, hi = j0 + nb;
    while (lo < hi) {
      int mid = (lo + hi) >> 1;
      if (idx[mid] < K) lo = mid + 1; else hi = mid;
    }
    if (lo < j0 + nb && idx[lo] == K)
      dv = val[(int64_t)blk * blk * j0 + (int64_t)q * nb * blk + (int64_t)(lo - j0) * blk + q];
  }
  if (diag) diag[row] = dv;
  if (!(dv > 0.0)) {
    *bad = 1;
    dinv[row] = 0.0;
  } else {
    dinv[row] = 1.0 / dv;
  }
}
void launch_diag_inv(int n, int blk, const int* ptr, const int* idx, const double* val, double* dinv, double* diag,
                     int* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_diag_inv, dim3((n + 255) / 256), dim3(256), 0, s, n, blk, ptr, idx, val, dinv, diag, bad);
  check_launch("k_diag_inv");
}

// Galerkin product, fine -> first agglomerated level (Section 4, inherited operators):
// A1[K,K'] = sum_{i in K free} phi^K(x_i) T_i^T,  T_i[q'] = sum_{j in K' free} A_ij phi^K'_q'(x_j).
// The host lists, per stored output block, the rows i of K whose sorted columns meet box K' with the column run
// [s, e).  A 256-thread workgroup takes one work item: a piece of one block's list.  Eight 32-lane groups take eight
// entries at a time: group g evaluates phi^K(x_i) and T_i into LDS; then every thread adds sum_g phi_g[q] T_g[q'] to
// the entries (q, q') it owns.  For T_i the group's 32 lanes take 32 entries of the run at a time: each loads its
// entry's column, value, owner and coordinates (all 32 chains in flight together) and puts A_ij l_0 and the products
// l_1 l_2 of x_j's 1D tables into LDS; then lane q' adds the products of those entries in the run's order.  A1 is
// symmetric, so only the blocks with K <= K' are formed and each off-diagonal one is also stored transposed as its
// mirror (K', K).  The summation order is fixed (deterministic): a block of several items is the sum of their partial
// blocks in list order (k_galerkin0_sum).
// Bound by LDS reads and latency.  A diagonal block lists nearly every row of its box (about 1,840), the others a few
// dozen, so with one workgroup per block a level of 64 boxes kept 64 of 256 compute units busy; and the T loop read
// five LDS words per product, now two.  3D Q2 24^3 (117,649 rows, 64 boxes, p' = 2): 3,061 -> 183 us.
constexpr int kGalTabs(int d, int k) { return d == 3 ? k + k * k : 2 * k; }
template <int D, int KB>
__global__ __launch_bounds__(256) void k_galerkin0(Basis1D<double> bs, const int4* __restrict__ item,
                                                   const int* __restrict__ up, const int* __restrict__ mir,
                                                   const int* __restrict__ brow, const int* __restrict__ bptr,
                                                   const int* __restrict__ gal_ent, const int* __restrict__ owner,
                                                   const double* __restrict__ xi, const int* __restrict__ col,
                                                   const double* __restrict__ val, double* part, double* out) {
  // dimension and degree are compile-time (lag1d_k and the digit arithmetic below unroll)
  constexpr int d = D, k = KB;
  constexpr int B = D == 3 ? KB * KB * KB : KB * KB;
  constexpr int EMAX = (B * B + 255) / 256;
  constexpr int TAB = kGalTabs(D, KB);
  constexpr int QMAX = (B + 31) / 32;
  __shared__ double spi[8][64];
  __shared__ double sT[8][64];
  // per group: of 32 entries j the values A_ij l_0[.] (0 for a constrained column) and the products l_1[.] l_2[.]
  __shared__ double sl[8][32][TAB];
  const int4 it = item[blockIdx.x];  // block up[it.x], its entries [it.y, it.z), partial slot it.w (-1: the whole block)
  const int64_t blkid = up[it.x];
  int qi[EMAX], qj[EMAX];
  double acc[EMAX];
#pragma unroll
  for (int m = 0; m < EMAX; ++m) {
    const int e = threadIdx.x + m * 256;
    qi[m] = e < B * B ? e / B : -1;
    qj[m] = e < B * B ? e % B : 0;
    acc[m] = 0;
  }
  const int g = threadIdx.x >> 5, lt = threadIdx.x & 31;
  const int en0 = it.y, en1 = it.z;
  for (int base = en0; base < en1; base += 8) {
    const int ent = base + g;
    if (ent < en1) {
      const int i = gal_ent[3 * ent], s = gal_ent[3 * ent + 1], e = gal_ent[3 * ent + 2];
      double li[3][4];
#pragma unroll
      for (int a = 0; a < d; ++a) lag1d_k<double, KB>(bs, xi[(int64_t)i * d + a], li[a]);
      for (int q = lt; q < B; q += 32) spi[g][q] = phi_q<double>(li, d, k, q);
      // lane lt owns q' = lt and lt + 32 (B <= 64); the digits of q' in base k pick the tables
      int q0[QMAX], q12[QMAX];
      double t[QMAX];
#pragma unroll
      for (int m = 0; m < QMAX; ++m) {
        const int q = min(lt + 32 * m, B - 1);
        q0[m] = q % k;
        q12[m] = k + q / k;
        t[m] = 0.0;
      }
      for (int p0 = s; p0 < e; p0 += 32) {
        const int p = min(p0 + lt, e - 1);  // clamped: every lane loads, the lanes past the run store nothing
        const int j = col[p];
        const double v = val[p];
        const int own = owner[j];
        double lj[3][4] = {};
#pragma unroll
        for (int a = 0; a < d; ++a) lag1d_k<double, KB>(bs, xi[(int64_t)j * d + a], lj[a]);
        if (p0 + lt < e) {
#pragma unroll
          for (int a = 0; a < k; ++a) sl[g][lt][a] = own >= 0 ? v * lj[0][a] : 0.0;
#pragma unroll
          for (int c = 0; c < (D == 3 ? KB : 1); ++c)
#pragma unroll
            for (int a = 0; a < k; ++a)
              sl[g][lt][k + c * k + a] = own < 0 ? 0.0 : D == 3 ? lj[1][a] * lj[2][c] : lj[1][a];
        }
        // the group is half a wave: its LDS writes and reads stay in program order within the wave
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const int cnt = min(32, e - p0);
        const double* L = &sl[g][0][0];
#pragma unroll 4
        for (int u = 0; u < cnt; ++u, L += TAB)
#pragma unroll
          for (int m = 0; m < QMAX; ++m) t[m] += L[q0[m]] * L[q12[m]];
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
#pragma unroll
      for (int m = 0; m < QMAX; ++m)
        if (lt + 32 * m < B) sT[g][lt + 32 * m] = t[m];
    } else {
      for (int q = lt; q < B; q += 32) {
        spi[g][q] = 0.0;
        sT[g][q] = 0.0;
      }
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < EMAX; ++m) {
      if (qi[m] >= 0) {
        double sacc = 0;
#pragma unroll
        for (int gg = 0; gg < 8; ++gg) sacc += spi[gg][qi[m]] * sT[gg][qj[m]];
        acc[m] += sacc;
      }
    }
    __syncthreads();
  }
  if (it.w >= 0) {
#pragma unroll
    for (int m = 0; m < EMAX; ++m)
      if (qi[m] >= 0) part[(int64_t)it.w * B * B + threadIdx.x + m * 256] = acc[m];
    return;
  }
  const int K = brow[blkid];
  const int slot = (int)(blkid - bptr[K]);
  const int nbK = bptr[K + 1] - bptr[K];
  const int64_t obase = (int64_t)B * B * bptr[K];
#pragma unroll
  for (int m = 0; m < EMAX; ++m)
    if (qi[m] >= 0) out[obase + (int64_t)qi[m] * nbK * B + (int64_t)slot * B + qj[m]] = acc[m];
  const int mb = mir[it.x];
  if (mb >= 0) {  // uniform over the workgroup
    const int Km = brow[mb], slm = mb - bptr[Km], nbm = bptr[Km + 1] - bptr[Km];
    const int64_t mbase = (int64_t)B * B * bptr[Km];
#pragma unroll
    for (int m = 0; m < EMAX; ++m)
      if (qi[m] >= 0) out[mbase + (int64_t)qj[m] * nbm * B + (int64_t)slm * B + qi[m]] = acc[m];
  }
}

// the blocks of several items: multi[t] = (index into up, first partial slot, number of partials)
__global__ __launch_bounds__(256) void k_galerkin0_sum(int B, const int4* __restrict__ multi, const int* __restrict__ up,
                                                       const int* __restrict__ mir, const int* __restrict__ brow,
                                                       const int* __restrict__ bptr, const double* __restrict__ part,
                                                       double* out) {
  const int4 w = multi[blockIdx.x];
  const int blkid = up[w.x], mb = mir[w.x];
  const int K = brow[blkid], slot = blkid - bptr[K], nbK = bptr[K + 1] - bptr[K];
  const int64_t obase = (int64_t)B * B * bptr[K];
  for (int e = threadIdx.x; e < B * B; e += 256) {
    const double* P = part + (int64_t)w.y * B * B + e;
    double t = 0;
#pragma unroll 4
    for (int c = 0; c < w.z; ++c) t += P[(int64_t)c * B * B];
    const int q = e / B, q2 = e - q * B;
    out[obase + (int64_t)q * nbK * B + (int64_t)slot * B + q2] = t;
    if (mb >= 0) {
      const int Km = brow[mb], slm = mb - bptr[Km], nbm = bptr[Km + 1] - bptr[Km];
      out[(int64_t)B * B * bptr[Km] + (int64_t)q2 * nbm * B + (int64_t)slm * B + q] = t;
    }
  }
}

void launch_galerkin0(const GalerkinWork& w, int d, int pc, const int* up, const int* mir, const int* brow,
                      const int* bptr, const int* gal_ent, const int* owner, const double* xi, const int* col,
                      const double* val, double* out, hipStream_t s) {
  Basis1D<double> bs = make_basis<double>(pc);
  if (w.nitem == 0) return;
  const int4* item = reinterpret_cast<const int4*>(w.item);
#define R3MG_G0(DD, KK)                                                                                              \
  hipLaunchKernelGGL((k_galerkin0<DD, KK>), dim3((unsigned)w.nitem), dim3(256), 0, s, bs, item, up, mir, brow, bptr, \
                     gal_ent, owner, xi, col, val, w.part, out)
  switch (d * 8 + pc + 1) {
    case 17: R3MG_G0(2, 1); break;
    case 18: R3MG_G0(2, 2); break;
    case 19: R3MG_G0(2, 3); break;
    case 20: R3MG_G0(2, 4); break;
    case 25: R3MG_G0(3, 1); break;
    case 26: R3MG_G0(3, 2); break;
    case 27: R3MG_G0(3, 3); break;
    case 28: R3MG_G0(3, 4); break;
    default: throw std::runtime_error("Galerkin product: unsupported dimension or degree");
  }
#undef R3MG_G0
  if (w.nmulti > 0) {
    const int k = pc + 1, B = d == 3 ? k * k * k : k * k;
    hipLaunchKernelGGL(k_galerkin0_sum, dim3((unsigned)w.nmulti), dim3(256), 0, s, B,
                       reinterpret_cast<const int4*>(w.multi), up, mir, brow, bptr, w.part, out);
  }
  check_launch("k_galerkin0");
}

// Galerkin product between agglomerated levels: A_{l+1}[G,G'] = sum_{C in G, C' in G'} P~_C^T A_l[C,C'] P~_C'.
// One workgroup per output block; A_l blocks and P~ blocks are staged in LDS (dynamic, 4 B^2 doubles).
template <int D, int KB>
__global__ __launch_bounds__(256) void k_galerkin_c(int shift, int nbox_in, const int* __restrict__ brow,
                                                    const int* __restrict__ bptr_out, const int* __restrict__ bcol_out,
                                                    const int* __restrict__ bptr_in, const int* __restrict__ bcol_in,
                                                    const double* __restrict__ val_in, const double* __restrict__ pt,
                                                    double* out) {
  extern __shared__ unsigned char smem_raw[];
  // dimension and degree are compile-time: the B-long loops and the index divisions below unroll or fold, with the
  // same operations in the same order
  constexpr int d = D, k = KB;
  constexpr int B = D == 3 ? KB * KB * KB : KB * KB;
  constexpr int bb = B * B;
  constexpr int EMAX = (bb + 255) / 256;
  double* sA = reinterpret_cast<double*>(smem_raw);
  double* sPc = sA + bb;
  double* sPp = sPc + bb;
  double* sT = sPp + bb;
  const int64_t blkid = blockIdx.x;
  const int G = brow[blkid];
  const int slot = (int)(blkid - bptr_out[G]);
  const int nbG = bptr_out[G + 1] - bptr_out[G];
  const int Gp = bcol_out[blkid];
  double acc[EMAX];
#pragma unroll
  for (int m = 0; m < EMAX; ++m) acc[m] = 0;
  const int c0 = G << shift, c1 = min(nbox_in, (G + 1) << shift);
  const int tlo = Gp << shift, thi = (Gp + 1) << shift;
  for (int C = c0; C < c1; ++C) {
    for (int e = threadIdx.x; e < bb; e += blockDim.x) sPc[e] = pt_entry(pt, C, d, k, e / B, e % B);
    const int j0 = bptr_in[C], nbC = bptr_in[C + 1] - j0;
    int lo = j0, hi = j0 + nbC;
    while (lo < hi) {
      int mid = (lo + hi) >> 1;
      if (bcol_in[mid] < tlo) lo = mid + 1; else hi = mid;
    }
    for (int jb = lo; jb < j0 + nbC && bcol_in[jb] < thi; ++jb) {
      const int Cp = bcol_in[jb];
      const int64_t vb = (int64_t)bb * j0 + (int64_t)(jb - j0) * B;
      __syncthreads();
      for (int e = threadIdx.x; e < bb; e += blockDim.x) {
        const int r = e / B, c = e % B;
        sA[e] = val_in[vb + (int64_t)r * nbC * B + c];
        sPp[e] = pt_entry(pt, Cp, d, k, r, c);
      }
      __syncthreads();
      for (int e = threadIdx.x; e < bb; e += blockDim.x) {  // T = A P~_C'
        const int r = e / B, c = e % B;
        double s = 0;
        for (int m = 0; m < B; ++m) s += sA[r * B + m] * sPp[m * B + c];
        sT[e] = s;
      }
      __syncthreads();
#pragma unroll
      for (int m = 0; m < EMAX; ++m) {  // acc += P~_C^T T
        const int e = threadIdx.x + m * blockDim.x;
        if (e < bb) {
          const int q = e / B, qq = e % B;
          double s = 0;
          for (int r = 0; r < B; ++r) s += sPc[r * B + q] * sT[r * B + qq];
          acc[m] += s;
        }
      }
    }
    __syncthreads();
  }
  const int64_t base = (int64_t)bb * bptr_out[G];
#pragma unroll
  for (int m = 0; m < EMAX; ++m) {
    const int e = threadIdx.x + m * blockDim.x;
    if (e < bb) out[base + (int64_t)(e / B) * nbG * B + (int64_t)slot * B + (e % B)] = acc[m];
  }
}

void launch_galerkin_c(int64_t nblocks, int d, int pc, int shift, int nbox_in, const int* brow, const int* bptr_out,
                       const int* bcol_out, const int* bptr_in, const int* bcol_in, const double* val_in,
                       const double* pt, double* out, hipStream_t s) {
  const int k = pc + 1;
  const int B = (d == 3) ? k * k * k : k * k;
  const int bb = B * B;
  const size_t shm = sizeof(double) * 4 * bb;
  if (nblocks == 0) return;
  if (shm > 65536) {  // only B = 64 (3D, degree 3)
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_galerkin_c<3, 4>),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) throw std::runtime_error("coarse Galerkin: LDS request too large for this device");
  }
  const int threads = bb <= 256 ? ((bb + 63) / 64) * 64 : 256;
#define R3MG_GC(DD, KK)                                                                                             \
  hipLaunchKernelGGL((k_galerkin_c<DD, KK>), dim3((unsigned)nblocks), dim3(threads), shm, s, shift, nbox_in, brow,  \
                     bptr_out, bcol_out, bptr_in, bcol_in, val_in, pt, out)
  switch (d * 8 + pc + 1) {
    case 17: R3MG_GC(2, 1); break;
    case 18: R3MG_GC(2, 2); break;
    case 19: R3MG_GC(2, 3); break;
    case 20: R3MG_GC(2, 4); break;
    case 25: R3MG_GC(3, 1); break;
    case 26: R3MG_GC(3, 2); break;
    case 27: R3MG_GC(3, 3); break;
    case 28: R3MG_GC(3, 4); break;
    default: throw std::runtime_error("coarse Galerkin product: unsupported dimension or degree");
  }
#undef R3MG_GC
  check_launch("k_galerkin_c");
}

// scatter the block rows of the coarsest level into a dense row-major matrix
__global__ void k_to_dense(int nbox, int B, const int* __restrict__ bptr, const int* __restrict__ bcol,
                           const double* __restrict__ val, double* dense) {
  const int row = blockIdx.x;  // one block per row
  const int K = row / B, q = row - K * B;
  const int j0 = bptr[K], nb = bptr[K + 1] - j0;
  const int nc = nbox * B;
  const int64_t vb = (int64_t)B * B * j0 + (int64_t)q * nb * B;
  for (int p = threadIdx.x; p < nb * B; p += blockDim.x) {
    const int j = p / B, c = p % B;
    dense[(int64_t)row * nc + (int64_t)bcol[j0 + j] * B + c] = val[vb + p];
  }
}
void launch_to_dense(int nbox, int B, const int* bptr, const int* bcol, const double* val, double* dense,
                     hipStream_t s) {
  hipLaunchKernelGGL(k_to_dense, dim3(nbox * B), dim3(256), 0, s, nbox, B, bptr, bcol, val, dense);
  check_launch("k_to_dense");
}

// Lanczos start vector v_i = ((u_i * 2654435761) mod 2^32) / 2^32 - 1/2, u_i = perm[i] (or i)
__global__ void k_lanczos_start(int n, const int* __restrict__ perm, double* v) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint64_t u = perm ? (uint64_t)perm[i] : (uint64_t)i;
  const uint64_t h = (u * 2654435761ull) & 0xffffffffull;
  v[i] = (double)h / 4294967296.0 - 0.5;
}
void launch_lanczos_start(int n, const int* perm, double* v, hipStream_t s) {
  hipLaunchKernelGGL(k_lanczos_start, dim3((n + 255) / 256), dim3(256), 0, s, n, perm, v);
  check_launch("k_lanczos_start");
}

__global__ void k_axpby(int64_t n, double a, const double* __restrict__ x, double b, double* y) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[i] = a * x[i] + b * y[i];
}
void launch_axpby(int64_t n, double a, const double* x, double b, double* y, hipStream_t s) {
  hipLaunchKernelGGL(k_axpby, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, a, x, b, y);
  check_launch("k_axpby");
}

// =============================================================================================
// Dense Cholesky factorisation and explicit inverse of the coarsest operator (float64, row-major, n x n).
// Blocked in 64 x 64 tiles; every tile product runs on the FP64 matrix cores (v_mfma_f64_16x16x4f64):
//   1. A = L L^T, right-looking by block columns k: the diagonal tile is factored in LDS and inverted
//      (D_k = L_kk^{-1}); the panel below becomes A[i,k] D_k^T; the trailing lower tiles lose A[i,k] A[j,k]^T.
//   2. Y = L^{-1}, forward by block rows k: Y[k, 0..k] <- D_k Y[k, 0..k] (Y starts at zero; Y[k,k] = D_k),
//      then Y[r, 0..k] -= L[r,k] Y[k, 0..k] for r > k.
//   3. A^{-1} = Y^T Y: upper tile (I, J), I <= J, sums Y[M,I]^T Y[M,J] over M >= J and is stored with its
//      mirror (L^{-T} L^{-1} = (L L^T)^{-1}).
// About n^3 / 3 flops in each step (the triangular structure is skipped), against n^3 / 3 + 2 n^3 for two full
// triangular solves on the identity.  Tiles reaching past n are padded with the identity on a diagonal tile
// and zeros elsewhere.  A non-positive pivot sets *bad (the factorisation then continues with pivot 1).
// =============================================================================================
constexpr int DT = 64;

// X[i][j] = M[(R + i) n + C + j] inside the matrix, outside it 1 on the diagonal of a diagonal tile (diag_pad)
// and 0 elsewhere; stored s[i][j], or s[j][i] with trans.  The tile product reads its operands as s[k][index]
// with the index running across the lanes, so an operand whose index is its row is loaded transposed.
// element (i, j) = (threadIdx.x / 64 + 4 q, threadIdx.x % 64) of tile (R, C), q < 16, from clamped addresses (all
// 16 loads issued before the first is used; entries outside the matrix are masked by dt_put)
constexpr int kDtK = DT * DT / 256;
__device__ inline void dt_fetch(double (&v)[kDtK], const double* __restrict__ M, int n, int R, int C) {
  const int j = threadIdx.x & 63, i0 = threadIdx.x >> 6;
  const int64_t cj = min(C + j, n - 1);
#pragma unroll
  for (int q = 0; q < kDtK; ++q) v[q] = M[(int64_t)min(R + i0 + 4 * q, n - 1) * n + cj];
}
// the fetched elements into LDS (transposed if trans); entries outside the matrix read as 0, or 1 on the diagonal
// (diag_pad)
__device__ inline void dt_put(double (*s)[DT + 1], const double (&v)[kDtK], int n, int R, int C, bool trans,
                              bool diag_pad) {
  const int j = threadIdx.x & 63, i0 = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < kDtK; ++q) {
    const int i = i0 + 4 * q;
    const double x = (R + i < n && C + j < n) ? v[q] : (diag_pad && i == j) ? 1.0 : 0.0;
    if (trans)
      s[j][i] = x;
    else
      s[i][j] = x;
  }
}
// tile (R, C) into LDS: the loads come from clamped addresses and are all issued before the first is used, and
// entries outside the matrix are masked afterwards (a load under a lane-dependent condition would be waited for
// on its own)
__device__ inline void dt_load(double (*s)[DT + 1], const double* __restrict__ M, int n, int R, int C, bool trans,
                               bool diag_pad) {
  double v[kDtK];
  dt_fetch(v, M, n, R, C);
  dt_put(s, v, n, R, C, trans, diag_pad);
}

// a 64 x 64 tile of 64 x 64 values stored contiguously (row-major) into LDS, transposed: s[e % 64][e / 64] = T[e]
// (all loads issued before the first store)
__device__ inline void dt_load_packed_t(double (*s)[DT + 1], const double* __restrict__ T) {
  constexpr int K = DT * DT / 256;
  double v[K];
#pragma unroll
  for (int q = 0; q < K; ++q) v[q] = T[threadIdx.x + 256 * q];
#pragma unroll
  for (int q = 0; q < K; ++q) {
    const int e = threadIdx.x + 256 * q;
    s[e & 63][e >> 6] = v[q];
  }
}

// acc += sum over k < 64 of Aop(i, k) Bop(k, j), Aop(i, k) = sa[k][i], Bop(k, j) = sb[k][j].  Wave w owns the
// output rows 32 (w / 2) .. + 31 and columns 32 (w % 2) .. + 31 as 2 x 2 subtiles of 16 x 16.  Lane l supplies
// A[l % 16][l / 16] of each 16 x 4 left operand and B[l / 16][l % 16] of each 4 x 16 right operand, and element r
// of its result is C[4 r + l / 16][l % 16] (the instruction's layout, checked on gfx950).
__device__ inline void dt_mfma(const double (*sa)[DT + 1], const double (*sb)[DT + 1], v4d acc[2][2]) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
  const int li = l & 15, lk = l >> 4;
#pragma unroll 4
  for (int k = 0; k < DT; k += 4) {
    const double a0 = sa[k + lk][r0 + li], a1 = sa[k + lk][r0 + 16 + li];
    const double b0 = sb[k + lk][c0 + li], b1 = sb[k + lk][c0 + 16 + li];
    acc[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0][0], 0, 0, 0);
    acc[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b1, acc[0][1], 0, 0, 0);
    acc[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1][0], 0, 0, 0);
    acc[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, acc[1][1], 0, 0, 0);
  }
}

__device__ inline void dt_zero(v4d acc[2][2]) {
  for (int s = 0; s < 2; ++s)
    for (int t = 0; t < 2; ++t) acc[s][t] = v4d{0.0, 0.0, 0.0, 0.0};
}

// f(row, col, value) for every element of the wave's part of the tile
template <typename F>
__device__ inline void dt_each(const v4d acc[2][2], F f) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
  for (int s = 0; s < 2; ++s)
    for (int t = 0; t < 2; ++t)
      for (int r = 0; r < 4; ++r) f(r0 + 16 * s + 4 * r + (l >> 4), c0 + 16 * t + (l & 15), acc[s][t][r]);
}

// the elements of tile (R, C) of M in the accumulator's layout (as dt_each visits them), from clamped addresses,
// all loads issued before the first is used
__device__ inline void dt_fetch_acc(double (&old)[2][2][4], const double* M, int n, int R, int C) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 16 * s + 4 * r + (l >> 4), j = c0 + 16 * t + (l & 15);
        old[s][t][r] = M[(int64_t)min(R + i, n - 1) * n + min(C + j, n - 1)];
      }
}

// M tile (R, C) = old - acc (sub) or = acc, inside the matrix
__device__ inline void dt_put_acc(const v4d acc[2][2], const double (&old)[2][2][4], double* M, int n, int R, int C,
                                  bool sub) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int r0 = 32 * (w >> 1), c0 = 32 * (w & 1);
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = r0 + 16 * s + 4 * r + (l >> 4), j = c0 + 16 * t + (l & 15);
        if (R + i < n && C + j < n) M[(int64_t)(R + i) * n + C + j] = sub ? old[s][t][r] - acc[s][t][r] : acc[s][t][r];
      }
}

// M tile (R, C) = acc, inside the matrix
__device__ inline void dt_store(const v4d acc[2][2], double* M, int n, int R, int C) {
  const double none[2][2][4] = {};
  dt_put_acc(acc, none, M, n, R, C, false);
}

// keeps fetched values ahead of a barrier (the compiler would otherwise sink their loads past it)
__device__ inline void dt_pin(const double (&old)[2][2][4]) {
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) asm volatile("" ::"v"(old[s][t][r]));
}

// 1. Diagonal tile k0: L with A_kk = L L^T (back to A, zero above the diagonal) and D = L^{-1} (to Dk, 64 x 64), by
// four waves, in four panels of 16 columns.
//   Panel: wave 0, lane l holding row l of the panel in registers, right-looking: column j is scaled by
//   1 / sqrt(pivot) and subtracted from the columns after it, the pivot and the factors L[c][j] coming from other
//   lanes by v_readlane.  Meanwhile wave 3 inverts the diagonal block of the panel before (lane c: column c, by
//   forward substitution) and waves 1 and 2 form the off-diagonal 16 x 16 blocks of the D row before that.
//   Then the four waves subtract the panel's products from the lower tiles behind it on the FP64 matrix cores.
// D_ij = -D_ii sum_{j <= k < i} L_ik D_kj, two chains of matrix instructions per block.
// Bound by the chain of 64 pivots, one after another (a reciprocal square root, a product, a lane read and a
// subtraction each), on one compute unit.  The earlier form (left-looking, a dot product from LDS, a square root, a
// shuffle and a division per column) took 38 us a tile on a 1,728-row level (27 tiles); this one 22.3 us (24.7 with the
// diagonal block inverted between the panels).
constexpr int kDiagLD = DT + 1;  // odd row stride in doubles: rows across the lanes spread over the banks
constexpr int kDiagP = 16;       // panel width

__device__ __forceinline__ double lane_value(double v, int lane) {  // lane: uniform
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                          __builtin_amdgcn_readlane(__double2loint(v), lane));
}

// a / g from y = 1 / g, corrected by the residual
__device__ __forceinline__ double diag_div(double a, double g, double y) {
  const double q = a * y;
  return fma(fma(-q, g, a), y, q);
}

// 16 x 16 tile product over LDS: C += sum over m < 16 of a[i * kDiagLD + m] B(m, j), B(m, j) = b[m * kDiagLD + j], or
// b[j * kDiagLD + m] with TB.  Lane l holds C[4 r + l / 16][l % 16], r < 4 (see dt_mfma).
template <bool TB>
__device__ __forceinline__ v4d diag_mfma16(const double* a, const double* b, v4d c) {
  const int li = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
#pragma unroll
  for (int m = 0; m < kDiagP; m += 4) {
    const double av = a[li * kDiagLD + m + lk];
    const double bv = TB ? b[li * kDiagLD + m + lk] : b[(m + lk) * kDiagLD + li];
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, c, 0, 0, 0);
  }
  return c;
}

// off-diagonal block (i, j) of D, by one wave (its own block of t holds the intermediate sum)
__device__ __forceinline__ void diag_inv_block(const double* s, double* t, int i, int j) {
  const int li = threadIdx.x & 15, lk = (threadIdx.x & 63) >> 4;
  v4d c = {0.0, 0.0, 0.0, 0.0};
  for (int k = j; k < i; ++k)
    c = diag_mfma16<false>(s + kDiagP * i * kDiagLD + kDiagP * k, t + kDiagP * k * kDiagLD + kDiagP * j, c);
  double* q = t + kDiagP * i * kDiagLD + kDiagP * j;
#pragma unroll
  for (int r = 0; r < 4; ++r) q[(4 * r + lk) * kDiagLD + li] = c[r];
  // the wave's LDS writes and reads stay in program order
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  c = diag_mfma16<false>(t + kDiagP * i * (kDiagLD + 1), q, v4d{0.0, 0.0, 0.0, 0.0});
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
  for (int r = 0; r < 4; ++r) q[(4 * r + lk) * kDiagLD + li] = -c[r];
}

// diagonal block p of D, by one wave: lane c < 16 solves L_pp d = e_c
__device__ __forceinline__ void diag_inv_diag(const double* s, double* t, const double* ivs, int p) {
  const int c0 = kDiagP * p, c = threadIdx.x & 15;
  double e[kDiagP];
#pragma unroll
  for (int i = 0; i < kDiagP; ++i) e[i] = i == c ? 1.0 : 0.0;
#pragma unroll
  for (int j = 0; j < kDiagP; ++j) {
    e[j] = diag_div(e[j], s[(c0 + j) * kDiagLD + c0 + j], ivs[c0 + j]);
#pragma unroll
    for (int i = j + 1; i < kDiagP; ++i) e[i] -= s[(c0 + i) * kDiagLD + c0 + j] * e[j];
  }
  if ((threadIdx.x & 63) < kDiagP) {
#pragma unroll
    for (int i = 0; i < kDiagP; ++i) t[(c0 + i) * kDiagLD + c0 + c] = e[i];
  }
}

__global__ __launch_bounds__(256) void k_dchol_diag(int n, int k0, double* A, double* Dk, int* bad) {
  __shared__ double s[DT * kDiagLD];  // the tile, then L
  __shared__ double t[DT * kDiagLD];  // D
  __shared__ double ivs[DT];          // 1 / L[j][j]
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  {
    double v[kDtK];
    dt_fetch(v, A, n, k0, k0);
#pragma unroll
    for (int q = 0; q < kDtK; ++q) {
      const int i = w + 4 * q;
      s[i * kDiagLD + l] = (k0 + i < n && k0 + l < n) ? v[q] : (i == l) ? 1.0 : 0.0;
      t[i * kDiagLD + l] = 0.0;
    }
  }
  __syncthreads();
  for (int p = 0; p < DT / kDiagP; ++p) {
    const int c0 = kDiagP * p;
    if (w == 0) {
      double r[kDiagP];
#pragma unroll
      for (int c = 0; c < kDiagP; ++c) r[c] = s[l * kDiagLD + c0 + c];
#pragma unroll
      for (int j = 0; j < kDiagP; ++j) {
        double piv = lane_value(r[j], c0 + j);
        if (!(piv > 0.0)) {
          if (l == 0) *bad = 1;
          piv = 1.0;
        }
        // g = sqrt(piv), y = 1 / g and the quotients r / g, each corrected by its residual (as accurate as a square
        // root and divisions, without their chains)
        const double y0 = rsqrt(piv);
        const double g0 = piv * y0, g = fma(fma(-g0, g0, piv), 0.5 * y0, g0);
        const double y = fma(fma(-g, y0, 1.0), y0, y0);
        const double lj = l < c0 + j ? 0.0 : l == c0 + j ? g : diag_div(r[j], g, y);
        r[j] = lj;
        if (l == 0) ivs[c0 + j] = y;
#pragma unroll
        for (int c = j + 1; c < kDiagP; ++c) r[c] -= lj * lane_value(lj, c0 + c);
      }
#pragma unroll
      for (int c = 0; c < kDiagP; ++c) s[l * kDiagLD + c0 + c] = r[c];
    } else if (w == 3) {
      if (p >= 1) diag_inv_diag(s, t, ivs, p - 1);
    } else if (w <= p - 2) {
      diag_inv_block(s, t, p - 2, w - 1);  // row p - 2 of D
    }
    __syncthreads();
    // lower tiles (a, b) behind the panel, p < b <= a < 4
    int q = 0;
    for (int a = p + 1; a < DT / kDiagP; ++a)
      for (int b = p + 1; b <= a; ++b, ++q) {
        if (q % 4 != w) continue;
        const v4d c = diag_mfma16<true>(s + kDiagP * a * kDiagLD + c0, s + kDiagP * b * kDiagLD + c0,
                                        v4d{0.0, 0.0, 0.0, 0.0});
#pragma unroll
        for (int r = 0; r < 4; ++r)
          s[(kDiagP * a + 4 * r + (l >> 4)) * kDiagLD + kDiagP * b + (l & 15)] -= c[r];
      }
    __syncthreads();
  }
  constexpr int last = DT / kDiagP - 1;
  if (w == 3)
    diag_inv_diag(s, t, ivs, last);
  else if (w >= 1)
    diag_inv_block(s, t, last - 1, w - 1);  // row last - 1 of D
  __syncthreads();
  if (w >= 1) diag_inv_block(s, t, last, w - 1);  // the last row of D
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kDtK; ++q) {
    const int i = w + 4 * q;
    Dk[i * DT + l] = t[i * kDiagLD + l];
    if (k0 + i < n && k0 + l < n) A[(int64_t)(k0 + i) * n + k0 + l] = s[i * kDiagLD + l];
  }
}

// 1. Panel: tile (k0 + 64 (1 + blockIdx.x), k0) of A becomes A_ik D_k^T (each workgroup owns its tile's rows).
__global__ __launch_bounds__(256) void k_dchol_panel(int n, int k0, double* A, const double* __restrict__ Dk) {
  __shared__ double sa[DT][DT + 1];
  __shared__ double sb[DT][DT + 1];
  const int R = k0 + DT * (1 + blockIdx.x);
  dt_load(sa, A, n, R, k0, true, false);   // Aop(i, k) = A_ik[i][k]
  // Bop(k, j) = D_k[j][k]
  dt_load_packed_t(sb, Dk);
  __syncthreads();
  v4d acc[2][2];
  dt_zero(acc);
  dt_mfma(sa, sb, acc);
  dt_store(acc, A, n, R, k0);
}

// 1. Trailing update of the lower tiles (I, J), k0 < J <= I: A_IJ -= A_Ik A_Jk^T, with I = k0/64 + 1 + a and
// J = k0/64 + 1 + b.  part 0: every pair (b <= a), enumerated row by row; part 1: the next column only (b = 0,
// a = blockIdx.x); part 2: the other columns (1 <= b <= a), enumerated row by row.
__global__ __launch_bounds__(256) void k_dchol_update(int n, int k0, double* A, int part) {
  __shared__ double sa[DT][DT + 1];
  __shared__ double sb[DT][DT + 1];
  int a, b;
  if (part == 1) {
    a = (int)blockIdx.x;
    b = 0;
  } else {
    a = (int)((sqrt(8.0 * blockIdx.x + 1.0) - 1.0) * 0.5);
    while ((a + 1) * (a + 2) / 2 <= (int)blockIdx.x) ++a;
    while (a * (a + 1) / 2 > (int)blockIdx.x) --a;
    b = (int)blockIdx.x - a * (a + 1) / 2;
    if (part == 2) {  // pairs of the triangle without column 0
      ++a;
      ++b;
    }
  }
  const int RI = k0 + DT * (1 + a), RJ = k0 + DT * (1 + b);
  double old[2][2][4];
  dt_fetch_acc(old, A, n, RI, RJ);           // the tile updated, in flight with the operands
  dt_load(sa, A, n, RI, k0, true, false);    // Aop(i, k) = A_Ik[i][k]
  dt_load(sb, A, n, RJ, k0, true, false);    // Bop(k, j) = A_Jk[j][k]
  dt_pin(old);
  __syncthreads();
  v4d acc[2][2];
  dt_zero(acc);
  dt_mfma(sa, sb, acc);
  dt_put_acc(acc, old, A, n, RI, RJ, true);
}

// 2. Block row k of Y: tile (k, j) for j = blockIdx.x <= k: Y_kj <- D_k Y_kj, except Y_kk = D_k.
__global__ __launch_bounds__(256) void k_dinv_row(int n, int kb, const double* __restrict__ Dk, double* Y) {
  __shared__ double sa[DT][DT + 1];
  __shared__ double sb[DT][DT + 1];
  const int j = blockIdx.x, R = DT * kb, C = DT * j;
  if (j == kb) {
    constexpr int K = DT * DT / 256;
    double v[K];
#pragma unroll
    for (int q = 0; q < K; ++q) v[q] = Dk[threadIdx.x + 256 * q];
#pragma unroll
    for (int q = 0; q < K; ++q) {
      const int e = threadIdx.x + 256 * q, r = e >> 6, c = e & 63;
      if (R + r < n && C + c < n) Y[(int64_t)(R + r) * n + C + c] = v[q];
    }
    return;
  }
  dt_load_packed_t(sa, Dk);   // Aop(i, k) = D_k[i][k]
  dt_load(sb, Y, n, R, C, false, false);                                         // Bop(k, j) = Y_kj[k][j]
  __syncthreads();
  v4d acc[2][2];
  dt_zero(acc);
  dt_mfma(sa, sb, acc);
  __syncthreads();
  dt_store(acc, Y, n, R, C);
}

// 2. Rows below block row k: tile (r, j), r = kb + 1 + blockIdx.x / (kb + 1), j = blockIdx.x % (kb + 1):
// Y_rj -= L_rk Y_kj.
__global__ __launch_bounds__(256) void k_dinv_update(int n, int kb, const double* __restrict__ L, double* Y) {
  __shared__ double sa[DT][DT + 1];
  __shared__ double sb[DT][DT + 1];
  const int r = kb + 1 + (int)blockIdx.x / (kb + 1), j = (int)blockIdx.x % (kb + 1);
  double old[2][2][4];
  dt_fetch_acc(old, Y, n, DT * r, DT * j);           // the tile updated, in flight with the operands
  dt_load(sa, L, n, DT * r, DT * kb, true, false);   // Aop(i, k) = L_rk[i][k]
  dt_load(sb, Y, n, DT * kb, DT * j, false, false);  // Bop(k, j) = Y_kj[k][j]
  dt_pin(old);
  __syncthreads();
  v4d acc[2][2];
  dt_zero(acc);
  dt_mfma(sa, sb, acc);
  dt_put_acc(acc, old, Y, n, DT * r, DT * j, true);
}

// 3. Upper tile (I, J) of A^{-1} = Y^T Y and its mirror; blockIdx.x enumerates the pairs I <= J row by row.
__global__ __launch_bounds__(256) void k_dinv_gram(int n, int nt, const double* __restrict__ Y, double* Inv) {
  __shared__ double sa[DT][DT + 1];
  __shared__ double sb[DT][DT + 1];
  int rem = (int)blockIdx.x, I = 0;
  while (rem >= nt - I) {
    rem -= nt - I;
    ++I;
  }
  const int J = I + rem;
  v4d acc[2][2];
  dt_zero(acc);
  // the tiles of step M + 1 are fetched into registers while step M's product runs from LDS
  double va[kDtK], vb[kDtK];
  dt_fetch(va, Y, n, DT * J, DT * I);
  dt_fetch(vb, Y, n, DT * J, DT * J);
  for (int M = J; M < nt; ++M) {
    dt_put(sa, va, n, DT * M, DT * I, false, false);   // Aop(i, k) = Y_MI[k][i]
    dt_put(sb, vb, n, DT * M, DT * J, false, false);   // Bop(k, j) = Y_MJ[k][j]
    __syncthreads();
    if (M + 1 < nt) {  // uniform over the workgroup
      dt_fetch(va, Y, n, DT * (M + 1), DT * I);
      dt_fetch(vb, Y, n, DT * (M + 1), DT * J);
    }
    dt_mfma(sa, sb, acc);
    __syncthreads();
  }
  dt_store(acc, Inv, n, DT * I, DT * J);
  if (I != J) {  // the mirror tile, staged in LDS so that its rows are written contiguously
    dt_each(acc, [&](int i, int j, double v) { sa[i][j] = v; });
    __syncthreads();
    for (int e = threadIdx.x; e < DT * DT; e += 256) {
      const int r = e >> 6, c = e & 63;  // mirror row r = tile column r
      if (DT * J + r < n && DT * I + c < n) Inv[(int64_t)(DT * J + r) * n + DT * I + c] = sa[c][r];
    }
  }
}

// ws: nt * 64 * 64 doubles (the inverted diagonal tiles); Y: n * n doubles of scratch
// The factorisation looks one step ahead: step kb's update of the next column (part 1) stays on s, while the
// update of the other columns (part 2) runs on a second stream from the end of panel kb on, so that part 1,
// diagonal tile and panel kb + 1, which touch column kb + 1 only, overlap it.  Part 1 of step kb + 1 writes column
// kb + 2, which part 2 of step kb also writes, so it waits for that; parts 2 follow one another on the second
// stream.
DenseLookAhead::~DenseLookAhead() {
  for (auto e : ev) (void)hipEventDestroy(e);
  if (s2) (void)hipStreamDestroy(s2);
}
// the stream and all events exist before the first launch, so that the host enqueues the steps ahead of the device
void DenseLookAhead::prepare(size_t count) {
  if (!s2 && hipStreamCreateWithFlags(&s2, hipStreamNonBlocking) != hipSuccess) {
    s2 = nullptr;
    throw std::runtime_error("dense Cholesky: stream creation failed");
  }
  while (ev.size() < count) {
    hipEvent_t e;
    if (hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess)
      throw std::runtime_error("dense Cholesky: event creation failed");
    ev.push_back(e);
  }
  next = 0;
}
hipEvent_t DenseLookAhead::event() {
  if (next == ev.size()) throw std::runtime_error("dense Cholesky: events exhausted");
  return ev[next++];
}

void dense_cholesky_inverse(int n, double* A, double* Inv, double* ws, double* Y, int* bad, DenseLookAhead& la,
                            hipStream_t s) {
  const int nt = (n + DT - 1) / DT;
  la.prepare(2 * (size_t)nt);
  hipEvent_t prev2 = nullptr;  // part 2 of the previous step done
  for (int kb = 0; kb < nt; ++kb) {
    const int k0 = kb * DT;
    double* Dk = ws + (size_t)kb * DT * DT;
    hipLaunchKernelGGL(k_dchol_diag, dim3(1), dim3(256), 0, s, n, k0, A, Dk, bad);
    const int below = nt - kb - 1;
    if (below > 0) {
      hipLaunchKernelGGL(k_dchol_panel, dim3(below), dim3(256), 0, s, n, k0, A, Dk);
      hipEvent_t done2 = nullptr;  // part 2 of this step done
      if (below > 1) {
        // part 2 needs this step's panel only (part 1 writes another column), so it is forked right after the
        // panel: no event then sits between part 1 and the next diagonal tile on s
        hipEvent_t main = la.event();
        if (hipEventRecord(main, s) != hipSuccess || hipStreamWaitEvent(la.s2, main, 0) != hipSuccess)
          throw std::runtime_error("dense Cholesky: event record failed");
        hipLaunchKernelGGL(k_dchol_update, dim3((below - 1) * below / 2), dim3(256), 0, la.s2, n, k0, A, 2);
        done2 = la.event();
        if (hipEventRecord(done2, la.s2) != hipSuccess) throw std::runtime_error("dense Cholesky: event record failed");
      }
      // part 1 writes the next column, which part 2 of the previous step also writes
      if (prev2 && hipStreamWaitEvent(s, prev2, 0) != hipSuccess)
        throw std::runtime_error("dense Cholesky: stream wait failed");
      hipLaunchKernelGGL(k_dchol_update, dim3(below), dim3(256), 0, s, n, k0, A, 1);
      if (done2) prev2 = done2;
    }
  }
  if (prev2 && hipStreamWaitEvent(s, prev2, 0) != hipSuccess)
    throw std::runtime_error("dense Cholesky: stream wait failed");
  check_launch("dense Cholesky");
  hipMemsetAsync(Y, 0, (size_t)n * n * sizeof(double), s);
  for (int kb = 0; kb < nt; ++kb) {
    hipLaunchKernelGGL(k_dinv_row, dim3(kb + 1), dim3(256), 0, s, n, kb, ws + (size_t)kb * DT * DT, Y);
    const int below = nt - kb - 1;
    if (below > 0) hipLaunchKernelGGL(k_dinv_update, dim3(below * (kb + 1)), dim3(256), 0, s, n, kb, A, Y);
  }
  hipLaunchKernelGGL(k_dinv_gram, dim3(nt * (nt + 1) / 2), dim3(256), 0, s, n, nt, Y, Inv);
  check_launch("dense inverse");
}

// =============================================================================================
// PCG (float64 outer iteration; scalars live on the device)
// =============================================================================================
// Every reduction is a vector kernel that stores per-block partial sums, followed by a one-block kernel that sums
// them in index order and updates the scalars in PcgState.  Vector kernels are grid-stride with at most
// kPcgBlocks blocks, so the partition of every reduction depends only on n and NR and a reduction's result never
// depends on the kernel that formed its operands.  (Finishing a reduction inside the vector kernel, in the block
// that arrives last, was measured slower: the device-scope release each block must issue before taking its
// ticket writes back its die's L2, and 1024 of them cost 60-80 us per kernel against ~4 us for the extra
// launch.)  Vectors are n x NR interleaved; thread t of a block always handles column t % NR of 256-row chunks
// (256 % NR == 0), so consecutive threads touch consecutive elements.

// Per-column block sums: butterfly over the lanes of one column, then the four waves in order; thread k < NR
// writes out[k].
template <int NR>
__device__ inline void column_partials(double acc, double* sh, double* out) {
#pragma unroll
  for (int off = 32; off >= NR; off >>= 1) acc += __shfl_xor(acc, off, 64);
  const int lane = threadIdx.x & 63;
  if (lane < NR) sh[(threadIdx.x >> 6) * NR + lane] = acc;
  __syncthreads();
  if (threadIdx.x < NR) {
    const int k = threadIdx.x;
    out[k] = (sh[k] + sh[NR + k]) + (sh[2 * NR + k] + sh[3 * NR + k]);
  }
}

// Column totals of part[b * stride + k] (k < NR, b < nb) by one 256-thread block: thread t sums blocks t / NR,
// t / NR + 256 / NR, ... of column t % NR in index order, then column_partials.  tot (shared) is valid in every
// thread on return.
template <int NR>
__device__ inline void column_totals(const double* __restrict__ part, int nb, int stride, double* sh, double* tot) {
  const int k = threadIdx.x % NR;
  constexpr int S = 256 / NR;
  double acc = 0;
  // U of the thread's partials at a time: loads issued together (clamped), added in index order.  With 1,024 partials
  // of 16 columns a thread has 64 of them: in batches of four, 16 round trips, k_pcg_beta of 16 columns took 9.6 us,
  // k_pcg_alpha 5.6 and the stop test 12.9-14.5; now 6.4, 4.7 and 4.7 (12.4 while one thread went through the columns)
  constexpr int U = NR >= 4 ? 16 : 4;
  for (int b0 = threadIdx.x / NR; b0 < nb; b0 += U * S) {
    double v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = part[(int64_t)min(b0 + u * S, nb - 1) * stride + k];
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (b0 + u * S < nb) acc += v[u];
  }
  column_partials<NR>(acc, sh, tot);
  __syncthreads();
}

// ---- Lanczos steps of the smoother set-up (D inner product), with alpha and beta on the device.  Each kernel ends in
// per-block partial sums that the next one totals itself (every block the same sums in the same order), so a step is
// the operator and three launches, and nothing is read back before the last step of the last level.  Reading each
// reduction back cost a round trip to the host of about 40 us, 21 of them per level, against 3 to 5 us a launch.

// partials of <x, y>_D
__global__ __launch_bounds__(256) void k_lanczos_dot(int64_t n, const double* __restrict__ diag,
                                                     const double* __restrict__ x, const double* __restrict__ y,
                                                     double* partials) {
  __shared__ double sh[4];
  double acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    acc += diag[i] * x[i] * y[i];
  const double t = block_sum256(acc, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}
// w = D^{-1} Av - beta vprev (vprev null: no such term); partials of <w, v>_D
__global__ __launch_bounds__(256) void k_lanczos_w(int64_t n, const double* __restrict__ dinv,
                                                   const double* __restrict__ Av, const double* __restrict__ beta,
                                                   const double* __restrict__ vprev, const double* __restrict__ diag,
                                                   const double* __restrict__ v, double* w, double* partials) {
  __shared__ double sh[4];
  const double bp = vprev ? *beta : 0.0;
  double acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    double t = dinv[i] * Av[i];
    if (vprev) t -= bp * vprev[i];
    w[i] = t;
    acc += diag[i] * t * v[i];
  }
  const double t = block_sum256(acc, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}
// alpha = the partials' total; w -= alpha v; partials of <w, w>_D into the second half
__global__ __launch_bounds__(256) void k_lanczos_alpha(int64_t n, const double* __restrict__ diag,
                                                       const double* __restrict__ v, double* w, double* partials,
                                                       double* alpha) {
  __shared__ double sh[4];
  __shared__ double tot[1];
  column_totals<1>(partials, gridDim.x, 1, sh, tot);
  const double a = tot[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) *alpha = a;
  double acc = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const double t = w[i] - a * v[i];
    w[i] = t;
    acc += diag[i] * t * t;
  }
  const double t = block_sum256(acc, sh);
  if (threadIdx.x == 0) partials[kLanczosBlocks + blockIdx.x] = t;
}
// beta = sqrt(the total of part); v = w / beta
__global__ __launch_bounds__(256) void k_lanczos_next(int64_t n, const double* w, const double* __restrict__ part,
                                                      double* v, double* beta) {
  __shared__ double sh[4];
  __shared__ double tot[1];
  column_totals<1>(part, gridDim.x, 1, sh, tot);
  const double bb = sqrt(tot[0]), s = 1.0 / bb;
  if (beta && blockIdx.x == 0 && threadIdx.x == 0) *beta = bb;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) v[i] = s * w[i];
}

static dim3 lanczos_grid(int64_t n) {
  return dim3((unsigned)std::max<int64_t>(1, std::min<int64_t>(kLanczosBlocks, (n + 255) / 256)));
}
void launch_lanczos_normalise(int64_t n, const double* diag, double* v, double* partials, hipStream_t s) {
  hipLaunchKernelGGL(k_lanczos_dot, lanczos_grid(n), dim3(256), 0, s, n, diag, v, v, partials);
  hipLaunchKernelGGL(k_lanczos_next, lanczos_grid(n), dim3(256), 0, s, n, v, partials, v, (double*)nullptr);
  check_launch("k_lanczos_next");
}
void launch_lanczos_step(int64_t n, const double* dinv, const double* diag, const double* Av, const double* v,
                         double* vprev, bool first, bool last, double* w, const double* beta_prev, double* alpha,
                         double* beta, double* partials, hipStream_t s) {
  hipLaunchKernelGGL(k_lanczos_w, lanczos_grid(n), dim3(256), 0, s, n, dinv, Av, beta_prev,
                     first ? (const double*)nullptr : vprev, diag, v, w, partials);
  hipLaunchKernelGGL(k_lanczos_alpha, lanczos_grid(n), dim3(256), 0, s, n, diag, v, w, partials, alpha);
  if (!last)
    hipLaunchKernelGGL(k_lanczos_next, lanczos_grid(n), dim3(256), 0, s, n, w, partials + kLanczosBlocks, vprev, beta);
  check_launch("k_lanczos_step");
}

// Two one-column totals at once, each exactly as column_totals<1> forms it (pa[b * sa] and pb[b * sb], b < nb):
// the loads of both are in flight together.  ta, tb (shared) are valid in every thread on return.
__device__ inline void column_totals2(const double* __restrict__ pa, int sa, const double* __restrict__ pb, int sb,
                                      int nb, double* sh, double* ta, double* tb) {
  double acca = 0, accb = 0;
  for (int b0 = threadIdx.x; b0 < nb; b0 += 4 * 256) {
    double va[4], vb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t b = min(b0 + u * 256, nb - 1);
      va[u] = pa[b * sa];
      vb[u] = pb[b * sb];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (b0 + u * 256 < nb) {
        acca += va[u];
        accb += vb[u];
      }
  }
  column_partials<1>(acca, sh, ta);
  __syncthreads();
  column_partials<1>(accb, sh, tb);
  __syncthreads();
}

// grid-stride steps of the one-column PCG vector kernels whose loads are issued together
constexpr int kPcgU = 4;
inline int pcg_grid(int n) {
  const int g = (n + 255) / 256;
  return std::max(1, std::min(g, kPcgBlocks));
}

#define R3_NR_SWITCH(nr, MACRO)                                   \
  switch (nr) {                                                   \
    case 1: MACRO(1); break;                                      \
    case 2: MACRO(2); break;                                      \
    case 4: MACRO(4); break;                                      \
    case 8: MACRO(8); break;                                      \
    case 16: MACRO(16); break;                                    \
    default: throw std::runtime_error("unsupported nrhs block");  \
  }

__device__ inline void pcg_set_alpha(PcgState* st, int k, double pq) {
  st->alpha[k] = st->done[k] ? 0.0 : st->gamma[k] / pq;
  const int j = st->iters[k];
  if (!st->done[k] && st->hist && j < st->hist_rows) st->hist[(int64_t)2 * j * kMaxNR + k] = st->alpha[k];
}

// <p, q> per column: partials[b * NR + k]
template <int NR>
__global__ __launch_bounds__(256) void k_pcg_dot(int n, const double* __restrict__ p, const double* __restrict__ q,
                                                 double* partials, const PcgState* __restrict__ st) {
  __shared__ double sh[4 * NR];
  if (st->all_done) return;
  double acc = 0;
  const int64_t tn = (int64_t)n * NR;
  // U grid-stride steps at a time: their loads are issued together (clamped addresses), then summed in the
  // element order of one step after another
  constexpr int U = NR >= 4 ? 1 : 4 / NR;
  const int64_t step = (int64_t)gridDim.x * 256 * NR;
  for (int64_t base = (int64_t)blockIdx.x * 256 * NR; base < tn; base += U * step) {
    double pv[U][NR], qv[U][NR];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int m = 0; m < NR; ++m) {
        const int64_t o = min(base + u * step + threadIdx.x + 256 * m, tn - 1);
        pv[u][m] = p[o];
        qv[u][m] = q[o];
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int m = 0; m < NR; ++m)
        if (base + u * step + threadIdx.x + 256 * m < tn) acc += pv[u][m] * qv[u][m];
  }
  column_partials<NR>(acc, sh, partials + (int64_t)blockIdx.x * NR);
}
template <int NR>
__global__ __launch_bounds__(256) void k_pcg_alpha_nr(PcgState* st, const double* __restrict__ partials, int nb) {
  __shared__ double sh[4 * NR];
  __shared__ double tot[NR];
  if (st->all_done) return;
  column_totals<NR>(partials, nb, NR, sh, tot);
  if (threadIdx.x < NR) pcg_set_alpha(st, threadIdx.x, tot[threadIdx.x]);
}
void launch_pcg_dot_alpha(int n, int nr, const double* p, const double* q, double* partials, PcgState* st,
                          hipStream_t s) {
  const int g = pcg_grid(n);
#define R3_DA(NRV)                                                                                 \
  hipLaunchKernelGGL((k_pcg_dot<NRV>), dim3(g), dim3(256), 0, s, n, p, q, partials, st);           \
  hipLaunchKernelGGL((k_pcg_alpha_nr<NRV>), dim3(1), dim3(256), 0, s, st, partials, g)
  R3_NR_SWITCH(nr, R3_DA)
#undef R3_DA
  check_launch("k_pcg_dot / k_pcg_alpha");
}

// alpha from partials formed by another kernel (the lanes kernel's fused dot: up to one partial per 32 rows),
// one 1024-thread block summing each column in a fixed order
__global__ __launch_bounds__(1024) void k_pcg_alpha(int nr, PcgState* st, const double* __restrict__ partials, int npart) {
  __shared__ double sh[16];
  if (st->all_done) return;
  for (int k = 0; k < nr; ++k) {
    double a0 = 0, a1 = 0, a2 = 0, a3 = 0;
    int b = threadIdx.x;
    for (; b + 3 * 1024 < npart; b += 4 * 1024) {
      a0 += partials[(int64_t)b * nr + k];
      a1 += partials[(int64_t)(b + 1024) * nr + k];
      a2 += partials[(int64_t)(b + 2048) * nr + k];
      a3 += partials[(int64_t)(b + 3072) * nr + k];
    }
    for (; b < npart; b += 1024) a0 += partials[(int64_t)b * nr + k];
    const double v = wave_sum((a0 + a1) + (a2 + a3), 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
      double pq = 0;
      for (int i = 0; i < 16; ++i) pq += sh[i];
      pcg_set_alpha(st, k, pq);
    }
    __syncthreads();
  }
}
void launch_pcg_alpha(int nr, PcgState* st, const double* partials, int npart, hipStream_t s) {
  hipLaunchKernelGGL(k_pcg_alpha, dim3(1), dim3(1024), 0, s, nr, st, partials, npart);
  check_launch("k_pcg_alpha");
}

// x += alpha p; r -= alpha q; ||r||^2 partials; V-cycle entry b0 = (T) r, d0 = dinv0 b0 / theta0
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_pcg_xr(int n, const PcgState* __restrict__ st, double* x, double* r,
                                                const double* __restrict__ p, const double* __restrict__ q,
                                                double* partials, T* b0, const T* __restrict__ dinv0, T* d0,
                                                T inv_theta0) {
  __shared__ double sh[4 * NR];
  if (st->all_done) return;
  const int k = threadIdx.x % NR;
  const double al = st->alpha[k];
  const int64_t tn = (int64_t)n * NR;
  double acc = 0;
  // U elements at a time, loads issued together (clamped addresses: loads under a lane's own condition are waited for
  // one by one), in the order of the elements.  3D Q3 16^3, 16 columns, float32 V-cycle 26 -> 19.4 us (80 MB), k_pcg_z
  // 15.1 -> 12.1
  constexpr int U = NR < 4 ? NR : 4;
  for (int64_t base = (int64_t)blockIdx.x * 256 * NR; base < tn; base += (int64_t)gridDim.x * 256 * NR)
#pragma unroll
    for (int m0 = 0; m0 < NR; m0 += U) {
      double xv[U], pv[U], rv[U], qv[U];
      T dv[U];
#pragma unroll
      for (int m = 0; m < U; ++m) {
        const int64_t o = min(base + threadIdx.x + 256 * (m0 + m), tn - 1);
        xv[m] = x[o];
        pv[m] = p[o];
        rv[m] = r[o];
        qv[m] = q[o];
        dv[m] = d0 ? dinv0[o / NR] : (T)0;
      }
#pragma unroll
      for (int m = 0; m < U; ++m) {
        const int64_t o = base + threadIdx.x + 256 * (m0 + m);
        if (o < tn) {
          x[o] = xv[m] + al * pv[m];
          const double r1 = rv[m] - al * qv[m];
          r[o] = r1;
          acc += r1 * r1;
          if (b0) {
            const T bv = (T)r1;
            b0[o] = bv;
            if (d0) d0[o] = dv[m] * bv * inv_theta0;
          } else if (d0) {
            d0[o] = dv[m] * (T)r1 * inv_theta0;
          }
        }
      }
    }
  column_partials<NR>(acc, sh, partials + (int64_t)blockIdx.x * NR);
}
// the stop test of every open column (iteration count, squared residual and its history, done flag), all_done
template <int NR>
__global__ __launch_bounds__(256) void k_pcg_check(PcgState* st, const double* __restrict__ partials, int nb) {
  __shared__ double sh[4 * NR];
  __shared__ double tot[NR];
  if (st->all_done) return;
  column_totals<NR>(partials, nb, NR, sh, tot);
  if (threadIdx.x < 64) {  // a lane per column
    const int c = threadIdx.x;
    int d = c < NR ? st->done[c] : 1;
    if (!d) {
      const double rr = tot[c];
      st->rr_prev[c] = st->rr[c];
      st->rr[c] = rr;
      const int j = st->iters[c] + 1;
      st->iters[c] = j;
      if (st->rhist && j <= st->hist_rows) st->rhist[(int64_t)j * kMaxNR + c] = rr;
      d = rr <= st->tau2[c];
      if (d) st->done[c] = 1;
    }
    const int all = __all(d);
    if (threadIdx.x == 0) st->all_done = all;
  }
}
template <typename T>
void launch_pcg_xr(int n, int nr, PcgState* st, double* x, double* r, const double* p, const double* q,
                   double* partials, T* b0, const T* dinv0, T* d0, double inv_theta0, hipStream_t s) {
  const int g = pcg_grid(n);
#define R3_XR(NRV)                                                                                              \
  hipLaunchKernelGGL((k_pcg_xr<T, NRV>), dim3(g), dim3(256), 0, s, n, st, x, r, p, q, partials, b0, dinv0, d0, \
                     (T)inv_theta0);                                                                           \
  hipLaunchKernelGGL((k_pcg_check<NRV>), dim3(1), dim3(256), 0, s, st, partials, g)
  R3_NR_SWITCH(nr, R3_XR)
#undef R3_XR
  check_launch("k_pcg_xr / k_pcg_check");
}
template void launch_pcg_xr<float>(int, int, PcgState*, double*, double*, const double*, const double*, double*,
                                   float*, const float*, float*, double, hipStream_t);
template void launch_pcg_xr<double>(int, int, PcgState*, double*, double*, const double*, const double*, double*,
                                    double*, const double*, double*, double, hipStream_t);

// z = x0 + dpend (in float64); mode 1: p = z; modes 1, 2: partials of <r, z> and (q set) <q, z>
template <typename T, int NR>
__global__ __launch_bounds__(256) void k_pcg_z(int n, const PcgState* __restrict__ st, int mode,
                                               const T* __restrict__ x0, const T* __restrict__ dp, double* z,
                                               const double* __restrict__ r, const double* __restrict__ q,
                                               double* pvec, double* partials) {
  __shared__ double sh[4 * NR];
  if (mode != 0 && st->all_done) return;
  const int64_t tn = (int64_t)n * NR;
  double a1 = 0, a2 = 0;
  constexpr int U = NR < 4 ? NR : 4;  // elements at a time, as in k_pcg_xr
  for (int64_t base = (int64_t)blockIdx.x * 256 * NR; base < tn; base += (int64_t)gridDim.x * 256 * NR)
#pragma unroll
    for (int m0 = 0; m0 < NR; m0 += U) {
      T vv[U], dv[U];
      double rv[U], qv[U];
#pragma unroll
      for (int m = 0; m < U; ++m) {
        const int64_t o = min(base + threadIdx.x + 256 * (m0 + m), tn - 1);
        vv[m] = x0[o];
        dv[m] = dp ? dp[o] : (T)0;
        rv[m] = mode != 0 ? r[o] : 0.0;
        qv[m] = mode != 0 && q ? q[o] : 0.0;
      }
#pragma unroll
      for (int m = 0; m < U; ++m) {
        const int64_t o = base + threadIdx.x + 256 * (m0 + m);
        if (o < tn) {
          T v = vv[m];
          if (dp) v += dv[m];
          const double zv = (double)v;
          z[o] = zv;
          if (mode == 1) pvec[o] = zv;
          if (mode != 0) {
            a1 += rv[m] * zv;
            if (q) a2 += qv[m] * zv;
          }
        }
      }
    }
  if (mode == 0) return;
  double* out = partials + (int64_t)blockIdx.x * 2 * NR;
  column_partials<NR>(a1, sh, out);
  __syncthreads();
  column_partials<NR>(a2, sh, out + NR);
}
// mode 1: gamma = <r, z>; mode 2: beta (standard gamma'/gamma, or flexible -alpha <q, z> / gamma) and gamma
template <int NR>
__global__ __launch_bounds__(256) void k_pcg_beta(PcgState* st, int mode, const double* __restrict__ partials,
                                                  int nb) {
  __shared__ double sh[4 * NR];
  __shared__ double rz[NR], qz[NR];
  if (st->all_done) return;
  column_totals<NR>(partials, nb, 2 * NR, sh, rz);
  column_totals<NR>(partials + NR, nb, 2 * NR, sh, qz);
  if (threadIdx.x < NR) {
    const int c = threadIdx.x;
    if (mode == 1) {
      st->gamma[c] = rz[c];
    } else if (!st->done[c]) {
      const double g = st->gamma[c];
      st->beta[c] = st->flexible ? (-st->alpha[c] * qz[c]) / g : rz[c] / g;
      st->gamma[c] = rz[c];
      const int j = st->iters[c] - 1;  // the stop test of iteration j has counted it
      if (st->hist && j >= 0 && j < st->hist_rows) st->hist[(int64_t)(2 * j + 1) * kMaxNR + c] = st->beta[c];
    }
  }
}
template <typename T>
void launch_pcg_z(int n, int nr, PcgState* st, int mode, const T* x0, const T* dpend, double* z, const double* r,
                  const double* q, double* p, double* partials, hipStream_t s) {
  const int g = pcg_grid(n);
#define R3_Z(NRV)                                                                                                  \
  hipLaunchKernelGGL((k_pcg_z<T, NRV>), dim3(g), dim3(256), 0, s, n, st, mode, x0, dpend, z, r, q, p, partials); \
  if (mode != 0) hipLaunchKernelGGL((k_pcg_beta<NRV>), dim3(1), dim3(256), 0, s, st, mode, partials, g)
  R3_NR_SWITCH(nr, R3_Z)
#undef R3_Z
  check_launch("k_pcg_z / k_pcg_beta");
}
template void launch_pcg_z<float>(int, int, PcgState*, int, const float*, const float*, double*, const double*,
                                  const double*, double*, double*, hipStream_t);
template void launch_pcg_z<double>(int, int, PcgState*, int, const double*, const double*, double*, const double*,
                                   const double*, double*, double*, hipStream_t);

__global__ void k_pcg_p(int n, int nr, const PcgState* __restrict__ st, const double* __restrict__ z, double* p) {
  if (st->all_done) return;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= (int64_t)n * nr) return;
  const int k = (int)(t % nr);
  if (st->done[k]) return;
  p[t] = z[t] + st->beta[k] * p[t];
}
void launch_pcg_p(int n, int nr, PcgState* st, const double* z, double* p, hipStream_t s) {
  const int64_t tot = (int64_t)n * nr;
  hipLaunchKernelGGL(k_pcg_p, dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, n, nr, st, z, p);
  check_launch("k_pcg_p");
}

// One right-hand side: the scalar steps folded into the vector kernels that follow their reductions.  Every block of
// the next kernel forms the reduction's total itself from the per-block partials (column_totals<1>: the same sums in
// the same order as the one-block kernels above, so the same bits in every block) and block 0 records it in the
// state; each reduction has its own partials area, so that no block overwrites partials another block still reads:
// area 0 (g entries) <p, q>, area 1 (g) ||r||^2, area 2 (2 g) <r, z> and <q, z>, g = pcg_grid(n).  gamma is formed
// from area 2 by the kernel that needs it, so no kernel writes a state scalar that another block of it reads.
int pcg_blocks(int n) { return pcg_grid(n); }

void launch_pcg_dot(int n, const double* p, const double* q, double* partials, PcgState* st, hipStream_t s) {
  hipLaunchKernelGGL((k_pcg_dot<1>), dim3(pcg_grid(n)), dim3(256), 0, s, n, p, q, partials, st);
  check_launch("k_pcg_dot");
}

// alpha = gamma / <p, q> (gamma = <r, z> from area 2); x += alpha p; r -= alpha q; ||r||^2 partials to area 1;
// V-cycle entry b0 = (T) r, d0 = dinv0 b0 / theta0
template <typename T>
__global__ __launch_bounds__(256) void k_pcg_xr1(int n, PcgState* st, double* x, double* r,
                                                 const double* __restrict__ p, const double* __restrict__ q,
                                                 double* partials, int g, T* b0, const T* __restrict__ dinv0, T* d0,
                                                 T inv_theta0) {
  __shared__ double sh[4];
  __shared__ double gam[1], pq[1];
  if (st->all_done) return;
  column_totals2(partials + 2 * g, 2, partials, 1, g, sh, gam, pq);
  const double al = st->done[0] ? 0.0 : gam[0] / pq[0];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->gamma[0] = gam[0];
    pcg_set_alpha(st, 0, pq[0]);
  }
  double acc = 0;
  // kPcgU grid-stride steps at a time, loads issued together (clamped addresses), in the element order of the
  // steps one after another
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t o0 = (int64_t)blockIdx.x * 256 + threadIdx.x; o0 < n; o0 += kPcgU * step) {
    double xv[kPcgU], pv[kPcgU], rv[kPcgU], qv[kPcgU];
    T dv[kPcgU];
#pragma unroll
    for (int u = 0; u < kPcgU; ++u) {
      const int64_t o = min(o0 + u * step, (int64_t)n - 1);
      xv[u] = x[o];
      pv[u] = p[o];
      rv[u] = r[o];
      qv[u] = q[o];
      dv[u] = d0 ? dinv0[o] : (T)0;
    }
#pragma unroll
    for (int u = 0; u < kPcgU; ++u) {
      const int64_t o = o0 + u * step;
      if (o < n) {
        x[o] = xv[u] + al * pv[u];
        const double r1 = rv[u] - al * qv[u];
        r[o] = r1;
        acc += r1 * r1;
        if (b0) {
          const T bv = (T)r1;
          b0[o] = bv;
          if (d0) d0[o] = dv[u] * bv * inv_theta0;
        } else if (d0) {
          d0[o] = dv[u] * (T)r1 * inv_theta0;
        }
      }
    }
  }
  column_partials<1>(acc, sh, partials + g + blockIdx.x);
}
template <typename T>
void launch_pcg_xr1(int n, PcgState* st, double* x, double* r, const double* p, const double* q, double* partials,
                    T* b0, const T* dinv0, T* d0, double inv_theta0, hipStream_t s) {
  const int g = pcg_grid(n);
  hipLaunchKernelGGL((k_pcg_xr1<T>), dim3(g), dim3(256), 0, s, n, st, x, r, p, q, partials, g, b0, dinv0, d0,
                     (T)inv_theta0);
  check_launch("k_pcg_xr1");
}
template void launch_pcg_xr1<float>(int, PcgState*, double*, double*, const double*, const double*, double*, float*,
                                    const float*, float*, double, hipStream_t);
template void launch_pcg_xr1<double>(int, PcgState*, double*, double*, const double*, const double*, double*,
                                     double*, const double*, double*, double, hipStream_t);

// check set: the stop test of the column (from the ||r||^2 partials of area 1, block 0 records it); z = x0 + dpend;
// <r, z> and (q set) <q, z> partials to area 2
template <typename T>
__global__ __launch_bounds__(256) void k_pcg_z1(int n, PcgState* st, int check, const T* __restrict__ x0,
                                                const T* __restrict__ dp, double* z, const double* __restrict__ r,
                                                const double* __restrict__ q, double* partials, int g) {
  __shared__ double sh[4];
  __shared__ double rr[1];
  if (st->all_done) return;
  // only block 0 records the stop test; the vector work below does not depend on it
  if (check && blockIdx.x == 0) column_totals<1>(partials + g, g, 1, sh, rr);
  if (check && blockIdx.x == 0 && threadIdx.x == 0 && !st->done[0]) {
    st->rr_prev[0] = st->rr[0];
    st->rr[0] = rr[0];
    const int j = st->iters[0] + 1;
    st->iters[0] = j;
    if (st->rhist && j <= st->hist_rows) st->rhist[(int64_t)j * kMaxNR] = rr[0];
    if (rr[0] <= st->tau2[0]) st->done[0] = 1;
    st->all_done = st->done[0];
  }
  double a1 = 0, a2 = 0;
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t o0 = (int64_t)blockIdx.x * 256 + threadIdx.x; o0 < n; o0 += kPcgU * step) {
    T xv[kPcgU], dv[kPcgU];
    double rv[kPcgU], qv[kPcgU];
#pragma unroll
    for (int u = 0; u < kPcgU; ++u) {
      const int64_t o = min(o0 + u * step, (int64_t)n - 1);
      xv[u] = x0[o];
      dv[u] = dp ? dp[o] : (T)0;
      rv[u] = r[o];
      qv[u] = q ? q[o] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < kPcgU; ++u) {
      const int64_t o = o0 + u * step;
      if (o < n) {
        T v = xv[u];
        if (dp) v += dv[u];
        const double zv = (double)v;
        z[o] = zv;
        a1 += rv[u] * zv;
        if (q) a2 += qv[u] * zv;
      }
    }
  }
  double* out = partials + 2 * g + (int64_t)blockIdx.x * 2;
  column_partials<1>(a1, sh, out);
  __syncthreads();
  column_partials<1>(a2, sh, out + 1);
}
template <typename T>
void launch_pcg_z1(int n, PcgState* st, bool check, const T* x0, const T* dpend, double* z, const double* r,
                   const double* q, double* partials, hipStream_t s) {
  const int g = pcg_grid(n);
  hipLaunchKernelGGL((k_pcg_z1<T>), dim3(g), dim3(256), 0, s, n, st, check ? 1 : 0, x0, dpend, z, r, q, partials,
                     g);
  check_launch("k_pcg_z1");
}
template void launch_pcg_z1<float>(int, PcgState*, bool, const float*, const float*, double*, const double*,
                                   const double*, double*, hipStream_t);
template void launch_pcg_z1<double>(int, PcgState*, bool, const double*, const double*, double*, const double*,
                                    const double*, double*, hipStream_t);

// the stop test alone (from area 1), for an iteration enqueued as two halves
void launch_pcg_check1(int n, PcgState* st, const double* partials, hipStream_t s) {
  const int g = pcg_grid(n);
  hipLaunchKernelGGL((k_pcg_check<1>), dim3(1), dim3(256), 0, s, st, partials + g, g);
  check_launch("k_pcg_check");
}

// beta (standard <r, z> / gamma or flexible -alpha <q, z> / gamma, from area 2; block 0 records it); p = z + beta p
__global__ __launch_bounds__(256) void k_pcg_p1(int n, PcgState* st, const double* __restrict__ z, double* p,
                                                const double* __restrict__ partials, int g) {
  __shared__ double sh[4];
  __shared__ double rz[1], qz[1];
  if (st->all_done || st->done[0]) return;
  column_totals2(partials + 2 * g, 2, partials + 2 * g + 1, 2, g, sh, rz, qz);
  const double gold = st->gamma[0];
  const double be = st->flexible ? (-st->alpha[0] * qz[0]) / gold : rz[0] / gold;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->beta[0] = be;
    const int j = st->iters[0] - 1;  // the stop test of iteration j has counted it
    if (st->hist && j >= 0 && j < st->hist_rows) st->hist[(int64_t)(2 * j + 1) * kMaxNR] = be;
  }
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t o0 = (int64_t)blockIdx.x * 256 + threadIdx.x; o0 < n; o0 += kPcgU * step) {
    double zv[kPcgU], pv[kPcgU];
#pragma unroll
    for (int u = 0; u < kPcgU; ++u) {
      const int64_t o = min(o0 + u * step, (int64_t)n - 1);
      zv[u] = z[o];
      pv[u] = p[o];
    }
#pragma unroll
    for (int u = 0; u < kPcgU; ++u) {
      const int64_t o = o0 + u * step;
      if (o < n) p[o] = zv[u] + be * pv[u];
    }
  }
}
void launch_pcg_p1(int n, PcgState* st, const double* z, double* p, const double* partials, hipStream_t s) {
  const int g = pcg_grid(n);
  hipLaunchKernelGGL(k_pcg_p1, dim3(g), dim3(256), 0, s, n, st, z, p, partials, g);
  check_launch("k_pcg_p1");
}

// ||b - q||^2 partials per column; with r set, r = b - q as well
template <int NR>
__global__ __launch_bounds__(256) void k_pcg_residual(int n, const double* __restrict__ b, const double* __restrict__ q,
                                                      double* r, double* partials) {
  __shared__ double sh[4 * NR];
  const int64_t tn = (int64_t)n * NR;
  double acc = 0;
  for (int64_t base = (int64_t)blockIdx.x * 256 * NR; base < tn; base += (int64_t)gridDim.x * 256 * NR)
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const int64_t o = base + threadIdx.x + 256 * m;
      if (o < tn) {
        const double v = b[o] - q[o];
        if (r) r[o] = v;
        acc += v * v;
      }
    }
  column_partials<NR>(acc, sh, partials + (int64_t)blockIdx.x * NR);
}
// the initial state (fresh solve, or a restart from the true residual that keeps tau^2, ||r_0||^2 and the
// iteration counts)
template <int NR>
__global__ __launch_bounds__(256) void k_pcg_init(PcgState* st, const double* __restrict__ partials, int nb,
                                                  int restart, double rtol, double atol, int nr_active, int flexible,
                                                  double* hist, double* rhist, int hist_rows) {
  __shared__ double sh[4 * NR];
  __shared__ double tot[NR];
  column_totals<NR>(partials, nb, NR, sh, tot);
  if (threadIdx.x == 0) {
    int all = 1;
    for (int c = 0; c < NR; ++c) {
      const double rr = tot[c];
      if (!restart) {
        st->rr0[c] = rr;
        st->tau2[c] = fmax(rtol * rtol * rr, atol * atol);  // ||r|| <= max(rtol ||r0||, atol)
        st->iters[c] = 0;
        if (rhist && hist_rows >= 0) rhist[c] = rr;
      }
      st->rr[c] = rr;
      st->rr_prev[c] = rr;
      st->rr_true[c] = rr;
      st->alpha[c] = 0;
      st->beta[c] = 0;
      st->done[c] = (c >= nr_active) || (rr <= st->tau2[c]);
      all &= st->done[c];
    }
    st->all_done = all;
    st->nr = NR;
    st->flexible = flexible;
    st->restart = 0;
    st->hist = hist;
    st->rhist = rhist;
    st->hist_rows = hist_rows;
  }
}
void launch_pcg_residual_init(int n, int nr, const double* b, const double* q, double* r, double* partials,
                              PcgState* st, int restart, double rtol, double atol, int nr_active, int flexible,
                              double* hist, double* rhist, int hist_rows, hipStream_t s) {
  const int g = pcg_grid(n);
#define R3_RI(NRV)                                                                                               \
  hipLaunchKernelGGL((k_pcg_residual<NRV>), dim3(g), dim3(256), 0, s, n, b, q, r, partials);                    \
  hipLaunchKernelGGL((k_pcg_init<NRV>), dim3(1), dim3(256), 0, s, st, partials, g, restart, rtol, atol, nr_active, \
                     flexible, hist, rhist, hist_rows)
  R3_NR_SWITCH(nr, R3_RI)
#undef R3_RI
  check_launch("k_pcg_residual / k_pcg_init");
}

// the true residual recorded, and a restart flagged when a column the recursive residual declared converged fails
// the stop rule with it
template <int NR>
__global__ __launch_bounds__(256) void k_pcg_true_check(PcgState* st, const double* __restrict__ partials, int nb) {
  __shared__ double sh[4 * NR];
  __shared__ double tot[NR];
  column_totals<NR>(partials, nb, NR, sh, tot);
  if (threadIdx.x == 0) {
    int rs = 0;
    for (int c = 0; c < NR; ++c) {
      st->rr_true[c] = tot[c];
      if (st->done[c] && tot[c] > st->tau2[c]) rs = 1;
    }
    st->restart = rs;
  }
}
void launch_pcg_true_residual(int n, int nr, const double* b, const double* q, double* partials, PcgState* st,
                              hipStream_t s) {
  const int g = pcg_grid(n);
#define R3_TR(NRV)                                                                                           \
  hipLaunchKernelGGL((k_pcg_residual<NRV>), dim3(g), dim3(256), 0, s, n, b, q, nullptr, partials);          \
  hipLaunchKernelGGL((k_pcg_true_check<NRV>), dim3(1), dim3(256), 0, s, st, partials, g)
  R3_NR_SWITCH(nr, R3_TR)
#undef R3_TR
  check_launch("k_pcg_residual / k_pcg_true_check");
}

// the state, word by word, into host-mapped pinned memory
__global__ void k_pcg_state_out(const uint64_t* __restrict__ src, uint64_t* dst, int words) {
  for (int i = threadIdx.x; i < words; i += blockDim.x) dst[i] = src[i];
}
void launch_pcg_state_out(const PcgState* st, PcgState* host_mapped, hipStream_t s) {
  static_assert(sizeof(PcgState) % 8 == 0, "PcgState is copied in 8-byte words");
  hipLaunchKernelGGL(k_pcg_state_out, dim3(1), dim3(256), 0, s, reinterpret_cast<const uint64_t*>(st),
                     reinterpret_cast<uint64_t*>(host_mapped), (int)(sizeof(PcgState) / 8));
  check_launch("k_pcg_state_out");
}

template <typename T>
__global__ void k_vc_prep(int64_t count, int nr, const double* __restrict__ r, T* b0, const T* __restrict__ dinv0,
                          T* d0, T inv_theta0, const int* __restrict__ skip) {
  if (skip && *skip) return;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= count) return;
  const T v = (T)r[t];
  if (b0) b0[t] = v;
  if (d0) d0[t] = dinv0[t / nr] * v * inv_theta0;
}
template <typename T>
void launch_vc_prep(int n, int nr, const double* r, T* b0, const T* dinv0, T* d0, double inv_theta0,
                    const int* skip, hipStream_t s) {
  const int64_t tot = (int64_t)n * nr;
  hipLaunchKernelGGL((k_vc_prep<T>), dim3((unsigned)((tot + 255) / 256)), dim3(256), 0, s, tot, nr, r, b0, dinv0, d0,
                     (T)inv_theta0, skip);
  check_launch("k_vc_prep");
}
template void launch_vc_prep<float>(int, int, const double*, float*, const float*, float*, double, const int*,
                                    hipStream_t);
template void launch_vc_prep<double>(int, int, const double*, double*, const double*, double*, double, const int*,
                                     hipStream_t);

// =============================================================================================
// FEM helpers for the differentiable solve
// =============================================================================================
// g_e = - sum_{a,b free} lam[c_ea] Ke[a,b] u[c_eb]; one wave per cell
__global__ __launch_bounds__(256) void k_cell_grad(int64_t ncells, int nloc, const int* __restrict__ cells,
                                                   const double* __restrict__ Ke, int64_t ke_stride,
                                                   const double* __restrict__ u, const double* __restrict__ lam,
                                                   const unsigned char* __restrict__ cons, double* g) {
  const int64_t e = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (e >= ncells) return;
  const int* c = cells + e * nloc;
  const double* K = Ke + e * ke_stride;
  double acc = 0;
  for (int a = 0; a < nloc; ++a) {
    const int ia = c[a];
    if (cons[ia]) continue;
    const double la = lam[ia];
    double s = 0;
    for (int b = lane; b < nloc; b += 64) {
      const int ib = c[b];
      if (!cons[ib]) s += K[(int64_t)a * nloc + b] * u[ib];
    }
    acc += la * s;
  }
  acc = wave_sum(acc, 64);
  if (lane == 0) g[e] = -acc;
}
void launch_cell_grad(int64_t ncells, int nloc, const int* cells, const double* Ke, int64_t ke_stride,
                      const double* u, const double* lam, const unsigned char* constrained_user, double* g,
                      hipStream_t s) {
  if (ncells == 0) return;
  hipLaunchKernelGGL(k_cell_grad, dim3((unsigned)((ncells + 3) / 4)), dim3(256), 0, s, ncells, nloc, cells, Ke,
                     ke_stride, u, lam, constrained_user, g);
  check_launch("k_cell_grad");
}

// vals[s] = sum over the contributions of slot s (cell e, local pair a*nloc+b, encoded e*nloc^2 + pair) of
// kappa_e Ke_e[a,b]; constrained diagonal slots get 1.0
__global__ void k_assemble(int64_t nnz, const int64_t* __restrict__ sp, const int64_t* __restrict__ contrib,
                           const double* __restrict__ kappa, const double* __restrict__ Ke, int64_t ke_stride,
                           int nloc, const unsigned char* __restrict__ diag_one, double* vals) {
  const int64_t s = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (s >= nnz) return;
  const bool one = diag_one[s];
  const int64_t m0 = sp[s], m1 = sp[s + 1];
  const int64_t nl2 = (int64_t)nloc * nloc;
  double acc = 0;
  // four contributions at a time, their loads issued together from clamped indices, summed in order
  for (int64_t m = m0; m < m1; m += 4) {
    int64_t code[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) code[u] = contrib[min(m + u, m1 - 1)];
    double kv[4], kev[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t e = code[u] / nl2, pr = code[u] - e * nl2;
      kv[u] = kappa[e];
      kev[u] = Ke[e * ke_stride + pr];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (m + u < m1) acc += kv[u] * kev[u];
  }
  vals[s] = one ? 1.0 : acc;
}
void launch_assemble(int64_t nnz, const int64_t* slot_ptr, const int64_t* contrib, const double* kappa,
                     const double* Ke, int64_t ke_stride, int nloc, const unsigned char* diag_one, double* vals,
                     hipStream_t s) {
  if (nnz == 0) return;
  hipLaunchKernelGGL(k_assemble, dim3((unsigned)((nnz + 255) / 256)), dim3(256), 0, s, nnz, slot_ptr, contrib, kappa,
                     Ke, ke_stride, nloc, diag_one, vals);
  check_launch("k_assemble");
}

}  // namespace r3mg
