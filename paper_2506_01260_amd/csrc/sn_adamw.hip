// The modified AdamW step of Sec. 5 (and the standard step it modifies).
//
// W (rows x cols, stored [out, in]: the paper's W_p2 transposed, so the
// paper's rows are the stored columns), its gradient G, first and second
// moments M and V (fp32):
//   M <- b1 M + (1 - b1) G,  V <- b2 V + (1 - b2) G^2
//   M^ = M / (1 - b1^t),     V^ = V / (1 - b2^t)
//   subspace:  alpha_c = 1 / (sqrt(mean over the column's rows of V^) + eps)
//   standard:  alpha   = 1 / (sqrt(V^) + eps) entry by entry
//   W <- W - lr alpha M^ - wd W
// A column-constant alpha scales each column of M^ by one number, so a W
// whose columns lie in S stays there when the gradients' columns do (Sec. 5,
// App. A): no projection is needed for W_p2.
//
// Memory-bound.  A thread owns 8 consecutive columns (16-byte loads of bf16
// G / W, 32-byte loads of M and V) over a few rows; the loads of many waves
// in flight, not the work per thread, set the speed.  Standard: one pass
// (22 bytes per bf16 element), 256 column threads x 4 rows per workgroup.
// Subspace: pass 1 updates V and writes per-block column sums of it (a
// workgroup is 64 column threads x 4 row groups of 8 rows, its 32-row column
// sums added across the row groups in LDS in a fixed order); pass 2 adds the
// blocks in a fixed order and forms alpha; pass 3 reads G again, updates M
// and W (24 bytes per element: G is read twice, M once).
// M, V and W are loaded and stored non-temporally (each is touched once per
// step) and G normally, so the Infinity Cache keeps G for pass 3's second
// read: subspace step on 4096 x 14336 bf16 298 -> 274 us, standard 252 -> 248.
#include "sn_device.h"
#include "sn_internal.h"

namespace sn {

namespace {

constexpr int kCols = 8;      // columns per thread
// workgroup geometry: column threads x row groups, rows per thread
constexpr int kStdCT = 256, kStdRG = 1, kStdR = 4;  // standard step
constexpr int kSubCT = 64, kSubRG = 4, kSubR = 8;   // subspace step (32-row blocks)
constexpr int kSubRows = kSubRG * kSubR;            // rows per column-sum block
constexpr int kAlphaWaves = 8;

struct AdamArgs {
  float b1, omb1, b2, omb2;   // beta1, 1 - beta1, beta2, 1 - beta2
  float inv_bc1, inv_bc2;     // 1 / (1 - beta^t)
  float lr, eps, wd;
};

template <typename T> struct Vec8;
// NT: non-temporal access (cache-policy hint), for data touched once per step.
template <typename V, bool NT>
__device__ __forceinline__ V ld_vec(const V *p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  return *p;
}
template <typename V, bool NT>
__device__ __forceinline__ void st_vec(V *p, V v) {
  if constexpr (NT)
    __builtin_nontemporal_store(v, p);
  else
    *p = v;
}

template <> struct Vec8<bf16_t> {
  template <bool NT>
  static __device__ __forceinline__ void load(const bf16_t *p, float (&x)[8]) {
    const u32x4 v = ld_vec<u32x4, NT>(reinterpret_cast<const u32x4 *>(p));
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = bf_lo(w[i]);
      x[2 * i + 1] = bf_hi(w[i]);
    }
  }
  template <bool NT>
  static __device__ __forceinline__ void store(bf16_t *p, const float (&x)[8]) {
    st_vec<u32x4, NT>(reinterpret_cast<u32x4 *>(p),
                      u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]),
                            pack_bf16x2(x[4], x[5]), pack_bf16x2(x[6], x[7])});
  }
};
template <> struct Vec8<float> {
  template <bool NT>
  static __device__ __forceinline__ void load(const float *p, float (&x)[8]) {
    const f32x4 a = ld_vec<f32x4, NT>(reinterpret_cast<const f32x4 *>(p));
    const f32x4 b = ld_vec<f32x4, NT>(reinterpret_cast<const f32x4 *>(p + 4));
    x[0] = a.x; x[1] = a.y; x[2] = a.z; x[3] = a.w;
    x[4] = b.x; x[5] = b.y; x[6] = b.z; x[7] = b.w;
  }
  template <bool NT>
  static __device__ __forceinline__ void store(float *p, const float (&x)[8]) {
    st_vec<f32x4, NT>(reinterpret_cast<f32x4 *>(p), f32x4{x[0], x[1], x[2], x[3]});
    st_vec<f32x4, NT>(reinterpret_cast<f32x4 *>(p + 4), f32x4{x[4], x[5], x[6], x[7]});
  }
};

// 8 columns of one row: vector access when VEC (cols % 8 == 0, 16-byte
// aligned rows), else element by element with a bound on the column
template <typename T, bool VEC, bool NT = false>
__device__ __forceinline__ void load8(const T *row, int64_t c0, int64_t cols, float (&x)[8]) {
  if constexpr (VEC) {
    Vec8<T>::template load<NT>(row + c0, x);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = c0 + i < cols ? to_f32(row[c0 + i]) : 0.0f;
  }
}

template <typename T, bool VEC, bool NT = false>
__device__ __forceinline__ void store8(T *row, int64_t c0, int64_t cols, const float (&x)[8]) {
  if constexpr (VEC) {
    Vec8<T>::template store<NT>(row + c0, x);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (c0 + i < cols) row[c0 + i] = from_f32<T>(x[i]);
  }
}

// Pass 1 (and the whole standard step when !SUB): the second moment and
// either its column sums (SUB) or the first moment and the W update with the
// entrywise rate.  Thread (x, y) of the workgroup: columns 8 x .. 8 x + 7 of
// the workgroup's column block, rows R y .. R y + R - 1 of its row block.
template <typename T, bool VEC, bool SUB, int CT, int RG, int R>
__global__ __launch_bounds__(CT * RG) void moments_kernel(T *__restrict__ W, int64_t ldw,
                                                           const T *__restrict__ G, int64_t ldg,
                                                           float *__restrict__ M,
                                                           float *__restrict__ V, int64_t ldm,
                                                           int64_t rows, int64_t cols, AdamArgs a,
                                                           float *__restrict__ colsum) {
  __shared__ float red[SUB ? RG : 1][SUB ? CT * kCols : 1];
  const int tx = threadIdx.x % CT, ty = threadIdx.x / CT;
  const int64_t c0 = (static_cast<int64_t>(blockIdx.x) * CT + tx) * kCols;
  const bool live = c0 < cols;
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * (RG * R) + ty * R;
  const int64_t r1 = !live ? r0 : (r0 + R < rows ? r0 + R : (r0 < rows ? rows : r0));
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  auto row = [&](int64_t r) {
    float g[8], v[8];
    load8<T, VEC>(G + r * ldg, c0, cols, g);
    load8<float, VEC, true>(V + r * ldm, c0, cols, v);
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = fmaf(a.b2, v[i], a.omb2 * (g[i] * g[i]));
    store8<float, VEC, true>(V + r * ldm, c0, cols, v);
    if constexpr (SUB) {
#pragma unroll
      for (int i = 0; i < 8; ++i) s[i] += v[i];
    } else {
      float m[8], w[8];
      load8<float, VEC, true>(M + r * ldm, c0, cols, m);
#pragma unroll
      for (int i = 0; i < 8; ++i) m[i] = fmaf(a.b1, m[i], a.omb1 * g[i]);
      store8<float, VEC, true>(M + r * ldm, c0, cols, m);
      load8<T, VEC, true>(W + r * ldw, c0, cols, w);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float alpha = 1.0f / (sqrtf(v[i] * a.inv_bc2) + a.eps);
        w[i] = w[i] - a.lr * alpha * (m[i] * a.inv_bc1) - a.wd * w[i];
      }
      store8<T, VEC, true>(W + r * ldw, c0, cols, w);
    }
  };
  // a full run of R rows is unrolled as one block (all its loads in flight
  // together); a short run at the bottom edge goes row by row
  if (r1 - r0 == R) {
#pragma unroll
    for (int j = 0; j < R; ++j) row(r0 + j);
  } else {
    for (int64_t r = r0; r < r1; ++r) row(r);
  }
  if constexpr (SUB) {
    // the row groups' sums of each column, added in row order
#pragma unroll
    for (int i = 0; i < 8; ++i) red[ty][tx * kCols + i] = s[i];
    __syncthreads();
    if (ty == 0 && live) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float t = red[0][tx * kCols + i];
#pragma unroll
        for (int y = 1; y < RG; ++y) t += red[y][tx * kCols + i];
        s[i] = t;
      }
      float *dst = colsum + static_cast<int64_t>(blockIdx.y) * cols;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (c0 + i < cols) dst[c0 + i] = s[i];
    }
  }
}

// Pass 2: alpha_c = 1 / (sqrt(sum_blocks colsum / (rows (1 - b2^t))) + eps), the
// row blocks added in float64: wave w of a workgroup the blocks w, w + 8, ...
// of its 64 columns, then the waves in order.  One thread per column left a
// chain of 128 loads on 112 workgroups: 11.9 -> 4.8 us at 4096 x 14336.
__global__ __launch_bounds__(64 * kAlphaWaves) void alpha_kernel(
    const float *__restrict__ colsum, int64_t nblk, int64_t rows, int64_t cols, double inv_bc2,
    double eps, float *__restrict__ alpha) {
  __shared__ double red[kAlphaWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t c = (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x) * 64 + lane;
  double s = 0.0;
  if (c < cols) {
#pragma unroll 8
    for (int64_t b = w; b < nblk; b += kAlphaWaves) s += static_cast<double>(colsum[b * cols + c]);
  }
  red[w][lane] = s;
  __syncthreads();
  if (w != 0 || c >= cols) return;
#pragma unroll
  for (int i = 1; i < kAlphaWaves; ++i) s += red[i][lane];
  const double nu = s * inv_bc2 / static_cast<double>(rows);
  alpha[c] = static_cast<float>(1.0 / (sqrt(nu) + eps));
}

// Pass 3: M <- b1 M + (1 - b1) G, then W <- W - lr alpha_c M^ - wd W with
// the column's rate (the geometry of pass 1).
template <typename T, bool VEC, int CT, int RG, int R>
__global__ __launch_bounds__(CT * RG) void apply_kernel(T *__restrict__ W, int64_t ldw,
                                                         const T *__restrict__ G, int64_t ldg,
                                                         float *__restrict__ M, int64_t ldm,
                                                         int64_t rows, int64_t cols, AdamArgs a,
                                                         const float *__restrict__ alpha) {
  const int tx = threadIdx.x % CT, ty = threadIdx.x / CT;
  const int64_t c0 = (static_cast<int64_t>(blockIdx.x) * CT + tx) * kCols;
  if (c0 >= cols) return;
  const int64_t r0 = static_cast<int64_t>(blockIdx.y) * (RG * R) + ty * R;
  const int64_t r1 = r0 + R < rows ? r0 + R : (r0 < rows ? rows : r0);
  float al[8];
  load8<float, VEC>(alpha, c0, cols, al);
#pragma unroll
  for (int i = 0; i < 8; ++i) al[i] *= a.lr * a.inv_bc1;
  auto row = [&](int64_t r) {
    float g[8], m[8], w[8];
    load8<T, VEC>(G + r * ldg, c0, cols, g);
    load8<float, VEC, true>(M + r * ldm, c0, cols, m);
    load8<T, VEC, true>(W + r * ldw, c0, cols, w);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      m[i] = fmaf(a.b1, m[i], a.omb1 * g[i]);
      w[i] = w[i] - al[i] * m[i] - a.wd * w[i];
    }
    store8<float, VEC, true>(M + r * ldm, c0, cols, m);
    store8<T, VEC, true>(W + r * ldw, c0, cols, w);
  };
  if (r1 - r0 == R) {
#pragma unroll
    for (int j = 0; j < R; ++j) row(r0 + j);
  } else {
    for (int64_t r = r0; r < r1; ++r) row(r);
  }
}

template <typename T, bool VEC>
hipError_t launch_t(void *Wv, int64_t ldw, const void *Gv, int64_t ldg, float *M, float *V,
                    int64_t ldm, int64_t rows, int64_t cols, const AdamArgs &a, double inv_bc2,
                    double eps, bool sub, void *ws, hipStream_t s) {
  T *W = static_cast<T *>(Wv);
  const T *G = static_cast<const T *>(Gv);
  if (!sub) {
    const dim3 grid(static_cast<unsigned>(ceil_div(cols, kStdCT * kCols)),
                    static_cast<unsigned>(ceil_div(rows, kStdRG * kStdR)));
    moments_kernel<T, VEC, false, kStdCT, kStdRG, kStdR><<<grid, kStdCT * kStdRG, 0, s>>>(
        W, ldw, G, ldg, M, V, ldm, rows, cols, a, nullptr);
    return hipGetLastError();
  }
  const dim3 grid(static_cast<unsigned>(ceil_div(cols, kSubCT * kCols)),
                  static_cast<unsigned>(ceil_div(rows, kSubRows)));
  float *colsum = static_cast<float *>(ws);
  float *alpha = colsum + static_cast<int64_t>(grid.y) * cols;
  moments_kernel<T, VEC, true, kSubCT, kSubRG, kSubR><<<grid, kSubCT * kSubRG, 0, s>>>(
      W, ldw, G, ldg, M, V, ldm, rows, cols, a, colsum);
  // a grid dimension holds fewer than 2^32 threads, 2^23 of these workgroups
  const int64_t groups = ceil_div(cols, 64), gx = groups < (1 << 22) ? groups : 1 << 22;
  const dim3 ga(static_cast<unsigned>(gx), static_cast<unsigned>(ceil_div(groups, gx)));
  alpha_kernel<<<ga, 64 * kAlphaWaves, 0, s>>>(
      colsum, grid.y, rows, cols, inv_bc2, eps, alpha);
  apply_kernel<T, VEC, kSubCT, kSubRG, kSubR><<<grid, kSubCT * kSubRG, 0, s>>>(
      W, ldw, G, ldg, M, ldm, rows, cols, a, alpha);
  return hipGetLastError();
}

bool a16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

}  // namespace

size_t adamw_workspace_bytes(int64_t rows, int64_t cols) {
  // column sums per block of kSubRows rows, then the rates (fp32)
  return align256(static_cast<size_t>(ceil_div(rows, kSubRows) + 1) * cols * sizeof(float));
}

hipError_t launch_adamw(int dt, void *W, int64_t ldw, const void *G, int64_t ldg, float *M,
                        float *V, int64_t ldm, int64_t rows, int64_t cols, int64_t t, double lr,
                        double beta1, double beta2, double eps, double wd, bool subspace,
                        void *ws, hipStream_t s) {
  const double bc1 = 1.0 - pow(beta1, static_cast<double>(t));
  const double bc2 = 1.0 - pow(beta2, static_cast<double>(t));
  AdamArgs a;
  a.b1 = static_cast<float>(beta1);
  a.omb1 = static_cast<float>(1.0 - beta1);
  a.b2 = static_cast<float>(beta2);
  a.omb2 = static_cast<float>(1.0 - beta2);
  a.inv_bc1 = static_cast<float>(1.0 / bc1);
  a.inv_bc2 = static_cast<float>(1.0 / bc2);
  a.lr = static_cast<float>(lr);
  a.eps = static_cast<float>(eps);
  a.wd = static_cast<float>(wd);
  const size_t es = dt == 0 ? 4 : 2;
  const bool vec = cols % kCols == 0 && a16(W) && a16(G) && a16(M) && a16(V) &&
                   (ldw * es) % 16 == 0 && (ldg * es) % 16 == 0 && (ldm * 4) % 16 == 0 &&
                   a16(ws);
  if (dt == 0)
    return vec ? launch_t<float, true>(W, ldw, G, ldg, M, V, ldm, rows, cols, a, 1.0 / bc2, eps,
                                       subspace, ws, s)
               : launch_t<float, false>(W, ldw, G, ldg, M, V, ldm, rows, cols, a, 1.0 / bc2, eps,
                                        subspace, ws, s);
  return vec ? launch_t<bf16_t, true>(W, ldw, G, ldg, M, V, ldm, rows, cols, a, 1.0 / bc2, eps,
                                      subspace, ws, s)
             : launch_t<bf16_t, false>(W, ldw, G, ldg, M, V, ldm, rows, cols, a, 1.0 / bc2, eps,
                                       subspace, ws, s);
}

}  // namespace sn
