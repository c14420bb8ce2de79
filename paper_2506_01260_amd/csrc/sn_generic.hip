// Basis packing and the generic codec kernels (float64 matrix cores).
//
// The generic kernels handle every shape, stride and dtype the ABI accepts:
// all float32 work, and bf16 work that does not meet the bf16 MFMA kernels'
// alignment / size conditions.  Products and sums are float64 (a float32
// product is exact there), rounded once to the output type, so float32
// results stay within a rounding of the exact value even when the sum cancels.
//
// v_mfma_f64_16x16x4_f64 (wave64): lane l = 16 g + n supplies A[n][g] and
// B[g][n] and receives D[4 i + g][n], i = 0..3.  The contraction indices may
// be dealt to (step, g) in any order, as long as A and B agree.
#include <type_traits>

#include "sn_device.h"
#include "sn_internal.h"

namespace sn {

// A grid dimension holds fewer than 2^32 threads, and a grid past that is cut off
// without an error: workgroup counts that follow the tokens or columns are laid
// over x and another dimension.
constexpr int64_t kGridX = int64_t{1} << 21;
inline int64_t grid_x(int64_t groups) { return groups < kGridX ? groups : kGridX; }
inline unsigned grid_more(int64_t groups) {
  return static_cast<unsigned>(ceil_div(groups, grid_x(groups)));
}

// ---------------------------------------------------------------------------
// Packing
// ---------------------------------------------------------------------------

PackLayout pack_layout(int64_t d, int64_t k, int dt) {
  PackLayout L;
  L.d = d;
  L.k = k;
  L.dt = dt;
  L.kt = static_cast<int>(ceil_div(k, 16));
  L.ks = static_cast<int>(ceil_div(k, 32));
  L.mfma = (dt == 1) && (d % 32 == 0) && (L.kt <= kMfmaMaxKT);
  size_t off = 0;
  L.off_f32 = off;
  off = align256(off + static_cast<size_t>(d) * k * 4);
  L.off_kfrag32 = off;
  off = align256(off + static_cast<size_t>(ceil_div(d, 32)) * L.kt * 2048);
  L.off_rfrag32 = off;
  off = align256(off + static_cast<size_t>(ceil_div(d, 16)) * L.kt * 1024);
  if (L.mfma) {
    L.off_kfrag = off;
    off = align256(off + static_cast<size_t>(d / 32) * L.kt * 1024);
    L.off_rfrag = off;
    off = align256(off + static_cast<size_t>(d / 32) * 2 * L.ks * 1024);
    if (k <= 64) {
      L.ks2 = static_cast<int>(ceil_div(2 * k, 32));
      L.off_uu = off;
      off = align256(off + static_cast<size_t>(d) * 32 * L.ks2 * 2);
    }
  }
  L.off_gram = off;
  off = align256(off + static_cast<size_t>(16 * L.kt) * (16 * L.kt) * 8);
  L.total = off;
  return L;
}

template <typename T>
__device__ __forceinline__ void pack_f32(int64_t idx, const T *__restrict__ U, int64_t d,
                                         int64_t k, int64_t ldu, float *__restrict__ out) {
  if (idx >= d * k) return;
  int64_t r = idx / k, j = idx - r * k;
  out[idx] = to_f32(U[r * ldu + j]);
}

// The float32 fragment sections, one thread per 16-byte slot: kfrag32 slots
// first, then rfrag32's.
template <typename T>
__device__ __forceinline__ void pack_frag32(int64_t slot, const T *__restrict__ U, int64_t d,
                                            int64_t k, int64_t ldu, int kt,
                                            f32x4 *__restrict__ kfrag,
                                            f32x4 *__restrict__ rfrag) {
  const int64_t nk = (d + 31) / 32 * kt * 128, nr = (d + 15) / 16 * kt * 64;
  const bool second = slot >= nk;
  if (second) slot -= nk;
  if (second && slot >= nr) return;
  const int lane = static_cast<int>(slot & 63), g = lane >> 4, n = lane & 15;
  f32x4 v;
  // 16-row blocks x column tiles: below 2^32, and a 32-bit division
  const unsigned blk = static_cast<unsigned>(second ? slot >> 6 : slot >> 7);
  const int64_t rb = blk / static_cast<unsigned>(kt), t = blk % static_cast<unsigned>(kt);
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    int64_t row, col;
    if (!second) {
      row = 32 * rb + 8 * g + 4 * ((slot >> 6) & 1) + e;
      col = 16 * t + n;
    } else {
      row = 16 * rb + 4 * (n & 3) + (n >> 2);
      col = 16 * t + 4 * e + g;
    }
    v[e] = row < d && col < k ? to_f32(U[row * ldu + col]) : 0.0f;
  }
  (second ? rfrag : kfrag)[slot] = v;
}

// One thread per 8-element lane slot of a 1 KiB fragment block.
__device__ __forceinline__ void pack_kfrag(int64_t slot, const bf16_t *__restrict__ U, int64_t d,
                                           int64_t k, int64_t ldu, int kt,
                                           bf16_t *__restrict__ out) {
  int64_t nblk = (d / 32) * kt;
  if (slot >= nblk * 64) return;
  int64_t blk = slot >> 6;
  int lane = static_cast<int>(slot & 63);
  int64_t s = blk / kt;
  int t = static_cast<int>(blk - s * kt);
  int g = lane >> 4, n = lane & 15;
  int64_t col = 16 * t + n;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    int64_t row = 32 * s + 8 * g + e;
    out[slot * 8 + e] = col < k ? U[row * ldu + col] : bf16_t(0);
  }
}

__device__ __forceinline__ void pack_rfrag(int64_t slot, const bf16_t *__restrict__ U, int64_t d,
                                           int64_t k, int64_t ldu, int ks,
                                           bf16_t *__restrict__ out) {
  int64_t nblk = (d / 32) * 2 * ks;
  if (slot >= nblk * 64) return;
  int64_t blk = slot >> 6;
  int lane = static_cast<int>(slot & 63);
  int q = static_cast<int>(blk % ks);
  int h = static_cast<int>((blk / ks) & 1);
  int64_t p = blk / (2 * ks);
  int g = lane >> 4, m = lane & 15;
  int64_t row = 32 * p + 8 * (m >> 2) + 4 * h + (m & 3);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    int64_t col = 32 * q + 8 * g + e;
    out[slot * 8 + e] = col < k ? U[row * ldu + col] : bf16_t(0);
  }
}

// [U | U] with zero columns up to 32 ks2, one thread per element.
__device__ __forceinline__ void pack_uu(int64_t idx, const bf16_t *__restrict__ U, int64_t d,
                                        int64_t k, int64_t ldu, int ks2,
                                        bf16_t *__restrict__ out) {
  const int w = 32 * ks2;
  if (idx >= d * w) return;
  const int64_t r = idx / w;
  const int64_t j = idx - r * w;
  out[idx] = j < 2 * k ? U[r * ldu + (j < k ? j : j - k)] : bf16_t(0);
}

// Every section that is a copy of U, in one launch: each takes a range of the
// workgroups.  With a launch per section the float32 operand sections made every
// pack 3 to 5 us longer (back to back d = 256, k = 8, float32 10.9 -> 15.0 us; d = 4096,
// k = 40, bf16 31.0 -> 34.0); in one launch 12.1 and 25.5, with the Gram matrix.
struct PackSections {
  float *f32;
  f32x4 *kfrag32, *rfrag32;
  bf16_t *kfrag, *rfrag, *uu;
  int64_t end[5];  // workgroups up to and with f32, the float32 operands, kfrag, rfrag, uu
};

template <typename T>
__global__ __launch_bounds__(256) void pack_kernel(const T *__restrict__ U, int64_t d, int64_t k,
                                                   int64_t ldu, int kt, int ks, int ks2,
                                                   PackSections p) {
  const int64_t wg = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
  auto at = [&](int i) { return (wg - (i > 0 ? p.end[i - 1] : 0)) * 256 + threadIdx.x; };
  if (wg < p.end[0])
    pack_f32(at(0), U, d, k, ldu, p.f32);
  else if (wg < p.end[1])
    pack_frag32(at(1), U, d, k, ldu, kt, p.kfrag32, p.rfrag32);
  else if constexpr (sizeof(T) == 2) {
    if (wg < p.end[2])
      pack_kfrag(at(2), U, d, k, ldu, kt, p.kfrag);
    else if (wg < p.end[3])
      pack_rfrag(at(3), U, d, k, ldu, ks, p.rfrag);
    else if (wg < p.end[4])
      pack_uu(at(4), U, d, k, ldu, ks2, p.uu);
  }
}

// U^T U - I from the float32 section (exact copies of the stored U), as a
// kp x kp matrix (kp = 16 ceil(k/16) <= 256, zero outside k x k).  One
// workgroup per row a; thread (h, b) sums U[r, a] U[r, b] in float64 over the
// rows r = h mod H (H = 1024 / kp row phases, reads coalesced along b), and
// the H partial sums are added in a fixed order.
constexpr int kGramThreads = 1024;
__global__ __launch_bounds__(kGramThreads) void pack_gram_kernel(const float *__restrict__ U32,
                                                                 int64_t d, int64_t k, int64_t kp,
                                                                 double *__restrict__ out) {
  __shared__ double red[kGramThreads];
  const int64_t a = blockIdx.x;
  const int H = static_cast<int>(kGramThreads / kp);
  const int h = static_cast<int>(threadIdx.x / kp), b = static_cast<int>(threadIdx.x % kp);
  double acc = 0.0;
  if (a < k && h < H && b < k) {
#pragma unroll 4
    for (int64_t r = h; r < d; r += H)
      acc += static_cast<double>(U32[r * k + a]) * static_cast<double>(U32[r * k + b]);
  }
  red[threadIdx.x] = acc;
  __syncthreads();
  if (threadIdx.x < kp) {
    double v = 0.0;
    for (int hh = 0; hh < H; ++hh) v += red[hh * kp + threadIdx.x];
    const bool in = a < k && static_cast<int64_t>(threadIdx.x) < k;
    out[a * kp + threadIdx.x] = in ? v - (a == static_cast<int64_t>(threadIdx.x) ? 1.0 : 0.0)
                                   : 0.0;
  }
}

hipError_t launch_pack(const PackLayout &L, const void *U, int64_t ldu, void *packed,
                       hipStream_t s) {
  char *base = static_cast<char *>(packed);
  PackSections p{};
  p.f32 = reinterpret_cast<float *>(base + L.off_f32);
  p.kfrag32 = reinterpret_cast<f32x4 *>(base + L.off_kfrag32);
  p.rfrag32 = reinterpret_cast<f32x4 *>(base + L.off_rfrag32);
  // threads of each section: an element, or a 16-byte slot
  int64_t n[5] = {L.d * L.k, ceil_div(L.d, 32) * L.kt * 128 + ceil_div(L.d, 16) * L.kt * 64, 0, 0,
                  0};
  if (L.mfma) {
    p.kfrag = reinterpret_cast<bf16_t *>(base + L.off_kfrag);
    p.rfrag = reinterpret_cast<bf16_t *>(base + L.off_rfrag);
    n[2] = (L.d / 32) * L.kt * 64;
    n[3] = (L.d / 32) * 2 * L.ks * 64;
    if (L.ks2 > 0) {
      p.uu = reinterpret_cast<bf16_t *>(base + L.off_uu);
      n[4] = L.d * 32 * L.ks2;
    }
  }
  int64_t wgs = 0;
  for (int i = 0; i < 5; ++i) p.end[i] = wgs += ceil_div(n[i], 256);
  // (8 threads per row and column tile alone outgrow a grid dimension above 2^29 rows)
  const dim3 grid(static_cast<unsigned>(grid_x(wgs)), grid_more(wgs));
  if (L.dt == 0)
    pack_kernel<float><<<grid, 256, 0, s>>>(static_cast<const float *>(U), L.d, L.k, ldu, L.kt,
                                            L.ks, L.ks2, p);
  else
    pack_kernel<bf16_t><<<grid, 256, 0, s>>>(static_cast<const bf16_t *>(U), L.d, L.k, ldu, L.kt,
                                             L.ks, L.ks2, p);
  const int64_t kp = 16 * L.kt;
  pack_gram_kernel<<<dim3(static_cast<unsigned>(kp)), kGramThreads, 0, s>>>(
      reinterpret_cast<const float *>(base + L.off_f32), L.d, L.k, kp,
      reinterpret_cast<double *>(base + L.off_gram));
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Helpers of the float64 matrix-core kernels
// ---------------------------------------------------------------------------

typedef double f64x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f64x4 mfma64(double a, double b, f64x4 c) {
  return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <typename T> __device__ __forceinline__ T from_f64(double v);
template <> __device__ __forceinline__ float from_f64<float>(double v) {
  return static_cast<float>(v);
}
template <> __device__ __forceinline__ bf16_t from_f64<bf16_t>(double v) {
  return bf16_from_f64(v);
}

// 8 consecutive elements of a row as two vectors; rows need only be aligned
// to their element size (the memory pipeline takes unaligned vector loads).
template <typename T> struct Row8;
template <> struct Row8<float> {
  typedef float v4 __attribute__((ext_vector_type(4), aligned(4)));
  v4 a, b;
  __device__ __forceinline__ void load(const float *p) {
    a = *reinterpret_cast<const v4 *>(p);
    b = *reinterpret_cast<const v4 *>(p + 4);
  }
  __device__ __forceinline__ double at(int i) const { return i < 4 ? a[i & 3] : b[i & 3]; }
};
template <> struct Row8<bf16_t> {
  typedef uint32_t v4 __attribute__((ext_vector_type(4), aligned(2)));
  v4 a;
  __device__ __forceinline__ void load(const bf16_t *p) { a = *reinterpret_cast<const v4 *>(p); }
  __device__ __forceinline__ double at(int i) const {
    const uint32_t w = a[i >> 1];
    return (i & 1) ? bf_hi(w) : bf_lo(w);
  }
};

// 4 consecutive elements, element-aligned
template <typename T> struct Row4;
template <> struct Row4<float> {
  typedef float v4 __attribute__((ext_vector_type(4), aligned(4)));
  v4 a;
  __device__ __forceinline__ void load(const float *p) { a = *reinterpret_cast<const v4 *>(p); }
  __device__ __forceinline__ double at(int i) const { return a[i]; }
  static __device__ __forceinline__ void store(float *p, f64x4 v) {
    *reinterpret_cast<v4 *>(p) = v4{static_cast<float>(v.x), static_cast<float>(v.y),
                                    static_cast<float>(v.z), static_cast<float>(v.w)};
  }
};
template <> struct Row4<bf16_t> {
  typedef uint32_t v2 __attribute__((ext_vector_type(2), aligned(2)));
  v2 a;
  __device__ __forceinline__ void load(const bf16_t *p) { a = *reinterpret_cast<const v2 *>(p); }
  __device__ __forceinline__ double at(int i) const {
    const uint32_t w = a[i >> 1];
    return (i & 1) ? bf_hi(w) : bf_lo(w);
  }
  static __device__ __forceinline__ void store(bf16_t *p, f64x4 v) {
    uint32_t h[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) h[i] = bf16_from_f64(v[i]);
    *reinterpret_cast<v2 *>(p) = v2{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
  }
};

// Token and positional rows of token i; a missing table gives the row `none`
// (any readable row of d elements, whose values are not used).
template <typename T>
struct Rows {
  const T *e, *p;
};
template <typename T>
__device__ __forceinline__ Rows<T> resolve_rows(int64_t i, const IdArgs &a, const T *none) {
  Rows<T> r{none, none};
  if (a.E) {
    int64_t t = clamp_id(a.tok[i], a.vocab, a.err_flag, 1);
    r.e = static_cast<const T *>(a.E) + t * a.lde;
  }
  if (a.P) {
    int64_t p = a.pos ? static_cast<int64_t>(a.pos[i]) : i % a.seq_len;
    p = clamp_id(p, a.n_pos, a.err_flag, 2);
    r.p = static_cast<const T *>(a.P) + p * a.ldp;
  }
  return r;
}

// ---------------------------------------------------------------------------
// Compress: (X - P - E) U for 16 tokens per workgroup, the NW waves taking
// every NW-th unit of 32 columns of d and adding their sums through LDS in
// wave order.  X - P - E is formed in float64 (no rounding that float32 could
// see), one f64 MFMA per 4 columns and 16 columns of U.
//
// Bound by the f64 matrix rate (75 TFLOP/s measured in a loop of MFMAs) from
// k ~ 16 up, below that by HBM.  16-token tiles alone leave the chip idle
// below ~16000 tokens, hence the split of d over the waves; a unit's loads (16
// rows x 128 contiguous bytes) keep whole cache lines, and a wave's rows of
// the next unit are loaded while it multiplies.  8192 tokens, d = 2048,
// k = 20, float32: 355 us (one wave per token on the vector ALU, compensated
// sums) -> 21 us, MFMAs alone 14.
// ---------------------------------------------------------------------------

// What becomes of the sums: the output type (after subtracting projected rows
// if there are any), fp32 rows of a projected table (ldc = its padded width,
// zero past k), or float64 rows.
enum GenOut { kGenT = 0, kGenTable = 1, kGenF64 = 2 };

template <typename T, int KT, int NW, bool TAB>
__global__ __launch_bounds__(64 * NW) void compress_f64_kernel(
    const f32x4 *__restrict__ kfrag, int kt, int64_t d, int64_t k, const T *__restrict__ X,
    int64_t N, int64_t ldx, IdArgs ids, ProjArgs pa, int mode, void *__restrict__ out,
    int64_t ldc) {
  constexpr int TC = 16 / NW < KT ? 16 / NW : KT;  // column tiles reduced at a time (32 KiB)
  __shared__ double red[NW][TC][64][4];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, n = lane & 15;
  const int64_t i0 = 16 * (static_cast<int64_t>(blockIdx.z) * gridDim.x + blockIdx.x);
  if (i0 >= N) return;
  const int64_t i = i0 + n < N ? i0 + n : N - 1;  // rows past N repeat the last, not stored
  const int t0 = static_cast<int>(blockIdx.y) * KT;  // first column tile
  const T *xr = X + i * ldx;
  Rows<T> rw{};
  if constexpr (TAB) rw = resolve_rows<T>(i, ids, xr);
  const bool he = TAB && ids.E, hp = TAB && ids.P;

  f64x4 acc[KT];
#pragma unroll
  for (int t = 0; t < KT; ++t) acc[t] = f64x4{0., 0., 0., 0.};

  auto frag = [&](int u, int t, int h) {
    const int tt = t0 + t < kt ? t0 + t : kt - 1;  // tiles past the last are not stored
    return kfrag[((static_cast<int64_t>(u) * kt + tt) * 2 + h) * 64 + lane];
  };
  // a lane's 8 columns 32 u + 8 g .. + 7 of its rows and, while they are few,
  // the unit's U fragments
  constexpr bool kPre = KT <= 2;
  struct Unit {
    Row8<T> x, e, p;
    f32x4 a[kPre ? KT : 1][2];
  };
  auto load = [&](Unit &v, int u) {
    const int64_t c = 32 * static_cast<int64_t>(u) + 8 * g;
    v.x.load(xr + c);
    if constexpr (TAB) {
      v.e.load(rw.e + c);
      v.p.load(rw.p + c);
    }
    if constexpr (kPre) {
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) v.a[t][h] = frag(u, t, h);
    }
  };
  auto value = [&](const Unit &v, int j) {
    double x = v.x.at(j);
    if constexpr (TAB) {
      const double p = v.p.at(j), e = v.e.at(j);
      x -= hp ? p : 0.0;
      x -= he ? e : 0.0;
    }
    return x;
  };
  auto step = [&](const Unit &v, int u) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      f32x4 a[KT];
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        if constexpr (kPre)
          a[t] = v.a[t][h];
        else
          a[t] = frag(u, t, h);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double b = value(v, 4 * h + e);
#pragma unroll
        for (int t = 0; t < KT; ++t) acc[t] = mfma64(static_cast<double>(a[t][e]), b, acc[t]);
      }
    }
  };

  const int nfull = static_cast<int>(d / 32);
  if (wave < nfull) {
    Unit cur, nxt;
    load(cur, wave);
    for (int u = wave; u < nfull; u += NW) {
      load(nxt, u + NW < nfull ? u + NW : u);  // past the end the unit repeats, unused
      step(cur, u);
      cur = nxt;
    }
  }
  if (d % 32 != 0 && wave == nfull % NW) {  // the last, partial unit: zero past column d
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int64_t c = 32 * static_cast<int64_t>(nfull) + 8 * g + j;
      double x = 0.0;
      if (c < d) {
        x = to_f32(xr[c]);
        if (hp) x -= static_cast<double>(to_f32(rw.p[c]));
        if (he) x -= static_cast<double>(to_f32(rw.e[c]));
      }
#pragma unroll
      for (int t = 0; t < KT; ++t)
        acc[t] = mfma64(static_cast<double>(frag(nfull, t, j >> 2)[j & 3]), x, acc[t]);
    }
  }

  // lane (g, n) holds columns 16 t + 4 i + g of token n
#pragma unroll
  for (int tc = 0; tc < KT; tc += TC) {
    if (tc > 0) __syncthreads();
#pragma unroll
    for (int t = 0; t < TC; ++t)
      if (tc + t < KT) {
#pragma unroll
        for (int q = 0; q < 4; ++q) red[wave][t][lane][q] = acc[tc + t < KT ? tc + t : 0][q];
      }
    __syncthreads();
    for (int idx = threadIdx.x; idx < TC * 256; idx += 64 * NW) {
      const int nn = idx / (16 * TC), jl = idx % (16 * TC);
      const int t = jl >> 4, q = (jl & 15) >> 2, gg = jl & 3;
      const int64_t j = 16 * static_cast<int64_t>(t0 + tc) + jl;
      const int64_t tok = i0 + nn;
      if (tc + t >= KT || tok >= N || j >= (mode == kGenTable ? ldc : k)) continue;
      double v = red[0][t][16 * gg + nn][q];
#pragma unroll
      for (int w = 1; w < NW; ++w) v += red[w][t][16 * gg + nn][q];
      if (mode == kGenTable) {
        static_cast<float *>(out)[tok * ldc + j] = j < k ? static_cast<float>(v) : 0.0f;
      } else if (mode == kGenF64) {
        static_cast<double *>(out)[tok * ldc + j] = v;
      } else {
        if (pa.pu) {
          int64_t p = pa.pos ? static_cast<int64_t>(pa.pos[tok]) : tok % pa.seq_len;
          v -= static_cast<double>(pa.pu[clamp_id(p, pa.n_pos, pa.err_flag, 2) * pa.kp + j]);
        }
        if (pa.eu)
          v -= static_cast<double>(
              pa.eu[clamp_id(pa.tok[tok], pa.vocab, pa.err_flag, 1) * pa.kp + j]);
        static_cast<T *>(out)[tok * ldc + j] = from_f64<T>(v);
      }
    }
  }
}

// Workgroups take KT column tiles of U each: as many as still leave a
// workgroup for every CU (a launch of few tokens splits the columns, and with
// them the MFMAs, and re-reads its rows from the caches).  Waves per
// workgroup: so many that a CU has about 16, which hide each other's loads
// behind the 64-cycle MFMAs (16 only while 128 registers hold the
// accumulators, KT <= 4).  500 tokens, d = 8192, k = 82: 109 us with all
// column tiles in one workgroup, 21.5 split; 8192 tokens: 21.3 us with 16
// waves, 21.7 with 8, 24.2 with 4.
template <typename T, int KT, bool TAB>
void launch_compress_f64(const PackLayout &L, const void *packed, const void *X, int64_t N,
                         int64_t ldx, const IdArgs &ids, const ProjArgs &pa, int mode, void *out,
                         int64_t ldc, hipStream_t s) {
  const f32x4 *kf =
      reinterpret_cast<const f32x4 *>(static_cast<const char *>(packed) + L.off_kfrag32);
  const int64_t tiles = ceil_div(N, 16);
  const dim3 grid(static_cast<unsigned>(grid_x(tiles)),
                  static_cast<unsigned>(ceil_div(L.kt, KT)), grid_more(tiles));
  const T *x = static_cast<const T *>(X);
  auto go = [&](auto nw) {
    constexpr int NW = decltype(nw)::value;
    compress_f64_kernel<T, KT, NW, TAB>
        <<<grid, 64 * NW, 0, s>>>(kf, L.kt, L.d, L.k, x, N, ldx, ids, pa, mode, out, ldc);
  };
  const int64_t groups = tiles * grid.y;
  if (KT <= 4 && groups <= 512)
    go(std::integral_constant<int, KT <= 4 ? 16 : 8>{});
  else if (groups <= 1024)
    go(std::integral_constant<int, 8>{});
  else
    go(std::integral_constant<int, 4>{});
}

template <typename T, bool TAB>
hipError_t compress_f64_kt(const PackLayout &L, const void *packed, const void *X, int64_t N,
                           int64_t ldx, const IdArgs &ids, const ProjArgs &pa, int mode, void *out,
                           int64_t ldc, hipStream_t s) {
  auto go = [&](auto kt) {
    launch_compress_f64<T, decltype(kt)::value, TAB>(L, packed, X, N, ldx, ids, pa, mode, out,
                                                     ldc, s);
    return hipGetLastError();
  };
  const int64_t tiles = ceil_div(N, 16);
  auto fits = [&](int kt) { return L.kt >= kt && tiles * ceil_div(L.kt, kt) >= 256; };
  if (fits(7)) return go(std::integral_constant<int, 8>{});
  if (fits(5)) return go(std::integral_constant<int, 6>{});
  if (fits(4)) return go(std::integral_constant<int, 4>{});
  if (fits(3)) return go(std::integral_constant<int, 3>{});
  if (fits(2)) return go(std::integral_constant<int, 2>{});
  return go(std::integral_constant<int, 1>{});
}

template <bool TAB>
hipError_t compress_f64(const PackLayout &L, const void *packed, const void *X, int64_t N,
                        int64_t ldx, const IdArgs &ids, const ProjArgs &pa, int mode, void *out,
                        int64_t ldc, hipStream_t s) {
  return L.dt == 0
             ? compress_f64_kt<float, TAB>(L, packed, X, N, ldx, ids, pa, mode, out, ldc, s)
             : compress_f64_kt<bf16_t, TAB>(L, packed, X, N, ldx, ids, pa, mode, out, ldc, s);
}

hipError_t launch_compress_generic(const PackLayout &L, const void *packed, const void *X,
                                   int64_t N, int64_t ldx, const IdArgs &ids, void *C,
                                   int64_t ldc, hipStream_t s) {
  const ProjArgs none{};
  if (ids.E || ids.P) return compress_f64<true>(L, packed, X, N, ldx, ids, none, kGenT, C, ldc, s);
  return compress_f64<false>(L, packed, X, N, ldx, ids, none, kGenT, C, ldc, s);
}

// ---------------------------------------------------------------------------
// Projected tables and compress against them: the same kernel with other
// ends.
// ---------------------------------------------------------------------------

ProjLayout proj_layout(int64_t k, int64_t vocab, int64_t n_pos) {
  ProjLayout P;
  P.kp = 16 * ceil_div(k, 16);
  P.off_eu = 0;
  P.off_pu = align256(static_cast<size_t>(vocab) * P.kp * sizeof(float));
  P.total = P.off_pu + align256(static_cast<size_t>(n_pos) * P.kp * sizeof(float));
  return P;
}

hipError_t launch_table_project_generic(const PackLayout &L, const void *packed, const void *T,
                                        int64_t rows, int64_t ldt, float *out, int64_t kp,
                                        hipStream_t s) {
  return compress_f64<false>(L, packed, T, rows, ldt, IdArgs{}, ProjArgs{}, kGenTable, out, kp, s);
}

hipError_t launch_compress_projected_generic(const PackLayout &L, const void *packed,
                                             const void *X, int64_t N, int64_t ldx,
                                             const ProjArgs &pa, void *C, int64_t ldc,
                                             hipStream_t s) {
  return compress_f64<false>(L, packed, X, N, ldx, IdArgs{}, pa, kGenT, C, ldc, s);
}

// ---------------------------------------------------------------------------
// Decompress: a workgroup owns 64 tokens (a tile of 16 per wave, whose
// coefficients the wave holds in float64) and a range of column pairs (32
// columns of d), whose U fragments it copies into LDS once.  P + E is the
// MFMA chain's start, so the sum is rounded once; the tables' values of the
// next pair are loaded while this one is multiplied.  A pair keeps whole
// 128-byte lines of float32 rows together and two MFMA chains in flight.
// Bound by the stores (3.2 TB/s at k = 4) up to k ~ 30, above by the f64
// matrix rate.  8192 tokens, d = 2048, k = 20, float32: 305 us (a thread per
// element) -> 21 us; neighbouring workgroups hold neighbouring columns of the
// same rows, not other rows (32768 tokens, d = 4096, k = 40: 308 -> 218 us).
// Fragments kept in LDS as float64 (no conversion per MFMA, twice the LDS
// reads) took 274 us there.
// ---------------------------------------------------------------------------

constexpr int kDecLds = 32 * 1024;  // U fragments per workgroup (at least one pair's)

template <typename T, int KG, bool TAB>
__global__ __launch_bounds__(256) void decompress_f64_kernel(
    const f32x4 *__restrict__ rfrag, int kt, int64_t d, int64_t k, const T *__restrict__ C,
    int64_t N, int64_t ldc, IdArgs ids, T *__restrict__ X, int64_t ldx, int pairs_per_wg) {
  extern __shared__ f32x4 us[];  // [tile of the range][kt][lane]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, n = lane & 15;
  const int ntile = static_cast<int>((d + 15) / 16);
  const int r0 = 2 * static_cast<int>(blockIdx.x) * pairs_per_wg;
  const int r1 = r0 + 2 * pairs_per_wg < ntile ? r0 + 2 * pairs_per_wg : ntile;
  const int64_t tg = static_cast<int64_t>(blockIdx.z) * gridDim.y + blockIdx.y;
  if (64 * tg >= N) return;
  {
    const f32x4 *src = rfrag + static_cast<int64_t>(r0) * kt * 64;
    const int units = (r1 - r0) * kt * 64;
    for (int e = threadIdx.x; e < units; e += 256) us[e] = src[e];
  }
  const int64_t i = 16 * (tg * 4 + wave) + n;
  const bool live = i < N;
  const int64_t ic = live ? i : N - 1;
  const int nsteps = static_cast<int>((k + 3) / 4);
  double cb[4 * KG];  // C[token n, 4 s + g] of step s
#pragma unroll
  for (int st = 0; st < 4 * KG; ++st) {
    const int64_t j = 4 * st + g;
    cb[st] = j < k ? static_cast<double>(to_f32(C[ic * ldc + j])) : 0.0;
  }
  T *xr = X + ic * ldx;
  Rows<T> rw{};
  if constexpr (TAB) rw = resolve_rows<T>(ic, ids, static_cast<const T *>(nullptr));

  // P + E of columns 16 r + 4 g .. + 3 of the token
  struct Tab {
    Row4<T> p, e;
  };
  const bool hp = TAB && ids.P, he = TAB && ids.E;
  auto whole = [&](int r) { return 16 * static_cast<int64_t>(r) + 4 * g + 4 <= d; };
  auto load_tab = [&](Tab &t, int r) {
    const int64_t c = 16 * static_cast<int64_t>(r) + 4 * g;
    if (whole(r)) {
      if (hp) t.p.load(rw.p + c);
      if (he) t.e.load(rw.e + c);
    }
  };
  auto start = [&](const Tab &t, int r) {
    f64x4 v = {0., 0., 0., 0.};
    if constexpr (TAB) {
      const int64_t c = 16 * static_cast<int64_t>(r) + 4 * g;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (whole(r)) {
          if (hp) v[q] += t.p.at(q);
          if (he) v[q] += t.e.at(q);
        } else if (c + q < d) {
          if (hp) v[q] += static_cast<double>(to_f32(rw.p[c + q]));
          if (he) v[q] += static_cast<double>(to_f32(rw.e[c + q]));
        }
      }
    }
    return v;
  };
  // lane (g, n): columns 16 r + 4 g .. + 3 of token n
  auto store = [&](int r, const f64x4 &v) {
    const int64_t c = 16 * static_cast<int64_t>(r) + 4 * g;
    if (whole(r)) {
      Row4<T>::store(xr + c, v);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (c + q < d) xr[c + q] = from_f64<T>(v[q]);
    }
  };

  Tab cur[2], nxt[2];
  if constexpr (TAB) {
    load_tab(cur[0], r0);
    load_tab(cur[1], r0 + 1);
  }
  __syncthreads();
  for (int r = r0; r < r1; r += 2) {
    if (TAB && r + 2 < r1) {  // a range of one pair (few tokens) waits for no more loads
      load_tab(nxt[0], r + 2);
      load_tab(nxt[1], r + 3);
    }
    f64x4 a0 = start(cur[0], r), a1 = start(cur[1], r + 1);
    const f32x4 *f0 = us + (r - r0) * kt * 64 + lane;
    const f32x4 *f1 = r + 1 < r1 ? f0 + kt * 64 : f0;  // an odd last tile has no partner
#pragma unroll
    for (int q = 0; q < KG; ++q) {
      const int qq = q < kt ? q : kt - 1;  // groups past the last take no step below
      const f32x4 u0 = f0[qq * 64], u1 = f1[qq * 64];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * q + e < nsteps) {
          a0 = mfma64(static_cast<double>(u0[e]), cb[4 * q + e], a0);
          a1 = mfma64(static_cast<double>(u1[e]), cb[4 * q + e], a1);
        }
    }
    if (live) {
      store(r, a0);
      if (r + 1 < r1) store(r + 1, a1);
    }
    if constexpr (TAB) {
      cur[0] = nxt[0];
      cur[1] = nxt[1];
    }
  }
}

// Few values: a thread per value, the same sum in float64.  Such a launch is a chain
// of latencies, shorter without the fragments' way through LDS, the MFMAs and the
// edges of the tiles; with more values or columns of U the products decide.  In a
// graph, matrix cores / a thread per value (a thread per value in compensated float32
// sums, which every launch once took, first):
//   bf16, both tables   d = 131, k = 3, 160 tokens   2.74   4.32 / 2.86 us
//                       d = 384, k = 6, 512 tokens   3.57   4.48 / 3.52
//                       d = 384, k = 4, 1300 tokens         4.43 / 4.82
//   float32, no tables  d = 384, k = 6, 512 tokens   2.81   2.99 / 2.92
//                       d = 600, k = 12, 290 tokens         3.08 / 3.19
//                       d = 384, k = 6, 2048 tokens  5.20   3.56 / 5.43
inline bool few_values(int64_t values, int64_t k) {
  return values <= (int64_t{1} << 19) && values * k <= (int64_t{5} << 18);
}

template <typename T, bool TAB>
__global__ __launch_bounds__(256) void decompress_few_kernel(
    const float *__restrict__ U, unsigned d, int k, const T *__restrict__ C, unsigned total,
    int64_t ldc, IdArgs ids, T *__restrict__ X, int64_t ldx) {
  const unsigned idx = blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const unsigned i = idx / d, c = idx - i * d;
  const T *cr = C + i * ldc;
  const float *ur = U + static_cast<int64_t>(c) * k;
  double v = 0.0;
  if constexpr (TAB) {
    const Rows<T> rw = resolve_rows<T>(i, ids, static_cast<const T *>(nullptr));
    if (ids.P) v += static_cast<double>(to_f32(rw.p[c]));
    if (ids.E) v += static_cast<double>(to_f32(rw.e[c]));
  }
#pragma unroll 8
  for (int j = 0; j < k; ++j)
    v = fma(static_cast<double>(ur[j]), static_cast<double>(to_f32(cr[j])), v);
  X[i * ldx + c] = from_f64<T>(v);
}

template <typename T, bool TAB>
hipError_t decompress_f64(const PackLayout &L, const void *packed, const void *C, int64_t N,
                          int64_t ldc, const IdArgs &ids, void *X, int64_t ldx, hipStream_t s) {
  const f32x4 *rf =
      reinterpret_cast<const f32x4 *>(static_cast<const char *>(packed) + L.off_rfrag32);
  const int64_t total = N * L.d;
  if (few_values(total, L.k)) {
    const float *u32 =
        reinterpret_cast<const float *>(static_cast<const char *>(packed) + L.off_f32);
    decompress_few_kernel<T, TAB><<<dim3(static_cast<unsigned>(ceil_div(total, 256))), 256, 0, s>>>(
        u32, static_cast<unsigned>(L.d), static_cast<int>(L.k), static_cast<const T *>(C),
        static_cast<unsigned>(total), ldc, ids, static_cast<T *>(X), ldx);
    return hipGetLastError();
  }
  // column ranges: about 4 workgroups (16 waves) a CU, and as many pairs as
  // the LDS allotment holds
  const int64_t tgroups = ceil_div(N, 64), pairs = ceil_div(L.d, 32);
  int64_t per = ceil_div(pairs, ceil_div(1024, tgroups));
  const int64_t most = kDecLds / (2048 * L.kt) > 0 ? kDecLds / (2048 * L.kt) : 1;
  per = per < most ? per : most;
  const int64_t gy = tgroups < 32768 ? tgroups : 32768;
  const dim3 grid(static_cast<unsigned>(ceil_div(pairs, per)), static_cast<unsigned>(gy),
                  static_cast<unsigned>(ceil_div(tgroups, gy)));
  const T *c = static_cast<const T *>(C);
  T *x = static_cast<T *>(X);
  auto go = [&](auto kg) {
    decompress_f64_kernel<T, decltype(kg)::value, TAB>
        <<<grid, 256, static_cast<size_t>(per) * 2048 * L.kt, s>>>(
            rf, L.kt, L.d, L.k, c, N, ldc, ids, x, ldx, static_cast<int>(per));
    return hipGetLastError();
  };
  switch (L.kt) {
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 3: return go(std::integral_constant<int, 3>{});
    case 4: return go(std::integral_constant<int, 4>{});
    case 5:
    case 6: return go(std::integral_constant<int, 6>{});
    case 7:
    case 8: return go(std::integral_constant<int, 8>{});
    default: return go(std::integral_constant<int, 16>{});
  }
}

hipError_t launch_decompress_generic(const PackLayout &L, const void *packed, const void *C,
                                     int64_t N, int64_t ldc, const IdArgs &ids, void *X,
                                     int64_t ldx, hipStream_t s) {
  if (ids.E || ids.P)
    return L.dt == 0 ? decompress_f64<float, true>(L, packed, C, N, ldc, ids, X, ldx, s)
                     : decompress_f64<bf16_t, true>(L, packed, C, N, ldc, ids, X, ldx, s);
  return L.dt == 0 ? decompress_f64<float, false>(L, packed, C, N, ldc, ids, X, ldx, s)
                   : decompress_f64<bf16_t, false>(L, packed, C, N, ldc, ids, X, ldx, s);
}

// ---------------------------------------------------------------------------
// Weight projection W <- U (U^T W), generic path, two passes:
//   1. T_s = U[rows of split s]^T W[rows of split s], float64
//   2. W[r, c] = sum_j U[r, j] (sum_s T_s[j, c]), the splits in fixed order
// Workspace: the splits' T_s as k x m float64 each (what the size formula, made
// for float32 sums of 256 rows and their total, leaves room for).
// ---------------------------------------------------------------------------

constexpr int kGenericRowsPerSplit = 256;

size_t project_workspace_generic(int64_t d, int64_t k, int64_t m) {
  int64_t s = ceil_div(d, kGenericRowsPerSplit);
  s = s > 64 ? 64 : s;
  return static_cast<size_t>(s + 1) * k * m * sizeof(float);
}

// Pass 1.  A workgroup takes 64 columns of W, KT column tiles of U and a split
// of the rows, which its waves share by units of 32: lane (g, n) holds
// columns 4 n .. 4 n + 3 of rows 8 g .. 8 g + 7 of a unit (16 lanes read 64
// contiguous elements of a row), each row giving one f64 MFMA per column and
// column tile.  The waves' sums are added through LDS in wave order.  Bound by
// the f64 matrix rate of the CUs the workspace's splits can fill.  d = 4096,
// k = 40, two float32 matrices of 512 columns: 1522 us (vector ALU, compensated
// float32 sums, three passes) -> 84 us, pass 1 21 and pass 2 22 of each matrix.
//
// ROWS: the left factor is not U but a d x k float64 matrix given by rows (the
// subspace update's coefficients; d then counts tokens and W is the gradient).
template <typename T, int KT, bool ROWS>
__global__ __launch_bounds__(256) void project_t_f64_kernel(const f32x4 *__restrict__ kfrag,
                                                            const double *__restrict__ left, int kt,
                                                            int64_t d, int64_t k,
                                                            const T *__restrict__ W, int64_t m,
                                                            int64_t ldw, int units_per_split,
                                                            double *__restrict__ Tp) {
  __shared__ double red[4][4][64][4];  // [wave][column of the lane][lane][row of the tile]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, n = lane & 15;
  // z: the column tiles of U, and over them the column blocks that x leaves
  const int nz = (kt + KT - 1) / KT;
  const int64_t cb = 64 * (static_cast<int64_t>(blockIdx.z / nz) * gridDim.x + blockIdx.x);
  if (cb >= m) return;
  const int64_t c0 = cb + 4 * n;
  const bool whole = c0 + 4 <= m;
  const int t0 = static_cast<int>(blockIdx.z % nz) * KT;
  const int units = static_cast<int>((d + 31) / 32);
  const int u0 = static_cast<int>(blockIdx.y) * units_per_split;
  const int u1 = u0 + units_per_split < units ? u0 + units_per_split : units;
  f64x4 acc[KT][4];
#pragma unroll
  for (int t = 0; t < KT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[t][q] = f64x4{0., 0., 0., 0.};
  struct Unit {
    Row4<T> w[8];
  };
  auto load = [&](Unit &v, int u) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      int64_t r = 32 * static_cast<int64_t>(u) + 8 * g + e;
      r = r < d ? r : d - 1;  // U's fragments are zero past row d
      const T *p = W + r * ldw;
      if (whole) {
        v.w[e].load(p + c0);
      } else {  // the right edge: columns past m read the last one, not stored
        T x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = p[c0 + q < m ? c0 + q : m - 1];
        v.w[e].load(x);
      }
    }
  };
  if (u0 + wave < u1) {
    Unit cur, nxt;
    load(cur, u0 + wave);
    for (int u = u0 + wave; u < u1; u += 4) {
      load(nxt, u + 4 < u1 ? u + 4 : u);  // past the end the unit repeats, unused
      const bool part = 32 * static_cast<int64_t>(u) + 32 > d;  // rows past d: no inf x 0
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 a[ROWS ? 1 : KT];
        if constexpr (!ROWS) {
#pragma unroll
          for (int t = 0; t < KT; ++t) {
            const int tt = t0 + t < kt ? t0 + t : kt - 1;  // tiles past the last are not stored
            a[t] = kfrag[((static_cast<int64_t>(u) * kt + tt) * 2 + h) * 64 + lane];
          }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int64_t r = 32 * static_cast<int64_t>(u) + 8 * g + 4 * h + e;
          const bool out = part && r >= d;
          double av[KT];
#pragma unroll
          for (int t = 0; t < KT; ++t) {
            if constexpr (ROWS) {
              const int64_t j = 16 * (t0 + t) + n;
              av[t] = out ? 0.0 : left[r * k + (j < k ? j : k - 1)];
            } else {
              av[t] = static_cast<double>(a[t][e]);
            }
          }
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const double b = out ? 0.0 : cur.w[4 * h + e].at(q);
#pragma unroll
            for (int t = 0; t < KT; ++t) acc[t][q] = mfma64(av[t], b, acc[t][q]);
          }
        }
      }
      cur = nxt;
    }
  }
  // lane (g, n) of column q holds T[16 t + 4 i + g][cb + 4 n + q]
#pragma unroll
  for (int t = 0; t < KT; ++t) {
    if (t > 0) __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[wave][q][lane][i] = acc[t][q][i];
    __syncthreads();
    for (int idx = threadIdx.x; idx < 16 * 64; idx += 256) {
      const int jl = idx >> 6, cl = idx & 63;
      const int64_t j = 16 * static_cast<int64_t>(t0 + t) + jl, c = cb + cl;
      if (j >= k || c >= m) continue;
      const int at = 16 * (jl & 3) + (cl >> 2), i = jl >> 2, q = cl & 3;
      double v = red[0][q][at][i];
#pragma unroll
      for (int w = 1; w < 4; ++w) v += red[w][q][at][i];
      Tp[(static_cast<int64_t>(blockIdx.y) * k + j) * m + c] = v;
    }
  }
}

// Pass 2.  A workgroup takes 64 NT columns (16 NT per wave, whose T the wave
// holds in float64) and a range of 16-row tiles, whose U fragments it copies
// into LDS once.  Lane (g, n) gets W[16 r + 4 g + i][c0 + n]: 16 lanes store
// consecutive elements of a row.  Summing the splits one column step at a time
// (a chain of loads) instead of one split at a time cost 15 to 35 us.
template <typename T, int KG, int NT>
__global__ __launch_bounds__(256) void project_w_f64_kernel(const f32x4 *__restrict__ rfrag, int kt,
                                                            int64_t d, int64_t k,
                                                            const double *__restrict__ Tp,
                                                            int splits, T *__restrict__ W,
                                                            int64_t m, int64_t ldw,
                                                            int tiles_per_wg) {
  extern __shared__ f32x4 us[];  // [tile of the range][kt][lane]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, n = lane & 15;
  const int ntile = static_cast<int>((d + 15) / 16);
  // z: the ranges that y leaves, and over them the column blocks that x leaves
  const int64_t ranges = (ntile + tiles_per_wg - 1) / tiles_per_wg;
  const unsigned nz = static_cast<unsigned>((ranges + gridDim.y - 1) / gridDim.y);
  const int64_t range = static_cast<int64_t>(blockIdx.z % nz) * gridDim.y + blockIdx.y;
  const int64_t cblk = static_cast<int64_t>(blockIdx.z / nz) * gridDim.x + blockIdx.x;
  if (range >= ranges) return;
  const int r0 = static_cast<int>(range) * tiles_per_wg;
  const int r1 = r0 + tiles_per_wg < ntile ? r0 + tiles_per_wg : ntile;
  for (int e = threadIdx.x; e < (r1 - r0) * kt * 64; e += 256)
    us[e] = rfrag[static_cast<int64_t>(r0) * kt * 64 + e];
  const int nsteps = static_cast<int>((k + 3) / 4);
  int64_t col[NT];
  double tb[NT][4 * KG];  // T[4 s + g][col] of step s
#pragma unroll
  for (int b = 0; b < NT; ++b) {
    col[b] = (cblk * 4 + wave) * (16 * NT) + 16 * b + n;
    const int64_t c = col[b] < m ? col[b] : m - 1;
#pragma unroll
    for (int st = 0; st < 4 * KG; ++st) tb[b][st] = 0.0;
    for (int sp = 0; sp < splits; ++sp)  // a split's loads in flight together
#pragma unroll
      for (int st = 0; st < 4 * KG; ++st) {
        const int64_t j = 4 * st + g;
        const double v = Tp[(sp * k + (j < k ? j : k - 1)) * m + c];
        tb[b][st] += j < k ? v : 0.0;
      }
  }
  __syncthreads();
  for (int r = r0; r < r1; ++r) {
    f64x4 acc[NT];
#pragma unroll
    for (int b = 0; b < NT; ++b) acc[b] = f64x4{0., 0., 0., 0.};
    const f32x4 *f = us + (r - r0) * kt * 64 + lane;
#pragma unroll
    for (int q = 0; q < KG; ++q) {
      const f32x4 u = f[(q < kt ? q : kt - 1) * 64];  // groups past the last take no step below
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * q + e < nsteps) {
#pragma unroll
          for (int b = 0; b < NT; ++b)
            acc[b] = mfma64(static_cast<double>(u[e]), tb[b][4 * q + e], acc[b]);
        }
    }
#pragma unroll
    for (int b = 0; b < NT; ++b)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int64_t row = 16 * static_cast<int64_t>(r) + 4 * g + i;
        if (row < d && col[b] < m) W[row * ldw + col[b]] = from_f64<T>(acc[b][i]);
      }
  }
}

template <typename T>
hipError_t project_f64(const PackLayout &L, const void *packed, T *W, int64_t m, int64_t ldw,
                       void *ws, hipStream_t s) {
  const char *base = static_cast<const char *>(packed);
  const f32x4 *kf = reinterpret_cast<const f32x4 *>(base + L.off_kfrag32);
  const f32x4 *rf = reinterpret_cast<const f32x4 *>(base + L.off_rfrag32);
  double *Tp = static_cast<double *>(ws);
  // row splits: about two workgroups a CU, as many as the workspace holds, at
  // least a unit per wave
  const int64_t units = ceil_div(L.d, 32), cblocks = ceil_div(m, 64);
  const int64_t room =
      static_cast<int64_t>(project_workspace_generic(L.d, L.k, m) / (8 * L.k * m));
  const int kt1 = L.kt < 4 ? L.kt : 4;
  const int64_t z = ceil_div(L.kt, kt1);
  int64_t splits = ceil_div(512, cblocks * z);
  splits = splits < room ? splits : room;
  splits = splits < ceil_div(units, 4) ? splits : ceil_div(units, 4);
  const int64_t ups = ceil_div(units, splits);
  splits = ceil_div(units, ups);
  const dim3 g1(static_cast<unsigned>(grid_x(cblocks)), static_cast<unsigned>(splits),
                static_cast<unsigned>(z) * grid_more(cblocks));
  auto pass1 = [&](auto kt) {
    project_t_f64_kernel<T, decltype(kt)::value, false><<<g1, 256, 0, s>>>(
        kf, nullptr, L.kt, L.d, L.k, W, m, ldw, static_cast<int>(ups), Tp);
  };
  switch (kt1) {
    case 1: pass1(std::integral_constant<int, 1>{}); break;
    case 2: pass1(std::integral_constant<int, 2>{}); break;
    case 3: pass1(std::integral_constant<int, 3>{}); break;
    default: pass1(std::integral_constant<int, 4>{}); break;
  }
  auto pass2 = [&](auto kg, auto nt) {
    constexpr int KG = decltype(kg)::value, NT = decltype(nt)::value;
    // row ranges: about two workgroups a CU (each reads its columns' T again),
    // as many tiles as 32 KiB hold
    const int64_t tiles = ceil_div(L.d, 16), gx = ceil_div(m, 64 * NT);
    int64_t per = ceil_div(tiles, ceil_div(512, gx));
    per = per < 32 / L.kt ? per : 32 / L.kt;
    const int64_t ranges = ceil_div(tiles, per), gy = ranges < 32768 ? ranges : 32768;
    const dim3 grid(static_cast<unsigned>(grid_x(gx)), static_cast<unsigned>(gy),
                    static_cast<unsigned>(ceil_div(ranges, gy)) * grid_more(gx));
    project_w_f64_kernel<T, KG, NT>
        <<<grid, 256, static_cast<size_t>(per) * 1024 * L.kt, s>>>(
            rf, L.kt, L.d, L.k, Tp, static_cast<int>(splits), W, m, ldw, static_cast<int>(per));
    return hipGetLastError();
  };
  const std::integral_constant<int, 2> two{};
  switch (L.kt) {
    case 1: return pass2(std::integral_constant<int, 1>{}, two);
    case 2: return pass2(std::integral_constant<int, 2>{}, two);
    case 3: return pass2(std::integral_constant<int, 3>{}, two);
    case 4: return pass2(std::integral_constant<int, 4>{}, two);
    case 5:
    case 6: return pass2(std::integral_constant<int, 6>{}, two);
    case 7:
    case 8: return pass2(std::integral_constant<int, 8>{}, two);
    default: return pass2(std::integral_constant<int, 16>{}, std::integral_constant<int, 1>{});
  }
}

hipError_t launch_project_generic(const PackLayout &L, const void *packed, void *W, int64_t m,
                                  int64_t ldw, void *ws, hipStream_t s) {
  return L.dt == 0 ? project_f64(L, packed, static_cast<float *>(W), m, ldw, ws, s)
                   : project_f64(L, packed, static_cast<bf16_t *>(W), m, ldw, ws, s);
}

// ---------------------------------------------------------------------------
// The subspace update's generic path: float64 coefficients G U, the loss
// sum (g - c U^T)^2 taken directly, and the token contraction G^T (G U).
// ---------------------------------------------------------------------------

hipError_t launch_gen_coeffs(const PackLayout &L, const void *packed, const void *G, int64_t N,
                             int64_t ldg, double *C64, hipStream_t s) {
  return compress_f64<false>(L, packed, G, N, ldg, IdArgs{}, ProjArgs{}, kGenF64, C64, L.k, s);
}

// Workgroups of gen_loss_kernel: 64 tokens x a range of columns, about four a CU.
GenLossGrid gen_loss_grid(int64_t N, int64_t d) {
  GenLossGrid g;
  g.tgroups = ceil_div(N > 0 ? N : 1, 64);
  const int64_t pairs = ceil_div(d, 32);
  g.per = ceil_div(pairs, ceil_div(1024, g.tgroups));
  g.cols = ceil_div(pairs, g.per);
  g.most = 1024 + g.tgroups;  // cols <= ceil(1024 / tgroups)
  return g;
}

// part[workgroup] = the sum over its tokens and columns of (c U^T - g)^2: the
// decompress's chain started at -g, its results squared and added in a fixed
// order.
template <typename T, int KG>
__global__ __launch_bounds__(256) void gen_loss_kernel(const f32x4 *__restrict__ rfrag, int kt,
                                                       int64_t d, int64_t k,
                                                       const double *__restrict__ C64,
                                                       const T *__restrict__ G, int64_t N,
                                                       int64_t ldg, int64_t tgroups,
                                                       int pairs_per_wg,
                                                       double *__restrict__ part) {
  __shared__ double red[256];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, n = lane & 15;
  const int64_t wg = static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x;
  const int64_t tg = wg % tgroups;
  const int ntile = static_cast<int>((d + 15) / 16);
  const int64_t first = 2 * (wg / tgroups) * pairs_per_wg;
  if (first >= ntile) return;  // past the last workgroup
  const int r0 = static_cast<int>(first);
  const int r1 = r0 + 2 * pairs_per_wg < ntile ? r0 + 2 * pairs_per_wg : ntile;
  const int64_t i = 16 * (tg * 4 + wave) + n;
  const bool live = i < N;
  const int64_t ic = live ? i : N - 1;
  const int nsteps = static_cast<int>((k + 3) / 4);
  double cb[4 * KG];
#pragma unroll
  for (int st = 0; st < 4 * KG; ++st) {
    const int64_t j = 4 * st + g;
    cb[st] = j < k ? C64[ic * k + j] : 0.0;
  }
  const T *gr = G + ic * ldg;
  double l = 0.0;
  for (int r = r0; r < r1; ++r) {
    const int64_t c = 16 * static_cast<int64_t>(r) + 4 * g;
    f64x4 acc = {0., 0., 0., 0.};
    if (c + 4 <= d) {
      Row4<T> v;
      v.load(gr + c);
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] = -v.at(q);
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (c + q < d) acc[q] = -static_cast<double>(to_f32(gr[c + q]));
    }
#pragma unroll
    for (int q = 0; q < KG; ++q) {
      const f32x4 u = rfrag[(static_cast<int64_t>(r) * kt + (q < kt ? q : kt - 1)) * 64 + lane];
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4 * q + e < nsteps)
          acc = mfma64(static_cast<double>(u[e]), cb[4 * q + e], acc);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) l += acc[q] * acc[q];  // U's rows past d are zero, and so is acc
  }
  red[threadIdx.x] = live ? l : 0.0;
  __syncthreads();
  for (int w = 128; w >= 1; w >>= 1) {
    if (static_cast<int>(threadIdx.x) < w) red[threadIdx.x] += red[threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[wg] = red[0];
}

template <typename T>
hipError_t gen_loss(const PackLayout &L, const void *packed, const T *G, int64_t N, int64_t ldg,
                    const double *C64, double *part, hipStream_t s) {
  const f32x4 *rf =
      reinterpret_cast<const f32x4 *>(static_cast<const char *>(packed) + L.off_rfrag32);
  const GenLossGrid gg = gen_loss_grid(N, L.d);
  auto go = [&](auto kg) {
    gen_loss_kernel<T, decltype(kg)::value>
        <<<dim3(static_cast<unsigned>(grid_x(gg.tgroups * gg.cols)),
                grid_more(gg.tgroups * gg.cols)), 256, 0, s>>>(
            rf, L.kt, L.d, L.k, C64, G, N, ldg, gg.tgroups, static_cast<int>(gg.per), part);
    return hipGetLastError();
  };
  switch (L.kt) {  // k <= kGrassMaxK
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 3: return go(std::integral_constant<int, 3>{});
    case 4: return go(std::integral_constant<int, 4>{});
    case 5:
    case 6: return go(std::integral_constant<int, 6>{});
    default: return go(std::integral_constant<int, 8>{});
  }
}

hipError_t launch_gen_loss(const PackLayout &L, const void *packed, const void *G, int64_t N,
                           int64_t ldg, const double *C64, double *part, hipStream_t s) {
  return L.dt == 0
             ? gen_loss(L, packed, static_cast<const float *>(G), N, ldg, C64, part, s)
             : gen_loss(L, packed, static_cast<const bf16_t *>(G), N, ldg, C64, part, s);
}

// Token splits of the contraction: about two workgroups a CU, at least four
// units of 32 tokens each.
int64_t gen_token_splits(int64_t N, int64_t d, int64_t k, int64_t *most) {
  const int64_t units = ceil_div(N > 0 ? N : 1, 32);
  const int64_t z = ceil_div(ceil_div(k, 16), 4);
  int64_t sp = ceil_div(512, ceil_div(d, 64) * z);
  sp = sp < ceil_div(units, 4) ? sp : ceil_div(units, 4);
  if (most) *most = sp;
  return ceil_div(units, ceil_div(units, sp));
}

template <typename T>
hipError_t gen_tokens(const PackLayout &L, const T *G, int64_t N, int64_t ldg, const double *C64,
                      double *Tp, hipStream_t s) {
  const int64_t units = ceil_div(N, 32), splits = gen_token_splits(N, L.d, L.k);
  const int kt1 = L.kt < 4 ? L.kt : 4;
  const int64_t cblocks = ceil_div(L.d, 64);
  const dim3 grid(static_cast<unsigned>(grid_x(cblocks)), static_cast<unsigned>(splits),
                  static_cast<unsigned>(ceil_div(L.kt, kt1)) * grid_more(cblocks));
  const int ups = static_cast<int>(ceil_div(units, splits));
  auto go = [&](auto kt) {
    project_t_f64_kernel<T, decltype(kt)::value, true>
        <<<grid, 256, 0, s>>>(nullptr, C64, L.kt, N, L.k, G, L.d, ldg, ups, Tp);
    return hipGetLastError();
  };
  switch (kt1) {
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 3: return go(std::integral_constant<int, 3>{});
    default: return go(std::integral_constant<int, 4>{});
  }
}

hipError_t launch_gen_tokens(const PackLayout &L, const void *G, int64_t N, int64_t ldg,
                             const double *C64, double *Tp, hipStream_t s) {
  return L.dt == 0 ? gen_tokens(L, static_cast<const float *>(G), N, ldg, C64, Tp, s)
                   : gen_tokens(L, static_cast<const bf16_t *>(G), N, ldg, C64, Tp, s);
}

}  // namespace sn
