// The bf16 compress for launches of few tokens, on the gfx950 matrix cores.
//
// C = (X - P[pos] - T_fixed[tok]) U for 16 tokens per workgroup, the eight
// waves splitting d: wave w takes the units (64 columns) w, w + 8, ..., with D
// units in flight, and the waves' fp32 sums are added through LDS in wave
// order.  X U, (-P) U and (-T_fixed) U go into one set of fp32 accumulators,
// as in compress_kernel.
//
// Why a second kernel: compress_kernel streams whole rows through one
// workgroup per 64 or 128 tokens, 64 columns at a time, so a launch of 1024
// tokens uses 16 CUs and takes as long as one of 16384.  Here a workgroup has
// 16 tokens and most of its rows' loads in flight at once, at the price of
// reading U once per 16 tokens instead of once per 64 or 128.  Bound by the
// bytes a CU takes in (786 KB of rows and U at d = 4096, k = 40) and by the
// latency of the ids, rows and sums before and after.  d = 4096, k = 40, both
// tables: 1024 tokens 35.4 -> 12.8 us, 4096 tokens 36.6 -> 21.3 us (16.6 where the
// activation and its embedding rows are cached from the call before).
//
// The rows go through LDS although each wave reads only its own: the MFMA
// operand layout gives consecutive lanes different rows, and a load like that
// takes a CU's L1 four times as long (37 bytes per ns against 140 measured with
// 8 lanes per 128-byte line).  So a wave copies 8 rows x 128 bytes per
// direct-to-LDS load, the 16-byte pieces of row r in the order p ^ (r & 7), and
// reads operands back from there; U's fragments are contiguous and go straight
// to registers.  Each ring slot is an LDS object of its own, which lets the
// compiler wait for that slot's copies only.
#include <type_traits>

#include "sn_mfma_common.h"

namespace sn {

namespace {

constexpr int kSW = 8;  // waves per workgroup
constexpr int kSThreads = 64 * kSW;
constexpr int kTok = 16;         // tokens per workgroup
constexpr int kTile = 128;       // 16-byte units of 16 rows x 64 columns

// 16-byte slot of piece p of row r in a 16 x 64 tile
__device__ __forceinline__ int tile_slot(int r, int p) { return 8 * r + (p ^ (r & 7)); }

// Units in flight: three while their buffers and the waves' sums fit in LDS and
// the fragments in 256 registers.
template <int KT, int TABS>
constexpr int s_depth() { return TABS > 0 && KT > 6 ? 2 : 3; }

enum SplitOut { kOutBf16 = 0, kOutProjected = 1, kOutF32 = 2, kOutGrass = 3 };

template <int KT, bool HE, bool HP, int OUT>
__global__ __launch_bounds__(kSThreads) void compress_split_kernel(
    const bf16_t *__restrict__ kfrag, int64_t d, int64_t k, const bf16_t *__restrict__ X,
    int64_t N, int64_t ldx, IdArgs ids, ProjArgs pa, void *__restrict__ Cout, int64_t ldc,
    GrassOut go) {
  constexpr int TABS = HE + HP, D = s_depth<KT, TABS>();
  constexpr int WT = (1 + TABS) * kTile;  // 16-byte units per wave and ring slot
  constexpr int kRed = kSW * KT * 64;     // the waves' sums take slot 0 afterwards
  constexpr int kBuf0 = kRed > kSW * WT ? kRed : kSW * WT;
  __shared__ u32x4 buf0[kBuf0], buf1[kSW * WT], buf2[D > 2 ? kSW * WT : 1];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 4, n = lane & 15;
  const int q = lane >> 3, m = lane & 7;
  const int64_t i0 = kTok * static_cast<int64_t>(blockIdx.x);

  // rows 8 i + q that this lane copies from (rows past N repeat the last)
  const bf16_t *xr[2], *er[2], *pr[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    int64_t i = i0 + 8 * h + q;
    i = i < N ? i : N - 1;
    xr[h] = X + i * ldx;
    if constexpr (HE) {
      const int64_t t = clamp_id(ids.tok[i], ids.vocab, ids.err_flag, 1);
      er[h] = static_cast<const bf16_t *>(ids.E) + t * ids.lde;
    }
    if constexpr (HP) {
      int64_t p = ids.pos ? static_cast<int64_t>(ids.pos[i]) : i % ids.seq_len;
      p = clamp_id(p, ids.n_pos, ids.err_flag, 2);
      pr[h] = static_cast<const bf16_t *>(ids.P) + p * ids.ldp;
    }
  }

  f32x4 acc[KT];
#pragma unroll
  for (int t = 0; t < KT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  double sq = 0.0;  // kOutGrass: sum of squares of the lane's elements of its row

  const int steps = static_cast<int>(d / 32), units = (steps + 1) / 2;
  auto copy = [&](const bf16_t *const(&row)[2], int u, u32x4 *dst) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int64_t c = 64 * static_cast<int64_t>(u) + 8 * (m ^ q);  // row 8 h + q: r & 7 = q
      // columns past d (the second half of an odd last unit) are not used
      __builtin_amdgcn_global_load_lds(static_cast<const void *>(row[h] + (c < d ? c : 0)),
                                       (__attribute__((address_space(3))) void *)(dst + 64 * h),
                                       16, 0, 0);
    }
  };
  struct Frags {
    u32x4 u[2][KT];
  };
  auto load = [&](Frags &f, u32x4 *buf, int u) {
    u32x4 *b = buf + wave * WT;
    copy(xr, u, b);
    if constexpr (HE) copy(er, u, b + kTile);
    if constexpr (HP) copy(pr, u, b + (1 + HE) * kTile);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      int s = 2 * u + j;
      s = s < steps ? s : steps - 1;  // an odd last step has no partner
#pragma unroll
      for (int t = 0; t < KT; ++t)
        f.u[j][t] = ld16(kfrag + (static_cast<int64_t>(s) * KT + t) * 512 + lane * 8);
    }
  };
  constexpr int kLoads = 2 * (1 + TABS) + 2 * KT;  // vector-memory instructions of load()
  auto step = [&](const Frags &f, const u32x4 *buf, int u) {
    const u32x4 *b = buf + wave * WT;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j == 1 && 2 * u + 1 >= steps) break;  // wave-uniform
      const u32x4 x = b[tile_slot(n, 4 * j + g)];
      u32x4 e, p;
      if constexpr (HE) e = neg8(b[kTile + tile_slot(n, 4 * j + g)]);
      if constexpr (HP) p = neg8(b[(1 + HE) * kTile + tile_slot(n, 4 * j + g)]);
      if constexpr (OUT == kOutGrass) {
        float s8 = 0.0f;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const float lo = bf_lo(x[w]), hi = bf_hi(x[w]);
          s8 = fmaf(lo, lo, s8);
          s8 = fmaf(hi, hi, s8);
        }
        sq += static_cast<double>(s8);
      }
#pragma unroll
      for (int t = 0; t < KT; ++t) {
        acc[t] = mfma(f.u[j][t], x, acc[t]);
        if constexpr (HP) acc[t] = mfma(f.u[j][t], p, acc[t]);
        if constexpr (HE) acc[t] = mfma(f.u[j][t], e, acc[t]);
      }
    }
  };

  if (wave < units) {
    const int cnt = (units - wave + kSW - 1) / kSW;  // this wave's units
    auto at = [&](int i) { return wave + kSW * (i < cnt ? i : cnt - 1); };
    wait_vmcnt<0>();  // nothing is outstanding: the compiler counts from here
    Frags f0, f1, f2;
    auto fill = [&](Frags &f, u32x4 *buf, int i) {  // past the end the last unit again
      __builtin_amdgcn_sched_barrier(0);  // the loads stay in unit order (the waits count them)
      load(f, buf, at(i));
      __builtin_amdgcn_sched_barrier(0);
    };
    auto use = [&](const Frags &f, const u32x4 *buf, int i) {  // unit i, in slot i % D
      wait_vmcnt<(D - 1) * kLoads <= 63 ? (D - 1) * kLoads : 63>();
      step(f, buf, at(i));
      // the operand reads are over before the slot is filled again
      __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
      asm volatile("" ::: "memory");
    };
    fill(f0, buf0, 0);
    fill(f1, buf1, 1);
    if constexpr (D > 2) fill(f2, buf2, 2);
    int i = 0;
    for (; i + D <= cnt; i += D) {  // whole rounds of the ring: no guards
      use(f0, buf0, i);
      fill(f0, buf0, i + D);
      use(f1, buf1, i + 1);
      fill(f1, buf1, i + 1 + D);
      if constexpr (D > 2) {
        use(f2, buf2, i + 2);
        fill(f2, buf2, i + 2 + D);
      }
    }
    if (i < cnt) use(f0, buf0, i);
    wait_vmcnt<0>();
    if (D > 2 && i + 1 < cnt) use(f1, buf1, i + 1);
  }

  __syncthreads();  // every slot is free
  f32x4 *red = reinterpret_cast<f32x4 *>(buf0);
#pragma unroll
  for (int t = 0; t < KT; ++t) red[(wave * KT + t) * 64 + lane] = acc[t];
  __syncthreads();
  // sum of the waves for column j of token row of the workgroup
  auto total = [&](int row, int j) {
    const int at = 16 * ((j & 15) >> 2) + row;
    const f32x4 *r = red + (j >> 4) * 64 + at;
    float v = r[0][j & 3];
#pragma unroll
    for (int w = 1; w < kSW; ++w) v += r[w * KT * 64][j & 3];
    return v;
  };

  if constexpr (OUT == kOutGrass) {
    // The rows' loss terms |g|^2 - |c|^2 + c D c^T (D = U^T U - I) and the
    // token contraction's operand, as compress_kernel's epilogue writes them.
    constexpr int KP = 16 * KT;
    __shared__ float cT[KP][kTok + 1];
    __shared__ double wsq[kSW][kTok], part[kSThreads];
    sq += __shfl_xor(sq, 16, 64);
    sq += __shfl_xor(sq, 32, 64);
    if (g == 0) wsq[wave][n] = sq;
    for (int e = threadIdx.x; e < KP * kTok; e += kSThreads) {
      const int row = e / KP, j = e % KP;
      cT[j][row] = i0 + row < N ? total(row, j) : 0.0f;
    }
    __syncthreads();
    // This thread's share of the workgroup's loss, in a fixed order: column a of R rows,
    // so that a load of D serves R sums and the waves are all in use.  One row at a
    // time, the threads taking turns, the loads of D held the workgroup up: accumulate
    // without Y, d = 1536, k = 96, 55 tokens 28.6 -> 17.9 us, d = 4096, k = 128, 1024
    // tokens 47.9 -> 27.8; R = 4 at k <= 16 cost 0.25.
    constexpr int R = KT == 1 ? 1 : 4;
    static_assert(KP * kTok / R <= kSThreads, "one pass over the columns and rows");
    double l = 0.0;
    if (static_cast<int>(threadIdx.x) < KP * kTok / R) {
      const int a = static_cast<int>(threadIdx.x) % KP, r0 = static_cast<int>(threadIdx.x) / KP * R;
      double dc[R] = {};
#pragma unroll 8
      for (int b = 0; b < KP; ++b) {
        const double w = go.dgram[b * KP + a];
#pragma unroll
        for (int r = 0; r < R; ++r) dc[r] += w * static_cast<double>(cT[b][r0 + r]);
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double ca = cT[a][r0 + r];
        l += ca * (dc[r] - ca);
        if (a == 0 && i0 + r0 + r < N) {
#pragma unroll
          for (int w = 0; w < kSW; ++w) l += wsq[w][r0 + r];
        }
      }
    }
    part[threadIdx.x] = l;
    if (go.frag) {
      // The workgroup holds half of a 32-row step: of slot (part p, column
      // tile t2, lane 16 g2 + n2), rows 8 g2 + 0..7 of operand column
      // 16 t2 + n2, it writes the lanes with g2 / 2 = its parity.
      const int ktb = go.ktb, half = static_cast<int>(blockIdx.x & 1);
      const int64_t per_part = (go.npad / 32) * ktb * 64;
      for (int sl = threadIdx.x; sl < go.nparts * ktb * 32; sl += kSThreads) {
        const int p = sl / (ktb * 32), t2 = (sl / 32) % ktb, l2 = 32 * half + (sl & 31);
        const int r8 = 8 * ((sl & 31) >> 4);  // first of the slot's rows in this workgroup
        const int64_t c2 = 16 * t2 + (l2 & 15);
        const bool lo = go.nparts == 1 ? c2 >= k : p == 1;
        const int64_t col = go.nparts == 1 && lo ? c2 - k : c2;
        uint32_t wd[4];
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          uint32_t h[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float x = col < k ? cT[col][r8 + 2 * qq + e] : 0.0f;
            const bf16_t hi = from_f32<bf16_t>(x);
            h[e] = lo ? from_f32<bf16_t>(x - to_f32(hi)) : hi;
          }
          wd[qq] = h[0] | (h[1] << 16);
        }
        const int64_t slot =
            p * per_part + (static_cast<int64_t>(blockIdx.x >> 1) * ktb + t2) * 64 + l2;
        *reinterpret_cast<u32x4 *>(reinterpret_cast<bf16_t *>(go.frag) + slot * 8) =
            u32x4{wd[0], wd[1], wd[2], wd[3]};
      }
    }
    __syncthreads();
    for (int w = kSThreads / 2; w >= 1; w >>= 1) {
      if (static_cast<int>(threadIdx.x) < w) part[threadIdx.x] += part[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) go.part[blockIdx.x] = part[0];
    if (!Cout) return;
  }

  for (int e = threadIdx.x; e < kTok * 16 * KT; e += kSThreads) {
    const int row = e / (16 * KT), j = e % (16 * KT);
    const int64_t tok = i0 + row;
    if (tok >= N) break;  // rows ascend with e
    if (OUT == kOutF32) {  // the full padded row, zero past column k
      static_cast<float *>(Cout)[tok * ldc + j] = j < k ? total(row, j) : 0.0f;
      continue;
    }
    if (j >= k) continue;
    float v = total(row, j);
    if constexpr (OUT == kOutProjected) {
      if (pa.pu) {
        int64_t p = pa.pos ? static_cast<int64_t>(pa.pos[tok]) : tok % pa.seq_len;
        v -= pa.pu[clamp_id(p, pa.n_pos, pa.err_flag, 2) * pa.kp + j];
      }
      if (pa.eu) v -= pa.eu[clamp_id(pa.tok[tok], pa.vocab, pa.err_flag, 1) * pa.kp + j];
    }
    static_cast<bf16_t *>(Cout)[tok * ldc + j] = from_f32<bf16_t>(v);
  }
}

template <int KT, bool HE, bool HP, int OUT>
void launch_split(const PackLayout &L, const void *packed, const void *X, int64_t N, int64_t ldx,
                  const IdArgs &ids, const ProjArgs &pa, void *C, int64_t ldc, const GrassOut &go,
                  hipStream_t s) {
  const bf16_t *kf =
      reinterpret_cast<const bf16_t *>(static_cast<const char *>(packed) + L.off_kfrag);
  // the subspace update's operand is written in whole steps of 32 rows
  const int64_t groups = OUT == kOutGrass ? 2 * ceil_div(N, 32) : ceil_div(N, kTok);
  compress_split_kernel<KT, HE, HP, OUT>
      <<<dim3(static_cast<unsigned>(groups)), kSThreads, 0, s>>>(
          kf, L.d, L.k, static_cast<const bf16_t *>(X), N, ldx, ids, pa, C, ldc, go);
}

template <int KT>
void launch_split_out(const PackLayout &L, const void *packed, const void *X, int64_t N,
                     int64_t ldx, const IdArgs &ids, const ProjArgs &pa, int out, void *C,
                     int64_t ldc, hipStream_t s) {
  const GrassOut go{};
  const bool he = ids.E != nullptr, hp = ids.P != nullptr;
  if (out == kOutProjected)
    launch_split<KT, false, false, kOutProjected>(L, packed, X, N, ldx, ids, pa, C, ldc, go, s);
  else if (out == kOutF32)
    launch_split<KT, false, false, kOutF32>(L, packed, X, N, ldx, ids, pa, C, ldc, go, s);
  else if (he && hp)
    launch_split<KT, true, true, kOutBf16>(L, packed, X, N, ldx, ids, pa, C, ldc, go, s);
  else if (he)
    launch_split<KT, true, false, kOutBf16>(L, packed, X, N, ldx, ids, pa, C, ldc, go, s);
  else if (hp)
    launch_split<KT, false, true, kOutBf16>(L, packed, X, N, ldx, ids, pa, C, ldc, go, s);
  else
    launch_split<KT, false, false, kOutBf16>(L, packed, X, N, ldx, ids, pa, C, ldc, go, s);
}

hipError_t split_kt(const PackLayout &L, const void *packed, const void *X, int64_t N, int64_t ldx,
                    const IdArgs &ids, const ProjArgs &pa, int out, void *C, int64_t ldc,
                    hipStream_t s) {
  auto go = [&](auto kt) {
    launch_split_out<decltype(kt)::value>(L, packed, X, N, ldx, ids, pa, out, C, ldc, s);
    return hipGetLastError();
  };
  switch (L.kt) {
    case 1: return go(std::integral_constant<int, 1>{});
    case 2: return go(std::integral_constant<int, 2>{});
    case 3: return go(std::integral_constant<int, 3>{});
    case 4: return go(std::integral_constant<int, 4>{});
    case 5: return go(std::integral_constant<int, 5>{});
    case 6: return go(std::integral_constant<int, 6>{});
    case 7: return go(std::integral_constant<int, 7>{});
    case 8: return go(std::integral_constant<int, 8>{});
    default: return hipErrorNotSupported;
  }
}

}  // namespace

hipError_t launch_compress_split(const PackLayout &L, const void *packed, const void *X, int64_t N,
                                 int64_t ldx, const IdArgs &ids, void *C, int64_t ldc,
                                 hipStream_t s) {
  return split_kt(L, packed, X, N, ldx, ids, ProjArgs{}, kOutBf16, C, ldc, s);
}

hipError_t launch_table_project_split(const PackLayout &L, const void *packed, const void *T,
                                      int64_t rows, int64_t ldt, float *out, int64_t kp,
                                      hipStream_t s) {
  return split_kt(L, packed, T, rows, ldt, IdArgs{}, ProjArgs{}, kOutF32, out, kp, s);
}

hipError_t launch_compress_projected_split(const PackLayout &L, const void *packed, const void *X,
                                           int64_t N, int64_t ldx, const ProjArgs &pa, void *C,
                                           int64_t ldc, hipStream_t s) {
  return split_kt(L, packed, X, N, ldx, IdArgs{}, pa, kOutProjected, C, ldc, s);
}

hipError_t launch_grass_compress_split(const PackLayout &L, const void *packed, const void *G,
                                       int64_t N, int64_t ldg, const GrassOut &go, void *Cwire,
                                       int64_t ldc, hipStream_t s) {
  auto run = [&](auto kt) {
    launch_split<decltype(kt)::value, false, false, kOutGrass>(
        L, packed, G, N, ldg, IdArgs{}, ProjArgs{}, Cwire, ldc, go, s);
    return hipGetLastError();
  };
  switch (L.kt) {
    case 1: return run(std::integral_constant<int, 1>{});
    case 2: return run(std::integral_constant<int, 2>{});
    case 3: return run(std::integral_constant<int, 3>{});
    case 4: return run(std::integral_constant<int, 4>{});
    case 5: return run(std::integral_constant<int, 5>{});
    case 6: return run(std::integral_constant<int, 6>{});
    case 7: return run(std::integral_constant<int, 7>{});
    case 8: return run(std::integral_constant<int, 8>{});
    default: return hipErrorNotSupported;
  }
}

}  // namespace sn
