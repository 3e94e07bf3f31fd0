// Apply kernel for heads of 128 in bf16 with one or two maps: both forms, both
// far-field normalisations, bands that fit the ring.  The general kernel
// (fmm_wide.hip) reads and advances the fp32 state record in global memory at
// this width, four waves and 132 KB per tile and map: 73000 cycles per 64-row
// tile, two thirds of them waiting.  Here
//   * one workgroup of 8 waves owns a CU: the state of both maps (128 KB in
//     fp32) is 64 registers of each lane, wave w holding feature block w, and
//     its bf16 operand fragments (64 KB) sit in LDS beside the K / V ring;
//   * a 16-row strip is shared by two waves (w and w + 4), each forming the
//     strip's scores and half of its output columns: 8 waves keep two on each
//     SIMD, and the scores done twice are a quarter of the products;
//   * the next tile's K, V and query rows are loaded while the current tile
//     computes, and phi_1 of the next keys comes from those registers.
// 8 slices of 16381 rows, rank 2, k = 64, causal: 543 -> 133 us (the call 593
// -> 166 us); non-causal, k = 20: 348 -> 85 us per call.
#include "fmm_apply.h"
#include "fmm_device.h"
#include "fmm_launch.h"

namespace fmm {
namespace {

typedef bf16_t T;
typedef QuadOf<T>::type Q;
constexpr int D = 128, NB = D / 16, DV = D / 2, NV = DV / 16;
constexpr int W8 = 8, NT8 = W8 * 64;
constexpr int ST = D + Lay<T>::PAD, ROW = ST * (int)sizeof(T);
constexpr int UNIT = 2 * 32 * ROW;  // K and V rows of a 32-key unit

// LDS: U units of K, then of V | phi rows of the tile's keys, one map
// (causal) | state fragments | z fragments
constexpr int frag_bytes(int R) { return R * NB * NB * 64 * (int)sizeof(Q); }
constexpr int lds_bytes(int R, bool causal, int U) {
  return U * UNIT + (causal ? TM * ROW : 0) + frag_bytes(R) + R * NB * 4 * (int)sizeof(Q);
}
constexpr int kMaxLds = 160 * 1024;

// phi_{l+1} of a chunk of 8 bf16 values (zero where !ok)
__device__ __forceinline__ uint4 phi_chunk(const uint4& x, int l, bool ok) {
  const uint16_t* e = reinterpret_cast<const uint16_t*>(&x);
  float f[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) f[i] = ok ? phi_l(bf16_to_f32(e[i]), l) : 0.f;
  return make_uint4(pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]),
                    pack_bf16x2(f[6], f[7]));
}

typedef RowCopy<T, D, NT8, 64> Rows;
// phi_1 of the 64 rows from t0 held in a RowCopy, as chunks of their LDS rows
// (rows at or beyond N give 0)
struct PhiCopy {
  uint4 p[Rows::IT];
  __device__ __forceinline__ void compute(const Rows& k, int t0, int N) {
#pragma unroll
    for (int it = 0; it < Rows::IT; ++it)
      p[it] = phi_chunk(k.r[it], 0, t0 + (int)(threadIdx.x + it * NT8) / Rows::CPR < N);
  }
  __device__ __forceinline__ void store(T* dst) const {
#pragma unroll
    for (int it = 0; it < Rows::IT; ++it) {
      const int t = threadIdx.x + it * NT8;
      *reinterpret_cast<uint4*>(dst + (t / Rows::CPR) * ST + (t % Rows::CPR) * 8) = p[it];
    }
  }
};

template <int R, bool CAUSAL, bool JOINT>
__global__ __launch_bounds__(NT8) void k_wide128(const T* __restrict__ q,
                                                 const T* __restrict__ k,
                                                 const T* __restrict__ v, T* __restrict__ out,
                                                 const float* __restrict__ recs,
                                                 const float* __restrict__ w_near,
                                                 const float* __restrict__ w_far, int H, int N,
                                                 int band_k, int L, int nseg, float scale2) {
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
  const int kc = (band_k + 31) >> 5;
  const int U = 2 + (CAUSAL ? kc : 2 * kc);
  T* sk = reinterpret_cast<T*>(dyn_smem);
  T* sv = sk + U * 32 * ST;
  T* spk = sv + U * 32 * ST;
  Q* sf = reinterpret_cast<Q*>(spk + (CAUSAL ? TM * ST : 0));
  Q* sz = sf + R * NB * NB * 64;
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = lin / nseg, seg = lin % nseg, h = bh % H;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sp = w & 3, e0 = (w >> 2) * NV;  // strip of the tile, first value block
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const size_t base = (size_t)bh * N * D;
  const T *qh = q + base, *kh = k + base, *vh = v + base;
  const size_t REC = (size_t)R * D * (D + 1);
  const float* rec = recs + (CAUSAL ? (size_t)bh * nseg + seg : (size_t)bh) * REC;
  const float sn = sigmoidf_exact(w_near[h]), sfw = sigmoidf_exact(w_far[h]);
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const int s0 = seg * L, s1 = min(N, s0 + L);
  const int ntile = (s1 - s0 + TM - 1) / TM;
  const RingMap map{(s0 >> 5) - kc, U};

  // the wave's feature block of the state: tiles (w, eb) and, in tile NB, z
  f32x4 acc[R][NB + 1];
#pragma unroll
  for (int l = 0; l < R; ++l) {
    const float* sl = rec + (size_t)l * D * (D + 1);
#pragma unroll
    for (int eb = 0; eb < NB; ++eb)
      acc[l][eb] = *reinterpret_cast<const f32x4*>(sl + ((w * NB + eb) * 64 + lane) * 4);
    acc[l][NB] =
        r == 0 ? *reinterpret_cast<const f32x4*>(sl + D * D + 16 * w + 4 * g) : zero;
  }
  auto to_quad = [](const f32x4& x) {
    const float f[4] = {x[0], x[1], x[2], x[3]};
    return f32_to_quad<T>(f);
  };
  auto store_frags = [&]() {
#pragma unroll
    for (int l = 0; l < R; ++l) {
#pragma unroll
      for (int eb = 0; eb < NB; ++eb)
        sf[((l * NB + eb) * NB + w) * 64 + lane] = to_quad(acc[l][eb]);
      if (r == 0) sz[(l * NB + w) * 4 + g] = to_quad(acc[l][NB]);
    }
  };
  Q qq[NB];
  load_q<T, D>(qh, s0 + 16 * sp + r, N, qq);
  Rows ck, cv;
  {
    // the first window, 64 rows at a time; the tile's own keys are among them
    auto ident = [](int i) { return i; };
    for (int x = 0; x < U * 32; x += 64) {
      const int m = min(64, U * 32 - x);
      ck.load(kh, map.ua0 * 32 + x, m, N);
      cv.load(vh, map.ua0 * 32 + x, m, N);
      ck.store(sk + x * ST, ST, m, ident);
      cv.store(sv + x * ST, ST, m, ident);
    }
    store_frags();
    if constexpr (CAUSAL) {
      ck.load(kh, s0, 64, N);
      PhiCopy ph;
      ph.compute(ck, s0, N);
      ph.store(spk);
    }
  }
  ck.load(kh, (map.ua0 + U) * 32, ntile > 1 ? 64 : 0, N);
  cv.load(vh, (map.ua0 + U) * 32, ntile > 1 ? 64 : 0, N);
  for (int t = 0; t < ntile; ++t) {
    const int t0 = s0 + t * TM, i0 = t0 + 16 * sp, row = i0 + r;
    const int rt[2] = {map(t0 >> 5), map((t0 >> 5) + 1)};  // ring rows of the tile's units
    __syncthreads();  // window, fragments and phi_1 rows of tile t are in LDS
    NearState<DV> st;
    st.init();
    const int lo = max(0, i0 - band_k), hi = min(N - 1, CAUSAL ? i0 + 15 : i0 + 15 + band_k);
    if (lo <= hi)
      near_units<T, D, CAUSAL, 2>(st, qq, sk, sv + 16 * e0, ST, map, lo >> 5, hi >> 5, i0, N,
                                  band_k, scale2);
    mfma_drain();
    f32x4 fo[NV], nsum[NV];
    near_out<DV>(st, sn, fo);
    float dsum = 0.f;
#pragma unroll
    for (int nb = 0; nb < NV; ++nb) nsum[nb] = zero;
#pragma unroll
    for (int l = 0; l < R; ++l) {
      Q pq[NB];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        float x[4], p[4];
        quad_to_f32(qq[cb], x);
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = phi_l(x[i], l);
        pq[cb] = f32_to_quad<T>(p);
      }
      // the query quads are dead after the last map: the next tile's rows
      if (l == R - 1)
        load_q<T, D>(qh, t0 + TM + 16 * sp + r, t + 1 < ntile ? N : 0, qq);
      f32x4 num[NV + 1];
#pragma unroll
      for (int nb = 0; nb <= NV; ++nb) num[nb] = zero;
      // the product with the state before the tile (non-causal: the total)
#pragma unroll
      for (int nb = 0; nb < NV; ++nb) {
        Q a[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) a[cb] = sf[((l * NB + e0 + nb) * NB + cb) * 64 + lane];
        num[nb] = contract<NB>(a, pq, num[nb]);
      }
      {
        Q a[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) a[cb] = sz[(l * NB + cb) * 4 + g];
        num[NV] = contract<NB>(a, pq, num[NV]);
      }
      if constexpr (CAUSAL) {
        const Q ones = quad_fill<T>(1.f);
        // keys of the tile up to the row: units 0 .. sp / 2, the last masked
        for (int u = 0; u <= (sp >> 1); ++u) {
          const bool diag = u == (sp >> 1);
          float a2[2][4];
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            Q ka[NB];
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
              ka[cb] = ld_quad(spk, 32 * u + 16 * b + r, 16 * cb + 4 * g, ST);
            const f32x4 at = contract<NB>(ka, pq, zero);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int j = t0 + 32 * u + 16 * b + 4 * g + i;
              a2[b][i] = (!diag || j <= row) ? at[i] : 0.f;
            }
          }
          const Q p0 = f32_to_quad<T>(a2[0]), p1 = f32_to_quad<T>(a2[1]);
          const T* vx = sv + rt[u] * ST + 16 * e0;
#pragma unroll
          for (int nb = 0; nb < NV; ++nb)
            num[nb] = mma_step2(ld_tquad(vx, 0, 16 * nb, ST), ld_tquad(vx, 16, 16 * nb, ST), p0,
                                p1, num[nb]);
          num[NV] = mma_step2(ones, ones, p0, p1, num[NV]);
        }
        mfma_drain();
      }
      if constexpr (JOINT) {
#pragma unroll
        for (int nb = 0; nb < NV; ++nb) nsum[nb] += num[nb];
        dsum += num[NV][0];
      } else {
        add_far_map<DV>(num, sfw, fo);
      }
      if constexpr (CAUSAL) {
        // the wave's state tiles take the tile's keys (after the last tile
        // nobody reads them)
        const Q one0 = quad_fill<T>(r == 0 ? 1.f : 0.f);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const Q a0 = ld_tquad(spk, 32 * u, 16 * w, ST);
          const Q a1 = ld_tquad(spk, 32 * u + 16, 16 * w, ST);
          const T* vx = sv + rt[u] * ST;
#pragma unroll
          for (int eb = 0; eb < NB; ++eb)
            acc[l][eb] = mma_step2(a0, a1, ld_tquad(vx, 0, 16 * eb, ST),
                                   ld_tquad(vx, 16, 16 * eb, ST), acc[l][eb]);
          acc[l][NB] = mma_step2(a0, a1, one0, one0, acc[l][NB]);
        }
        if (l + 1 < R) {
          __syncthreads();  // every wave has read map l's phi rows
          // the next map's, from the tile's key rows in the ring (the causal
          // form of two maps already spills 26 to 31 registers; kept from the
          // prefetch they would be eight more)
#pragma unroll
          for (int it = 0; it < Rows::IT; ++it) {
            const int x = threadIdx.x + it * NT8, i = x / Rows::CPR, c = 8 * (x % Rows::CPR);
            const int kr = (i < 32 ? rt[0] : rt[1]) + (i & 31);
            const uint4 raw = *reinterpret_cast<const uint4*>(sk + kr * ST + c);
            *reinterpret_cast<uint4*>(spk + i * ST + c) = phi_chunk(raw, l + 1, t0 + i < N);
          }
          __syncthreads();
        }
      }
    }
    if constexpr (JOINT) {
      const float f = sfw > 0.f ? sfw * fast_rcp(dsum) : 0.f;
#pragma unroll
      for (int nb = 0; nb < NV; ++nb) fo[nb] += nsum[nb] * f;
    }
    {
      const Rsrc rs = rows_rsrc<T, D>(out + base, i0, 16, N);
#pragma unroll
      for (int nb = 0; nb < NV; ++nb)
        buf_st(rs, (r * D + 16 * (e0 + nb) + 4 * g) * (int)sizeof(T), to_quad(fo[nb]));
    }
    PhiCopy ph;
    if constexpr (CAUSAL) ph.compute(ck, t0 + TM, N);  // the prefetched rows: the next keys
    __syncthreads();  // every wave is done with tile t's LDS
    const int ua_new = map.ua0 + 2 * t + U;
    const int ra = map(ua_new), rb = map(ua_new + 1);
    auto rowmap = [=](int i) { return (i < 32 ? ra : rb) + (i & 31); };
    ck.store(sk, ST, 64, rowmap);
    cv.store(sv, ST, 64, rowmap);
    if constexpr (CAUSAL) {
      ph.store(spk);
      store_frags();
    }
    const bool pf = t + 2 < ntile;
    ck.load(kh, (ua_new + 2) * 32, pf ? 64 : 0, N);
    cv.load(vh, (ua_new + 2) * 32, pf ? 64 : 0, N);
  }
}

template <int R, bool CAUSAL, bool JOINT>
hipError_t launch_k(const LaunchArgs& a, Launcher& L, const float* recs) {
  static std::atomic<unsigned long long> lds_set{0};
  if (L.note(lds_limit_once((const void*)k_wide128<R, CAUSAL, JOINT>, kMaxLds, lds_set)) !=
      hipSuccess)
    return L.err;
  const int kc = (a.band_k + 31) / 32;
  const int nseg = CAUSAL ? a.nseg : a.nseg_apply, Lw = CAUSAL ? a.L : a.L_apply;
  L(CAUSAL ? FMM_KERNEL_CAUSAL_APPLY : FMM_KERNEL_BAND_APPLY, k_wide128<R, CAUSAL, JOINT>,
    dim3(a.B * a.H * nseg), dim3(NT8), (size_t)lds_bytes(R, CAUSAL, 2 + (CAUSAL ? kc : 2 * kc)),
    (hipStream_t)a.stream, (const T*)a.q, (const T*)a.k, (const T*)a.v, (T*)a.out, recs,
    a.w_near, a.w_far, a.H, a.N, a.band_k, Lw, nseg, 1.4426950408889634f / sqrtf((float)D));
  return L.err;
}

template <int R>
hipError_t launch_r(const LaunchArgs& a, Launcher& L, const float* recs) {
  const bool joint = a.far_norm == FMM_FAR_NORM_JOINT;
  if (a.causal)
    return joint ? launch_k<R, true, true>(a, L, recs) : launch_k<R, true, false>(a, L, recs);
  return joint ? launch_k<R, false, true>(a, L, recs) : launch_k<R, false, false>(a, L, recs);
}

}  // namespace

bool wide128_applies(const LaunchArgs& a) {
  if (a.dtype != FMM_DTYPE_BF16 || a.d != D || a.rank > 2) return false;
  const long long kc = ((long long)a.band_k + 31) / 32;
  return kc <= 2 && lds_bytes(a.rank, a.causal, 2 + (int)(a.causal ? kc : 2 * kc)) <= kMaxLds;
}

hipError_t launch_wide128(const LaunchArgs& a, Launcher& L, const float* recs) {
  return a.rank == 1 ? launch_r<1>(a, L, recs) : launch_r<2>(a, L, recs);
}

}  // namespace fmm
