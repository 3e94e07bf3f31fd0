// Backward pass of the FMMformer attention operator: the gradients of a loss
// L through g = dL/dout with respect to q, k, v and the two blend logits.
// For one (batch, head) slice, with a = sigmoid(w_near), c = sigmoid(w_far):
//
//   near field (Eq. (3)), p_ij the banded softmax of tau q_i.k_j:
//     D_i = a g_i . near_i
//     ds_ij = p_ij (a g_i . v_j - D_i)
//     dq_i += tau sum_j ds_ij k_j,  dk_j += tau sum_i ds_ij q_i,
//     dv_j += a sum_i p_ij g_i
//   far field (Eq. (7)-(9)), per map l with num_i = phi(q_i)^T S(i),
//   den_i = phi(q_i)^T z(i):
//     dnum_i = c g_i / den_i,  dden_i = -c g_i . num_i / den_i^2
//     dphi(q_i) = S(i) dnum_i + z(i) dden_i
//     dS(j) = sum_{i in G(j)} phi(q_i) dnum_i^T,  dz(j) = sum_{i in G(j)} phi(q_i) dden_i
//             (G(j): every row; causal: the rows i >= j, a suffix sum)
//     dphi(k_j) = dS(j) v_j + dz(j),  dv_j += dS(j)^T phi(k_j)
//     dq += phi'(q) * dphi(q),  dk += phi'(k) * dphi(k)
//   blend (Eq. (11)): dw_near = a (1 - a) sum g . near, dw_far = c (1 - c) sum g . far
//   joint normalisation (far = sum_l num_l / Den, Den = sum_l den_l): the
//   same with dnum_i = c g_i / Den_i and dden_i = -c g_i . far_i / Den_i for
//   every map, which the row pass forms in a first sweep over the maps
//
// Launch sequence (after the forward state k_seg_state + k_state_combine):
//   k_bwd_rows   per row segment (non-causal: the apply split; causal: the
//                state segments), walking 64-row tiles: near-field softmax
//                statistics, D_i and dq; per map y = S g, from which the far
//                numerator's gradient product, dden and dq of the far field
//                follow (causal: plus the intra-tile part and the running
//                state); writes dq, the per-row softmax statistics and
//                (1/den, dden) per map, and the segment's sums of g . near and
//                g . far
//   k_seg_grad   per state segment: the partial dS = sum phi(q_i) [dnum_i |
//                dden_i]^T from q, dout and those quotients
//   k_state_combine
//                the dS partials summed per slice (non-causal) or turned into
//                exclusive suffix sums over segments (causal)
//   k_bwd_keys   per key segment (split likewise), walking 64-key tiles (last
//                tile first in the causal form): near-field dk and dv over the
//                rows whose band holds the key, the far-field dk and dv from
//                dS (causal: the segment's suffix record advanced tile by tile
//                plus the intra-tile rows i >= j); writes dk, dv; H further
//                workgroups sum the blend-logit gradients in a fixed order
//
// Fragment conventions are those of fmm_device.h: a 16-row strip per wave,
// row-quad accumulators (lane 16g + r holds row r, columns 16cb + 4g + {0..3}),
// products over 32 buffer rows through the transposed LDS reads.
#include "fmm_apply.h"
#include "fmm_device.h"
#include "fmm_launch.h"

namespace fmm {

// The fp32 passes, defined in this file's other translation units (see its
// end).
hipError_t launch_backward_f32(const BwdArgs& a, Launcher& L);
hipError_t launch_backward_f32_d128(const BwdArgs& a, Launcher& L);

namespace {

// R: feature maps.  TWO: an LDS budget of half a CU's LDS, so that two
// workgroups (two waves per SIMD) share a CU, where the rounds still hold a
// tile (FITS); else the budget of one workgroup per CU.
template <typename T, int D, int R, bool TWO = false>
struct BwdCfg {
  static constexpr int ST = D + Lay<T>::PAD;
  static constexpr int ROW = ST * (int)sizeof(T);
  static constexpr int TILE = TM * ROW;         // 64 staged rows
  static constexpr int UNIT2 = 2 * 32 * ROW;    // two buffers of one 32-row unit
  static constexpr int STAT_UNIT = 32 * 3 * 4;  // key pass: m, 1/l, D per row
  // the far-field state of the maps as rows of S (operand type) and z (fp32),
  // kept in LDS for widths up to 64; at d = 128 the fp32 records stay in
  // global memory, read through the caches
  static constexpr bool REC_LDS = D <= 64;
  static constexpr int REC_BYTES = REC_LDS ? R * D * (ROW + 4) : 0;
  // causal: the feature rows of the tile, for MG maps at a time
  static constexpr int MG = D > 64 && sizeof(T) == 4 ? 1 : R;
  static constexpr int FAR_BYTES = R * 2 * TM * 4;  // key pass: c / den, dden per map and row
  static constexpr int FIXED = MG * TILE + FAR_BYTES + 64 + REC_BYTES;
  static constexpr bool FITS = (80 * 1024 - FIXED) / (UNIT2 + STAT_UNIT) >= 2;
  static constexpr int BUDGET = TWO && FITS ? 80 * 1024 : 150 * 1024;
  static constexpr int UR_FIT = (BUDGET - FIXED) / (UNIT2 + STAT_UNIT);
  static constexpr int UR = UR_FIT > 8 ? 8 : UR_FIT;
  static_assert(UR >= 2, "a round must hold one tile");
  static constexpr int WK = 32 * UR;  // rows per staging round
  // [buffer A: WK rows][buffer B: WK rows][feature rows: MG tiles][far][stats]
  // [block sums][S rows][z]
  static constexpr int FAR_OFF = 2 * WK * ROW + MG * TILE;
  static constexpr int STAT_OFF = FAR_OFF + FAR_BYTES;
  static constexpr int RED_OFF = STAT_OFF + WK * 12;
  static constexpr int REC_OFF = RED_OFF + 64;
  static constexpr int LDS = REC_OFF + REC_BYTES;
  // windows of at most 128 rows (causal: k <= 64, else k <= 32): buffers A and
  // B are rings of 128 rows (row j at j mod 128), and only the 64 rows that the
  // next tile adds are loaded, while the current tile computes
  static constexpr bool RING = D * (int)sizeof(T) <= 128 && WK >= 128;
  // the row pass loads the tile's own q and dout rows a tile ahead (8 slices of
  // 65536 rows, d = 64, rank 2, k = 64, causal, bf16: 157 us; 161 without); the
  // key pass loads its k and v rows when the tile starts (a tile ahead it spilled:
  // 251 us; 218 so).  Both unroll the maps.  Not at d = 128, whose registers hold
  // neither; the narrower widths, with fewer registers, follow d = 64
  static constexpr bool AHEAD = D <= 64;
  static constexpr int UL = D <= 64 ? R : 1;
};

constexpr int SWB = 8;          // waves of k_seg_grad
constexpr int SNTB = SWB * 64;

// Rows [r0, r0 + n) of two [N, D] tensors (rows at or beyond kend read as
// zero) into row-major LDS buffers of stride ST.
template <typename T, int D>
__device__ __forceinline__ void stage_pair(T* sa, T* sb, const T* ha, const T* hb, int r0, int n,
                                           int kend) {
  constexpr int ST = D + Lay<T>::PAD;
  auto ident = [](int i) { return i; };
  for (int x = 0; x < n; x += 64) {
    const int m = min(64, n - x);
    RowCopy<T, D, NT, 64> ca, cb;
    ca.load(ha, r0 + x, m, kend);
    cb.load(hb, r0 + x, m, kend);
    ca.store(sa + x * ST, ST, m, ident);
    cb.store(sb + x * ST, ST, m, ident);
  }
}

// LDS row of a staged 32-row unit: rows counted from ks (a round) or mod 128
// (the ring: ks = 0).
struct StageMap {
  int ks, mask;
  __device__ __forceinline__ int operator()(int ua) const { return (ua * 32 - ks) & mask; }
};
constexpr int kRingRows = 128;

// A value loaded here whatever follows: without it, loads that only unmasked
// lanes use are sunk into branches over those lanes.
__device__ __forceinline__ void keep(float4& x) {
  asm volatile("" : "+v"(x.x), "+v"(x.y), "+v"(x.z), "+v"(x.w));
}

// The feature maps of x and their derivatives (l: 0-based map), from one
// e = exp(-|x|) for the first two.
struct PhiX {
  float x, e;
  __device__ __forceinline__ explicit PhiX(float v) : x(v), e(__expf(-fabsf(v))) {}
  __device__ __forceinline__ float phi(int l) const {
    return l == 2 ? tanhf(x) : fmaxf(1.f + (l == 0 ? x : -x), e);
  }
  __device__ __forceinline__ float dphi(int l) const {
    if (l == 0) return x > 0.f ? 1.f : e;
    if (l == 1) return x < 0.f ? -1.f : -e;
    const float t = tanhf(x);
    return 1.f - t * t;
  }
};

// The count n of a loop over maps; at d = 128 hidden from the compiler, so that
// even a single map stays a loop (flattened, its record loads all move up and
// 200 registers spill).
template <int D>
__device__ __forceinline__ int map_count(int n) {
  if constexpr (D > 64) asm volatile("" : "+s"(n));
  return n;
}

// phi_l, l = l0 .. l0 + MG - 1, of 64 rows staged at src (stride ST) into the
// tiles dst, dst + TM * ST, ...; rows at or beyond N - r0 give 0.
template <typename T, int D, int MG>
__device__ __forceinline__ void stage_phi_rows(const T* src, int r0, int N, int l0, T* dst) {
  using LY = Lay<T>;
  constexpr int ST = D + LY::PAD, CPR = D / LY::EPC;
#pragma unroll
  for (int t = threadIdx.x; t < TM * CPR; t += NT) {
    const int row = t / CPR, c = t % CPR;
    const uint4 raw = *reinterpret_cast<const uint4*>(src + row * ST + c * LY::EPC);
    const bool ok = r0 + row < N;
    float p[MG][LY::EPC];
#pragma unroll
    for (int i = 0; i < LY::EPC; ++i) {
      float x;
      if constexpr (sizeof(T) == 2) x = bf16_to_f32(reinterpret_cast<const uint16_t*>(&raw)[i]);
      else x = reinterpret_cast<const float*>(&raw)[i];
      const PhiX px(x);
#pragma unroll
      for (int m = 0; m < MG; ++m) p[m][i] = ok ? px.phi(l0 + m) : 0.f;
    }
#pragma unroll
    for (int m = 0; m < MG; ++m) {
      uint4 outw;
      if constexpr (sizeof(T) == 2) {
        outw = make_uint4(pack_bf16x2(p[m][0], p[m][1]), pack_bf16x2(p[m][2], p[m][3]),
                          pack_bf16x2(p[m][4], p[m][5]), pack_bf16x2(p[m][6], p[m][7]));
      } else {
        outw = make_uint4(__float_as_uint(p[m][0]), __float_as_uint(p[m][1]),
                          __float_as_uint(p[m][2]), __float_as_uint(p[m][3]));
      }
      *reinterpret_cast<uint4*>(dst + m * TM * ST + row * ST + c * LY::EPC) = outw;
    }
  }
}

template <typename T>
__device__ __forceinline__ typename QuadOf<T>::type rec_quad(const float* p) {
  const float4 v = *reinterpret_cast<const float4*>(p);
  const float f[4] = {v.x, v.y, v.z, v.w};
  return f32_to_quad<T>(f);
}

// Transposed values of a tile-order record: lane (r, g) gets
// X[16cb + r][16eb + 4g + {0..3}] where the record tile (cb, eb) stores
// X[16cb + 4g' + i][16eb + r'] at lane 16g' + r'.
__device__ __forceinline__ f32x4 rec_t(const float* rl, int NB, int cb, int eb) {
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const float* p = rl + ((cb * NB + eb) * 64 + 16 * (r >> 2) + 4 * g) * 4 + (r & 3);
  return f32x4{p[0], p[4], p[8], p[12]};
}

template <typename T>
__device__ __forceinline__ typename QuadOf<T>::type to_quad(const f32x4& x) {
  const float f[4] = {x[0], x[1], x[2], x[3]};
  return f32_to_quad<T>(f);
}

// The far-field state of a workgroup (forward: S_l, z_l; key pass: dS_l, dz_l).
// For d <= 64 it sits in LDS as rows S_l[c][e] in the operand type, which give
// both orders of operand (row quads along e, transposed reads along c), and z
// in fp32; the causal form carries the fp32 sums in registers, the groups (l,
// feature block cb) spread over the waves (with fewer groups than waves, some
// waves carry the same one and write the same values), and rewrites the rows
// after each tile.  At d = 128 it is the fp32 record in global memory.
template <typename T, int D, int R, bool CAUSAL>
struct FarState {
  using Q = typename QuadOf<T>::type;
  static constexpr int NB = D / 16, ST = D + Lay<T>::PAD;
  static constexpr bool REGS = CAUSAL && D <= 64;
  static constexpr int AG = R * NB, GPW = (AG + NW - 1) / NW;
  T* rows;     // [R][D][ST] (d <= 64)
  float* zs;   // [R][D]
  float* rec;  // the record (d = 128)
  f32x4 acc[REGS ? GPW : 1][NB], zacc[REGS ? GPW : 1];  // lane r: row c = 16cb + r

  __device__ __forceinline__ static int group(int w, int a) { return (w + NW * a) % AG; }
  __device__ __forceinline__ static float* map_rec(float* rc, int l) {
    return rc + (size_t)l * D * (D + 1);
  }
  __device__ __forceinline__ void init(unsigned char* lds, float* grec, int w) {
    rows = reinterpret_cast<T*>(lds);
    zs = reinterpret_cast<float*>(lds + R * D * ST * sizeof(T));
    rec = grec;
    const int lane = threadIdx.x & 63, r = lane & 15;
    if constexpr (REGS) {
#pragma unroll
      for (int a = 0; a < GPW; ++a) {
        const int ag = group(w, a), l = ag / NB, cb = ag % NB;
        const float* rl = map_rec(grec, l);
#pragma unroll
        for (int eb = 0; eb < NB; ++eb) acc[a][eb] = rec_t(rl, NB, cb, eb);
        const float z = rl[D * D + 16 * cb + r];
        zacc[a] = f32x4{z, z, z, z};
      }
      publish(w);
    } else if constexpr (D <= 64) {
      for (int t = threadIdx.x >> 6; t < R * NB * NB; t += NW) {
        const int l = t / (NB * NB), cb = t / NB % NB, eb = t % NB;
        *reinterpret_cast<Q*>(rows + (l * D + 16 * cb + r) * ST + 16 * eb + 4 * (lane >> 4)) =
            to_quad<T>(rec_t(map_rec(grec, l), NB, cb, eb));
      }
      for (int t = threadIdx.x; t < R * D; t += NT) zs[t] = map_rec(grec, t / D)[D * D + t % D];
    }
  }
  // the registers' state into the LDS rows (the caller synchronises)
  __device__ __forceinline__ void publish(int w) {
    const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
#pragma unroll
    for (int a = 0; a < GPW; ++a) {
      const int ag = group(w, a), l = ag / NB, cb = ag % NB;
#pragma unroll
      for (int eb = 0; eb < NB; ++eb)
        *reinterpret_cast<Q*>(rows + (l * D + 16 * cb + r) * ST + 16 * eb + 4 * g) =
            to_quad<T>(acc[a][eb]);
      if (g == 0) zs[l * D + 16 * cb + r] = zacc[a][0];
    }
  }
  // operand along e of feature row c = 16cb + r; operand along c of column
  // e = 16eb + r; z[16cb + 4g ..]
  __device__ __forceinline__ Q along_e(int l, int cb, int eb) const {
    const int lane = threadIdx.x & 63;
    if constexpr (D <= 64) return ld_quad(rows + (l * D + 16 * cb) * ST, lane & 15, 16 * eb + 4 * (lane >> 4), ST);
    else return to_quad<T>(rec_t(map_rec(rec, l), NB, cb, eb));
  }
  __device__ __forceinline__ Q along_c(int l, int cb, int eb) const {
    if constexpr (D <= 64) return ld_tquad(rows + (l * D + 16 * cb) * ST, 0, 16 * eb, ST);
    else return rec_quad<T>(map_rec(rec, l) + ((cb * NB + eb) * 64 + (threadIdx.x & 63)) * 4);
  }
  __device__ __forceinline__ float4 z(int l, int cb) const {
    const int g = (threadIdx.x & 63) >> 4;
    const float* p = D <= 64 ? zs + l * D : map_rec(rec, l) + D * D;
    return *reinterpret_cast<const float4*>(p + 16 * cb + 4 * g);
  }
};

// rec_l += phi(X)^T [s Y | y] over the 64 staged rows, s and y one value per
// row (SCALED: scale, else 1; y: ycol, else 1): px holds phi_l of the rows, py
// the second factor's (stride ST).  For d <= 64 into the wave's registers,
// product transposed (lane: feature c), the scale taken into phi.
template <typename T, int D, int R, bool SCALED>
__device__ __forceinline__ void state_add(FarState<T, D, R, true>& fs, const T* px, const T* py,
                                          const float* scale, const float* ycol, int l0, int MG,
                                          int w) {
  using Q = typename QuadOf<T>::type;
  using F = FarState<T, D, R, true>;
  constexpr int NB = D / 16, ST = F::ST;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  auto scaled = [&](const Q& x, const float* sc) {
    float f[4];
    quad_to_f32(x, f);
    const float4 s = *reinterpret_cast<const float4*>(sc);
    f[0] *= s.x, f[1] *= s.y, f[2] *= s.z, f[3] *= s.w;
    return f32_to_quad<T>(f);
  };
  auto col = [&](const float* y) { return rec_quad<T>(y); };
  const Q ones = quad_fill<T>(1.f);
  if constexpr (F::REGS) {
#pragma unroll
    for (int a = 0; a < F::GPW; ++a) {
      const int ag = F::group(w, a), l = ag / NB, cb = ag % NB;
      const T* p = px + l * TM * ST;
      const float* sc = scale + l * 2 * TM;
      const float* yc = ycol + l * 2 * TM;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int k0 = 32 * u + 4 * g, k1 = k0 + 16;
        const Q a0 = ld_tquad(p, 32 * u, 16 * cb, ST), a1 = ld_tquad(p, 32 * u + 16, 16 * cb, ST);
        Q s0 = a0, s1 = a1;
        if constexpr (SCALED) s0 = scaled(a0, sc + k0), s1 = scaled(a1, sc + k1);
#pragma unroll
        for (int eb = 0; eb < NB; ++eb)
          fs.acc[a][eb] = mma_step2(ld_tquad(py, 32 * u, 16 * eb, ST),
                                    ld_tquad(py, 32 * u + 16, 16 * eb, ST), s0, s1,
                                    fs.acc[a][eb]);
        if constexpr (SCALED)
          fs.zacc[a] = mma_step2(col(yc + k0), col(yc + k1), a0, a1, fs.zacc[a]);
        else
          fs.zacc[a] = mma_step2(ones, ones, a0, a1, fs.zacc[a]);
      }
    }
  } else {
    // d = 128: the record in global memory, MG maps from l0 (their feature
    // rows at px), wave w on feature blocks w, w + 4
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    for (int l = l0; l < l0 + MG; ++l) {
      float* rl = F::map_rec(fs.rec, l);
      const T* p = px + (l - l0) * TM * ST;
      const float* sc = scale + l * 2 * TM;
      const float* yc = ycol + l * 2 * TM;
      for (int cb = w; cb < NB; cb += NW) {
        f32x4 acc[NB + 1];
#pragma unroll
        for (int eb = 0; eb < NB; ++eb)
          acc[eb] = *reinterpret_cast<const f32x4*>(rl + ((cb * NB + eb) * 64 + lane) * 4);
        acc[NB] = r == 0 ? *reinterpret_cast<const f32x4*>(rl + D * D + 16 * cb + 4 * g) : zero;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int k0 = 32 * u + 4 * g, k1 = k0 + 16;
          const Q a0 = ld_tquad(p, 32 * u, 16 * cb, ST),
                  a1 = ld_tquad(p, 32 * u + 16, 16 * cb, ST);
          Q s0 = a0, s1 = a1;
          if constexpr (SCALED) s0 = scaled(a0, sc + k0), s1 = scaled(a1, sc + k1);
#pragma unroll
          for (int eb = 0; eb < NB; ++eb)
            acc[eb] = mma_step2(s0, s1, ld_tquad(py, 32 * u, 16 * eb, ST),
                                ld_tquad(py, 32 * u + 16, 16 * eb, ST), acc[eb]);
          if constexpr (SCALED) acc[NB] = mma_step2(a0, a1, col(yc + k0), col(yc + k1), acc[NB]);
          else acc[NB] = mma_step2(a0, a1, ones, ones, acc[NB]);
        }
        mfma_drain();
#pragma unroll
        for (int eb = 0; eb < NB; ++eb)
          *reinterpret_cast<f32x4*>(rl + ((cb * NB + eb) * 64 + lane) * 4) = acc[eb];
        if (r == 0) *reinterpret_cast<f32x4*>(rl + D * D + 16 * cb + 4 * g) = acc[NB];
      }
    }
  }
}

// Band validity of key j (unit-local offset 16b + 4g + i from j0) for query
// row `row`: the interval logic of near_units.
template <bool CAUSAL>
__device__ __forceinline__ void band_interval(int row, int j0, int g, int N, int band_k, int& lo,
                                              int& span) {
  lo = max(row - band_k, 0) - j0 - 4 * g;
  span = min(CAUSAL ? row : row + band_k, N - 1) - j0 - 4 * g - lo;
  if (span < 0) {
    lo = 64;
    span = 0;
  }
}

// ------------------------------------------------------------------ row pass
// Near-field dq of the strip over key units [ua_lo, ua_hi] staged through map:
// dq += tau sum_j p_ij (a g_i . v_j - D_i) k_j with p from the final row
// statistics (maximum m of the raw scores, 1/l).
template <typename T, int D, bool CAUSAL, class Map>
__device__ __forceinline__ void near_dq_units(f32x4* dq, const typename QuadOf<T>::type* qq,
                                              const typename QuadOf<T>::type* gq, const T* kr,
                                              const T* vr, int ST, Map map, int ua_lo, int ua_hi,
                                              int i0, int N, int band_k, float scale2, float ms,
                                              float inv_l, float Di, float a_tau, float a) {
  using Q = typename QuadOf<T>::type;
  constexpr int NB = D / 16;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int row = i0 + r;
  for (int ua = ua_lo; ua <= ua_hi; ++ua) {
    const T* kx = kr + map(ua) * ST;
    const T* vx = vr + map(ua) * ST;
    int lo, span;
    band_interval<CAUSAL>(row, ua * 32, g, N, band_k, lo, span);
    float ds[2][4];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      Q ka[NB], va[NB];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        ka[cb] = ld_quad(kx, 16 * b + r, 16 * cb + 4 * g, ST);
        va[cb] = ld_quad(vx, 16 * b + r, 16 * cb + 4 * g, ST);
      }
      const f32x4 s = contract<NB>(ka, qq, f32x4{0.f, 0.f, 0.f, 0.f});
      const f32x4 dp = contract<NB>(va, gq, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool ok = (unsigned)(16 * b + i - lo) <= (unsigned)span;
        const float p = ok ? __builtin_amdgcn_exp2f(fmaf(s[i], scale2, -ms)) * inv_l : 0.f;
        ds[b][i] = p * fmaf(a, dp[i], -Di) * a_tau;
      }
    }
    const Q d0 = f32_to_quad<T>(ds[0]), d1 = f32_to_quad<T>(ds[1]);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb)
      dq[cb] = mma_step2(ld_tquad(kx, 0, 16 * cb, ST), ld_tquad(kx, 16, 16 * cb, ST), d0, d1,
                         dq[cb]);
  }
  mfma_drain();
}

// Near field of the strip in one sweep, for a band of at most NUH staged units:
// the scores s = K q and dp = V g of all of them in registers, so that K and V
// are read once and no P V product is needed (g . near = sum p dp / sum p).
// Sets the scaled maximum, 1/l and D, adds dq, and returns this lane's share of
// g . near.
template <typename T, int D, bool CAUSAL, int NUH>
__device__ __forceinline__ float near_hold(f32x4* dq, const typename QuadOf<T>::type* qq,
                                           const typename QuadOf<T>::type* gq, const T* kr,
                                           const T* vr, int ST, StageMap map, int ul, int nu,
                                           int i0, int N, int band_k, float scale2, float tau,
                                           float a, bool row_ok, float& ms, float& inv_l,
                                           float& Di) {
  using Q = typename QuadOf<T>::type;
  constexpr int NB = D / 16;
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  f32x4 sc[NUH][2], dp[NUH][2];
  float m = -INFINITY;
#pragma unroll
  for (int gi = 0; gi < NUH; ++gi) {
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      sc[gi][b] = f32x4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
      dp[gi][b] = zero;
    }
    if (gi < nu) {
      const int ua = ul + gi, j0 = ua * 32;
      const T* kx = kr + map(ua) * ST;
      const T* vx = vr + map(ua) * ST;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        Q ka[NB], va[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          ka[cb] = ld_quad(kx, 16 * b + r, 16 * cb + 4 * g, ST);
          va[cb] = ld_quad(vx, 16 * b + r, 16 * cb + 4 * g, ST);
        }
        sc[gi][b] = contract<NB>(ka, qq, zero);
        dp[gi][b] = contract<NB>(va, gq, zero);
      }
      mfma_drain();  // (read on both sides of the branch)
      const bool interior = j0 >= 0 && j0 + 31 < N && j0 >= i0 + 15 - band_k &&
                            (CAUSAL ? j0 + 31 <= i0 : j0 + 31 <= i0 + band_k);
      if (!interior) {
        int lo, span;
        band_interval<CAUSAL>(i0 + r, j0, g, N, band_k, lo, span);
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if ((unsigned)(16 * b + i - lo) > (unsigned)span) sc[gi][b][i] = -INFINITY;
      }
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) m = fmaxf(m, sc[gi][b][i]);
    }
  }
  m = col_max(m);
  ms = (m == -INFINITY ? 0.f : m) * scale2;
  float l = 0.f, gn = 0.f;
#pragma unroll
  for (int gi = 0; gi < NUH; ++gi)
    if (gi < nu) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float p = __builtin_amdgcn_exp2f(fmaf(sc[gi][b][i], scale2, -ms));
          sc[gi][b][i] = p;
          l += p;
          gn = fmaf(p, dp[gi][b][i], gn);
        }
    }
  l = col_sum(l);
  inv_l = row_ok ? 1.f / l : 0.f;
  Di = a * col_sum(gn) * inv_l;
  const float it = inv_l * tau;
#pragma unroll
  for (int gi = 0; gi < NUH; ++gi)
    if (gi < nu) {
      float ds[2][4];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          ds[b][i] = sc[gi][b][i] * it * fmaf(a, dp[gi][b][i], -Di);
      const Q d0 = f32_to_quad<T>(ds[0]), d1 = f32_to_quad<T>(ds[1]);
      const T* kx = kr + map(ul + gi) * ST;
#pragma unroll
      for (int cb = 0; cb < NB; ++cb)
        dq[cb] = mma_step2(ld_tquad(kx, 0, 16 * cb, ST), ld_tquad(kx, 16, 16 * cb, ST), d0, d1,
                           dq[cb]);
    }
  mfma_drain();
  return gn * inv_l;
}

// The far field needs no numerators: with y_l = S_l g_i (one product, shared by
// the rest), g_i . num_l = phi_l(q_i) . y_l and S_l dnum_l = c y_l / den_l, and
// likewise within the tile from B_ij = v_j . g_i, which all maps share; den_l
// is a dot product with z_l.  (Forming num_l and S_l dnum_l apart took 52
// instead of about 28 products per strip and map, rounded dnum to the operand
// type, and read the state in both orders.)
template <typename T, int D, bool CAUSAL, int R, bool TWO, bool JOINT>
__global__ __launch_bounds__(NT, TWO ? 2 : 1) void k_bwd_rows(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const T* __restrict__ dout, T* __restrict__ dq, float* __restrict__ recs,
    float* __restrict__ rowstat, float* __restrict__ rowfar,
    float* __restrict__ dwpart, const float* __restrict__ w_near, const float* __restrict__ w_far,
    int H, int N, int band_k, int L, int nseg, float scale2) {
  using Q = typename QuadOf<T>::type;
  using C = BwdCfg<T, D, R, TWO>;
  constexpr int NB = D / 16, ST = C::ST, MG = C::MG, NUH = D > 64 ? 0 : CAUSAL ? 3 : 5;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
  T* sk = reinterpret_cast<T*>(dyn_smem);
  T* sv = sk + C::WK * ST;
  T* tb = sv + C::WK * ST;  // feature rows of the tile's keys (causal)
  float* red = reinterpret_cast<float*>(dyn_smem + C::RED_OFF);
  const int lin = xcd_remap(blockIdx.x, gridDim.x);
  const int bh = lin / nseg, seg = lin % nseg, h = bh % H;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const size_t base = (size_t)bh * N * D;
  const size_t REC = (size_t)R * D * (D + 1);
  const T *kh = k + base, *vh = v + base;
  FarState<T, D, R, CAUSAL> fs;
  fs.init(dyn_smem + C::REC_OFF, CAUSAL ? recs + ((size_t)bh * nseg + seg) * REC
                                        : recs + (size_t)bh * REC, w);
  const float sn = sigmoidf_exact(w_near[h]), sfw = sigmoidf_exact(w_far[h]);
  const float tau = scale2 * 0.69314718055994531f;  // 1/sqrt(d)
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  float acc_near = 0.f, acc_far = 0.f;  // this lane's share of g . near and g . far
  const int nmap = map_count<D>(R);
  const int s0 = seg * L, s1 = min(N, s0 + L);
  // key window [ka, hi) of the tile at t0
  auto window = [&](int t0, int& ka, int& hi) {
    ka = (max(0, t0 - band_k) >> 5) << 5;
    hi = CAUSAL ? t0 + TM : ((min(N, t0 + TM + band_k) + 31) & ~31);
  };
  // the ring's window of the tile at t0 ends at t0 + LEAD; the next tile's new
  // rows and its query and dout rows are loaded while the current one computes
  constexpr int LEAD = CAUSAL ? TM : TM + 32;
  const bool ring = C::RING && band_k <= (CAUSAL ? 64 : 32);
  RowCopy<T, D, NT, 64> pk, pv;
  Q qn[NB], gn[NB];
  if constexpr (C::RING) {
    if (ring)
      for (int x = s0 + LEAD - kRingRows; x < s0 + LEAD; x += 64) {
        auto at = [=](int i) { return (x + i) & (kRingRows - 1); };
        pk.load(kh, x, 64, N);
        pv.load(vh, x, 64, N);
        pk.store(sk, ST, 64, at);
        pv.store(sv, ST, 64, at);
      }
  }
  auto prefetch = [&](int t0) {
    const int row = t0 + 16 * w + r;
    if constexpr (C::AHEAD) {
      load_q<T, D>(q + base, row, t0 < s1 ? N : 0, qn);
      load_q<T, D>(dout + base, row, t0 < s1 ? N : 0, gn);
    }
    if constexpr (C::RING) {
      const int n = ring && t0 > s0 && t0 < s1 ? 64 : 0;
      pk.load(kh, t0 + LEAD - 64, n, N);
      pv.load(vh, t0 + LEAD - 64, n, N);
    }
  };
  prefetch(s0);
  for (int t0 = s0; t0 < s1; t0 += TM) {
    const int i0 = t0 + 16 * w, row = i0 + r;
    const bool row_ok = row < N;
    Q qq[NB], gq[NB];
    if constexpr (C::AHEAD) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        qq[cb] = qn[cb];
        gq[cb] = gn[cb];
      }
    } else {
      load_q<T, D>(q + base, row, N, qq);
      load_q<T, D>(dout + base, row, N, gq);
    }
    int ka, hi;
    window(t0, ka, hi);
    const int nr = ring ? 1 : (hi - ka + C::WK - 1) / C::WK;
    int ks = ring ? 0 : ka;
    const int mask = ring ? kRingRows - 1 : -1;
    f32x4 dqa[NB];
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) dqa[cb] = zero;
    float ms, inv_l, Di;
    // ---- near field
    const int blo = max(0, i0 - band_k), bhi = min(N - 1, CAUSAL ? i0 + 15 : i0 + 15 + band_k);
    if (nr == 1) {
      __syncthreads();  // every wave is done with the previous tile
      if (ring) {
        auto at = [=](int i) { return (t0 + LEAD - 64 + i) & (kRingRows - 1); };
        if (t0 > s0) {
          pk.store(sk, ST, 64, at);
          pv.store(sv, ST, 64, at);
        }
      } else {
        stage_pair<T, D>(sk, sv, kh, vh, ka, hi - ka, N);
      }
      __syncthreads();
      prefetch(t0 + TM);
      if constexpr (CAUSAL) stage_phi_rows<T, D, MG>(sk + ((t0 - ks) & mask) * ST, t0, N, 0, tb);
    }
    const int nu = blo <= bhi ? (bhi >> 5) - (blo >> 5) + 1 : 0;
    bool held = false;
    if constexpr (NUH > 0) {
      if (nr == 1 && nu <= NUH) {
        held = true;
        acc_near += near_hold<T, D, CAUSAL, NUH>(dqa, qq, gq, sk, sv, ST, StageMap{ks, mask},
                                                 blo >> 5, nu, i0, N, band_k, scale2, tau, sn, row_ok, ms,
                                                 inv_l, Di);
      }
    }
    if (!held) {
      // wider bands: the statistics first, then dq in a second sweep
      NearState<D> st;
      st.init();
      for (int rr = nr - 1; rr >= 0; --rr) {
        const int ke = hi - rr * C::WK;
        if (nr > 1) {
          ks = max(ka, ke - C::WK);
          __syncthreads();
          stage_pair<T, D>(sk, sv, kh, vh, ks, ke - ks, N);
          __syncthreads();
        }
        const int lo = nr > 1 ? max(blo, ks) : blo, hj = min(bhi, ke - 1);
        if (lo <= hj)
          near_units<T, D, CAUSAL, 2>(st, qq, sk, sv, ST, StageMap{ks, mask}, lo >> 5, hj >> 5, i0, N,
                                      band_k, scale2);
      }
      mfma_drain();
      inv_l = row_ok ? 1.f / st.o[NB][0] : 0.f;
      float gs = 0.f;  // g . (unnormalised near) over this lane's columns
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float gf[4];
        quad_to_f32(gq[nb], gf);
#pragma unroll
        for (int i = 0; i < 4; ++i) gs = fmaf(gf[i], st.o[nb][i], gs);
      }
      acc_near += gs * inv_l;
      Di = sn * col_sum(gs) * inv_l;
      ms = (st.m == -INFINITY ? 0.f : st.m) * scale2;
      for (int rr = nr - 1; rr >= 0; --rr) {
        const int ke = hi - rr * C::WK;
        if (nr > 1) {
          ks = max(ka, ke - C::WK);
          __syncthreads();
          stage_pair<T, D>(sk, sv, kh, vh, ks, ke - ks, N);
          __syncthreads();
        }
        const int lo = nr > 1 ? max(blo, ks) : blo, hj = min(bhi, ke - 1);
        if (lo <= hj)
          near_dq_units<T, D, CAUSAL>(dqa, qq, gq, sk, sv, ST, StageMap{ks, mask}, lo >> 5, hj >> 5, i0,
                                      N, band_k, scale2, ms, inv_l, Di, tau, sn);
      }
      if (nr > 1) {
        prefetch(t0 + TM);
        if constexpr (CAUSAL) stage_phi_rows<T, D, MG>(sk + (t0 - ks) * ST, t0, N, 0, tb);
      }
    }
    if (row_ok && g == 0) {
      float* sp = rowstat + ((size_t)bh * N + row) * 3;
      sp[0] = ms;
      sp[1] = inv_l;
      sp[2] = Di;
    }
    // ---- far field; the tile's keys sit at rows t0 - ks of the last round
    const int rt = (t0 - ks) & mask;
    const T* vt = sv + rt * ST;
    f32x4 B[2][2];  // v_j . g_i of the tile's keys up to the strip's unit
    if constexpr (CAUSAL) {
      __syncthreads();  // the feature rows are in tb
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          B[u][b] = zero;
          if (u <= (w >> 1)) {
            Q va[NB];
#pragma unroll
            for (int eb = 0; eb < NB; ++eb)
              va[eb] = ld_quad(vt, 32 * u + 16 * b + r, 16 * eb + 4 * g, ST);
            B[u][b] = contract<NB>(va, gq, zero);
          }
        }
      mfma_drain();
    }
    // key 32u + 16b + 4g + i of the tile is at or before the lane's row
    auto seen = [&](int u, int b, int i) { return 32 * u + 16 * b + 4 * g + i <= 16 * w + r; };
    // the feature rows of map l in tb (staged again where tb holds fewer maps)
    auto map_rows = [&](int l) -> const T* {
      if constexpr (MG < R && CAUSAL) {
        __syncthreads();
        stage_phi_rows<T, D, MG>(sk + rt * ST, t0, N, l, tb);
        __syncthreads();
        return tb;
      } else {
        return tb + l * TM * ST;
      }
    };
    auto product_y = [&](int l, f32x4* y) {
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        Q a[NB];
#pragma unroll
        for (int eb = 0; eb < NB; ++eb) a[eb] = fs.along_e(l, cb, eb);
        y[cb] = contract<NB>(a, gq, zero);
      }
    };
    // this lane's shares of den and g . num of map l, given y
    auto sums = [&](int l, const T* px, const f32x4* y, float& den, float& gnum) {
      Q pq[NB];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        const float4 z4 = fs.z(l, cb);
        const float zf[4] = {z4.x, z4.y, z4.z, z4.w};
        float x[4], p[4];
        quad_to_f32(qq[cb], x);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          p[i] = PhiX(x[i]).phi(l);
          den = fmaf(p[i], zf[i], den);
          gnum = fmaf(p[i], y[cb][i], gnum);
        }
        pq[cb] = f32_to_quad<T>(p);
      }
      if constexpr (CAUSAL) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (u <= (w >> 1)) {
            f32x4 at[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
              Q ka2[NB];
#pragma unroll
              for (int cb = 0; cb < NB; ++cb)
                ka2[cb] = ld_quad(px, 32 * u + 16 * b + r, 16 * cb + 4 * g, ST);
              at[b] = contract<NB>(ka2, pq, zero);
            }
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const float s = seen(u, b, i) ? at[b][i] : 0.f;
                den += s;
                gnum = fmaf(s, B[u][b][i], gnum);
              }
          }
      }
    };
    // dq of map l: phi_l'(q) (c y / den + dden z + the tile's keys)
    auto far_dq = [&](int l, const T* px, const f32x4* y, float cid, float dden) {
      f32x4 dph[NB];
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        const float4 z4 = fs.z(l, cb);
        const float zf[4] = {z4.x, z4.y, z4.z, z4.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) dph[cb][i] = fmaf(cid, y[cb][i], dden * zf[i]);
      }
      if constexpr (CAUSAL) {
#pragma unroll
        for (int u = 0; u < 2; ++u)
          if (u <= (w >> 1)) {
            float c2[2][4];
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int i = 0; i < 4; ++i)
                c2[b][i] = seen(u, b, i) ? fmaf(cid, B[u][b][i], dden) : 0.f;
            const Q p0 = f32_to_quad<T>(c2[0]), p1 = f32_to_quad<T>(c2[1]);
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
              dph[cb] = mma_step2(ld_tquad(px, 32 * u, 16 * cb, ST),
                                  ld_tquad(px, 32 * u + 16, 16 * cb, ST), p0, p1, dph[cb]);
          }
        mfma_drain();
      }
#pragma unroll
      for (int cb = 0; cb < NB; ++cb) {
        float x[4];
        quad_to_f32(qq[cb], x);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          dqa[cb][i] = fmaf(PhiX(x[i]).dphi(l), dph[cb][i], dqa[cb][i]);
      }
    };
    auto put_far = [&](int l, float inv_den, float dden) {
      if (row_ok && g == 0)
        *reinterpret_cast<float2*>(rowfar + (((size_t)bh * N + row) * R + l) * 2) =
            make_float2(inv_den, dden);
    };
    // advance the forward prefix by the tile's keys of the maps in tb, unless
    // this is the segment's last tile (d <= 64: in registers, all maps at once)
    auto advance = [&](int l) {
      if constexpr (CAUSAL && D > 64) {
        if (t0 + TM < s1) {
          __syncthreads();  // every wave has read the records
          state_add<T, D, R, false>(fs, MG < R ? tb : tb + l * TM * ST, vt, nullptr, nullptr, l, 1,
                                    w);
        }
      }
    };
    if constexpr (!JOINT) {
#pragma unroll C::UL
      for (int l = 0; l < nmap; ++l) {
        const T* px = map_rows(l);
        f32x4 y[NB];
        product_y(l, y);
        float den = 0.f, gnum = 0.f;
        sums(l, px, y, den, gnum);
        const float inv_den = row_ok ? fast_rcp(col_sum(den)) : 0.f;
        acc_far += gnum * inv_den;
        const float dden = -sfw * col_sum(gnum) * inv_den * inv_den;
        put_far(l, inv_den, dden);
        far_dq(l, px, y, sfw * inv_den, dden);
        advance(l);
      }
    } else {
      // one quotient for all maps: far = sum_l num_l / Den, Den = sum_l den_l,
      // so dnum_l = c g / Den and dden_l = -c g . (sum_l num_l) / Den^2
      float den = 0.f, gsum = 0.f;
#pragma unroll C::UL
      for (int l = 0; l < nmap; ++l) {
        const T* px = map_rows(l);
        f32x4 y[NB];
        product_y(l, y);
        sums(l, px, y, den, gsum);
      }
      const float inv_den = row_ok ? fast_rcp(col_sum(den)) : 0.f;
      acc_far += gsum * inv_den;
      const float dden = -sfw * col_sum(gsum) * inv_den * inv_den;
#pragma unroll C::UL
      for (int l = 0; l < nmap; ++l) {
        const T* px = map_rows(l);
        f32x4 y[NB];
        product_y(l, y);
        put_far(l, inv_den, dden);
        far_dq(l, px, y, sfw * inv_den, dden);
        advance(l);
      }
    }
    store_row<T, D>(dq + base, row, N, dqa);
    if constexpr (CAUSAL && D <= 64) {
      if (t0 + TM < s1) {
        state_add<T, D, R, false>(fs, tb, vt, nullptr, nullptr, 0, R, w);
        mfma_drain();
        __syncthreads();  // every wave has read the state's rows
        fs.publish(w);
      }
    }
  }
  // the segment's sums of g . near and g . far, in a fixed order: a butterfly
  // within each wave, then the waves in order
  acc_near = wave_sum(acc_near);
  acc_far = wave_sum(acc_far);
  __syncthreads();
  if (lane == 0) {
    red[2 * w] = acc_near;
    red[2 * w + 1] = acc_far;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    float s = 0.f;
#pragma unroll
    for (int t = 0; t < NW; ++t) s += red[2 * t + threadIdx.x];
    dwpart[((size_t)bh * nseg + seg) * 2 + threadIdx.x] = s;
  }
}

// ------------------------------------------------------------------ dS partials
// Per state segment, the far-field gradient state of map l:
//   dS_l = sum_i phi_l(q_i) dnum_i^T,  dz_l = sum_i phi_l(q_i) dden_i,
//   dnum_i = c g_i / den_l,i  (c = sigmoid(w_far[h]))
// from q, dout and the row pass's (1/den, dden), in the record's tile order.
// Same structure as k_seg_state: 8 waves, (rs, cb) = wave split of the
// 32-row units and feature block, 64-row chunks staged in LDS, a fixed-order
// tree over the waves sharing a feature block.
template <typename T, int D, int R>
__global__ __launch_bounds__(SNTB) void k_seg_grad(const T* __restrict__ q,
                                                   const T* __restrict__ dout,
                                                   const float* __restrict__ rowfar,
                                                   const float* __restrict__ w_far,
                                                   float* __restrict__ dpart, int H, int N, int L,
                                                   int nseg) {
  using Q = typename QuadOf<T>::type;
  constexpr int NB = D / 16;
  constexpr int ST = D + Lay<T>::PAD;
  constexpr int RS = SWB / NB > 0 ? SWB / NB : 1;
  constexpr int TK = 64;
  // two 64-row chunks of q and dout double-buffered (the next chunk's loads
  // in flight during the current one's products), reused for the reduction
  // tree at the end
  constexpr int STAGE = 2 * 2 * TK * ST * (int)sizeof(T);
  constexpr int REDB = SWB / 2 * (NB + 1) * 64 * 16;
  __shared__ __attribute__((aligned(16))) unsigned char s_buf[STAGE > REDB ? STAGE : REDB];
  __shared__ __attribute__((aligned(16))) float s_sc[2][R][TK], s_dd[2][R][TK];
  const int seg = blockIdx.x % nseg, bh = blockIdx.x / nseg, h = bh % H;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int cbw = w % NB, rs = w / NB;
  const bool owner = w < NB * RS;
  const int r0 = seg * L, r1 = min(N, r0 + L);
  const size_t base = (size_t)bh * N * D;
  const float sfw = sigmoidf_exact(w_far[h]);
  const int nchunk = (r1 - r0 + TK - 1) / TK;
  f32x4 acc[R][NB + 1];
#pragma unroll
  for (int l = 0; l < R; ++l)
#pragma unroll
    for (int eb = 0; eb <= NB; ++eb) acc[l][eb] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto ident = [](int i) { return i; };
  // a chunk's per-row (c / den, dden) pairs: thread t < R TK holds map t / TK,
  // row t % TK (zeros past the segment)
  // (a buffer over the segment's rows: pairs past it read as zeros, so the
  // loads need no branch)
  static_assert(R * TK <= SNTB, "one pair per thread");
  const __amdgpu_buffer_rsrc_t far_rs = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(rowfar + ((size_t)bh * N + r0) * R * 2), 0, (r1 - r0) * R * 8,
      0x00020000);
  auto load_far = [&](int c0) {
    const int t = threadIdx.x, l = t / TK, i = t % TK;
    const bool on = t < R * TK && c0 + i < r1;
    const uint32_t off = on ? (uint32_t)(((c0 - r0 + i) * R + l) * 8) : 0x80000000u;
    return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(far_rs, off, 0, 0));
  };
  auto store_far = [&](int buf, float2 f) {
    const int t = threadIdx.x;
    if (t < R * TK) {
      s_sc[buf][t / TK][t % TK] = sfw * f.x;
      s_dd[buf][t / TK][t % TK] = f.y;
    }
  };
  auto sq_of = [&](int buf) { return reinterpret_cast<T*>(s_buf) + buf * 2 * TK * ST; };
  // the first two chunks' loads together, the first stored
  RowCopy<T, D, SNTB, TK> cq, cg, cq0, cg0;
  cq0.load(q + base, r0, min(TK, r1 - r0), r1);
  cg0.load(dout + base, r0, min(TK, r1 - r0), r1);
  float2 f0 = load_far(r0);
  cq.load(q + base, r0 + TK, min(TK, r1 - r0 - TK), r1);
  cg.load(dout + base, r0 + TK, min(TK, r1 - r0 - TK), r1);
  float2 f1 = load_far(r0 + TK);
  cq0.store(sq_of(0), ST, TK, ident);
  cg0.store(sq_of(0) + TK * ST, ST, TK, ident);
  store_far(0, f0);
  for (int c = 0; c < nchunk; ++c) {
    const int c0 = r0 + c * TK;
    __syncthreads();  // chunk c is in its buffer; chunk c - 1's buffer is free
    if (c + 1 < nchunk) {
      cq.store(sq_of((c + 1) & 1), ST, TK, ident);
      cg.store(sq_of((c + 1) & 1) + TK * ST, ST, TK, ident);
      store_far((c + 1) & 1, f1);
    }
    if (c + 2 < nchunk) {
      const int cn = c0 + 2 * TK;
      cq.load(q + base, cn, min(TK, r1 - cn), r1);
      cg.load(dout + base, cn, min(TK, r1 - cn), r1);
      f1 = load_far(cn);
    }
    const T* s_q = sq_of(c & 1);
    const T* s_g = s_q + TK * ST;
    const float(*sc)[TK] = s_sc[c & 1];
    const float(*dd)[TK] = s_dd[c & 1];
    if (owner) {
#pragma unroll
      for (int u = 0; u < TK / 32; ++u) {
        if ((u % RS) != rs) continue;
        // dS = (phi(q) c / den)^T g: the scale goes into phi, one operand for
        // every value block, and g stays as read (scaling g took 3 vector
        // instructions per value, map and block)
        float qf[2][4];
        Q g0[NB], g1[NB];
#pragma unroll
        for (int b = 0; b < 2; ++b) quad_to_f32(ld_tquad(s_q, 32 * u + 16 * b, 16 * cbw, ST), qf[b]);
#pragma unroll
        for (int eb = 0; eb < NB; ++eb) {
          g0[eb] = ld_tquad(s_g, 32 * u, 16 * eb, ST);
          g1[eb] = ld_tquad(s_g, 32 * u + 16, 16 * eb, ST);
        }
#pragma unroll
        for (int l = 0; l < R; ++l) {
          float pa[2][4], ps[2][4], zb[2][4];
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            const int r4 = 32 * u + 16 * b + 4 * g;
            const float4 s4 = *reinterpret_cast<const float4*>(&sc[l][r4]);
            const float4 d4 = *reinterpret_cast<const float4*>(&dd[l][r4]);
            const float sf[4] = {s4.x, s4.y, s4.z, s4.w}, df[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              pa[b][i] = c0 + r4 + i < r1 ? PhiX(qf[b][i]).phi(l) : 0.f;
              ps[b][i] = pa[b][i] * sf[i];
              zb[b][i] = r == 0 ? df[i] : 0.f;
            }
          }
          const Q a0 = f32_to_quad<T>(ps[0]), a1 = f32_to_quad<T>(ps[1]);
#pragma unroll
          for (int eb = 0; eb < NB; ++eb) acc[l][eb] = mma_step2(a0, a1, g0[eb], g1[eb], acc[l][eb]);
          acc[l][NB] = mma_step2(f32_to_quad<T>(pa[0]), f32_to_quad<T>(pa[1]),
                                 f32_to_quad<T>(zb[0]), f32_to_quad<T>(zb[1]), acc[l][NB]);
        }
      }
    }
  }
  mfma_drain();
  // fixed-order tree over the RS waves of a feature block, through s_q
  f32x4* red = reinterpret_cast<f32x4*>(s_buf);
#pragma unroll
  for (int l = 0; l < R; ++l) {
#pragma unroll
    for (int st = RS / 2; st >= 1; st >>= 1) {
      __syncthreads();
      if (owner && rs >= st && rs < 2 * st)
#pragma unroll
        for (int eb = 0; eb <= NB; ++eb)
          red[(((rs - st) * NB + cbw) * (NB + 1) + eb) * 64 + lane] = acc[l][eb];
      __syncthreads();
      if (owner && rs < st)
#pragma unroll
        for (int eb = 0; eb <= NB; ++eb)
          acc[l][eb] += red[((rs * NB + cbw) * (NB + 1) + eb) * 64 + lane];
    }
  }
  if (!owner || rs != 0) return;
  float* outp = dpart + ((size_t)bh * nseg + seg) * (R * D * (D + 1));
#pragma unroll
  for (int l = 0; l < R; ++l) {
    float* sl = outp + (size_t)l * D * (D + 1);
#pragma unroll
    for (int eb = 0; eb < NB; ++eb)
      *reinterpret_cast<f32x4*>(sl + ((cbw * NB + eb) * 64 + lane) * 4) = acc[l][eb];
    if (r == 0) *reinterpret_cast<f32x4*>(sl + D * D + 16 * cbw + 4 * g) = acc[l][NB];
  }
}

// ------------------------------------------------------------------ dw
// The blend-logit gradients of head h from the row pass's sums per segment
// and batch, by one workgroup: each thread's share in index order, then a
// butterfly per wave and the waves in order (float64, so that the order of
// thousands of partial sums does not show).  Runs as H extra workgroups of the
// key pass: as a kernel of its own with one thread per head it was a chain of
// B * nseg dependent loads (16.8 us at B = 32, nseg = 6; 7-8 us for the other
// shapes) after everything else had ended.
__device__ __forceinline__ void dw_reduce(const float* dwpart, const float* w_near,
                                          const float* w_far, float* dw_near, float* dw_far,
                                          int h, int B, int H, int nseg, double* red) {
  double s[2] = {0.0, 0.0};
  const long long n = (long long)B * nseg;
  for (long long t = threadIdx.x; t < n; t += NT) {
    const size_t b = (size_t)(t / nseg), sg = (size_t)(t % nseg);
    const float2 p = *reinterpret_cast<const float2*>(dwpart + ((b * H + h) * nseg + sg) * 2);
    s[0] += p.x;
    s[1] += p.y;
  }
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1)
#pragma unroll
    for (int x = 0; x < 2; ++x) s[x] += __shfl_xor(s[x], m);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[2 * w] = s[0];
    red[2 * w + 1] = s[1];
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double x = 0.0;
#pragma unroll
    for (int t = 0; t < NW; ++t) x += red[2 * t + threadIdx.x];
    const float a = sigmoidf_exact((threadIdx.x == 0 ? w_near : w_far)[h]);
    (threadIdx.x == 0 ? dw_near : dw_far)[h] = a * (1.f - a) * (float)x;
  }
}

// ------------------------------------------------------------------ key pass
// The last H workgroups of the grid form the blend-logit gradients.
// Within the tile (causal, rows i >= j), with E_ij = phi_l(q_i) . phi_l(k_j) and
// B_ij = g_i . v_j shared by the maps: dphi_l(k_j) += sum_i phi_l(q_i) (c B_ij /
// den_i + dden_i), and dv_j += sum_i g_i sum_l c E_ij / den_i, one product for
// all maps.  The rows of the unit before the strip's are all earlier than its
// keys and have weight zero, but a product with a zero still carries a NaN or
// infinity: there both products read the strip's own unit instead (leaving
// them out behind a branch spilled: whole forward and backward at 2^16 tokens
// 551 us, 494 so).
template <typename T, int D, bool CAUSAL, int R, bool TWO>
__global__ __launch_bounds__(NT, TWO ? 2 : 1) void k_bwd_keys(
    const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
    const T* __restrict__ dout, T* __restrict__ dk, T* __restrict__ dv, float* __restrict__ drecs,
    const float* __restrict__ rowstat, const float* __restrict__ rowfar,
    const float* __restrict__ w_near, const float* __restrict__ w_far, int H, int N, int band_k,
    int L, int nseg, float scale2, const float* __restrict__ dwpart,
    float* __restrict__ dw_near, float* __restrict__ dw_far, int Bn) {
  using Q = typename QuadOf<T>::type;
  using C = BwdCfg<T, D, R, TWO>;
  constexpr int NB = D / 16, ST = C::ST, MG = C::MG;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
  const int nwalk = gridDim.x - H;
  if ((int)blockIdx.x >= nwalk) {
    dw_reduce(dwpart, w_near, w_far, dw_near, dw_far, blockIdx.x - nwalk, Bn, H, nseg,
              reinterpret_cast<double*>(dyn_smem));
    return;
  }
  T* sq = reinterpret_cast<T*>(dyn_smem);
  T* sg = sq + C::WK * ST;
  T* tb = sg + C::WK * ST;  // feature rows of the tile's query rows (causal)
  float* far = reinterpret_cast<float*>(dyn_smem + C::FAR_OFF);  // [R][c / den, dden][64]
  float* sm = reinterpret_cast<float*>(dyn_smem + C::STAT_OFF);  // per staged row
  float* sli = sm + C::WK;
  float* sD = sm + 2 * C::WK;
  const int lin = xcd_remap(blockIdx.x, nwalk);
  const int bh = lin / nseg, seg = lin % nseg, h = bh % H;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const size_t base = (size_t)bh * N * D;
  const size_t REC = (size_t)R * D * (D + 1);
  const T *qh = q + base, *gh = dout + base;
  FarState<T, D, R, CAUSAL> fs;
  fs.init(dyn_smem + C::REC_OFF, CAUSAL ? drecs + ((size_t)bh * nseg + seg) * REC
                                        : drecs + (size_t)bh * REC, w);
  const float sn = sigmoidf_exact(w_near[h]), sfw = sigmoidf_exact(w_far[h]);
  const float tau = scale2 * 0.69314718055994531f;
  const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
  const int nmap = map_count<D>(MG);
  const int s0 = seg * L, s1 = min(N, s0 + L);
  const int ntile = (s1 - s0 + TM - 1) / TM;
  // causal: last tile first, so that the suffix record covers the rows after
  // the tile
  auto tile_at = [&](int tt) { return CAUSAL ? s0 + (ntile - 1 - tt) * TM : s0 + tt * TM; };
  // rows [ra, rb) whose band can hold the tile's keys (causal: at least the
  // tile's own, which the far part reads)
  auto window = [&](int t0, int& ra, int& rb) {
    ra = CAUSAL ? t0 : (max(0, t0 - band_k) >> 5) << 5;
    rb = (min(N, t0 + TM + band_k) + 31) & ~31;
    if (CAUSAL) rb = max(rb, t0 + TM);
  };
  // the ring holds the rows [t0, t0 + 128) (causal, walked downwards) or
  // [t0 - 32, t0 + 96); the next tile's new rows, their statistics and
  // its rows' far quotients are loaded while the current one computes
  const bool ring = C::RING && band_k <= (CAUSAL ? 64 : 32);
  const int mask = ring ? kRingRows - 1 : -1;
  auto new_rows = [&](int t0) { return CAUSAL ? t0 : t0 + 32; };
  RowCopy<T, D, NT, 64> pq, pg;
  float pst[3];
  float2 pfar = make_float2(0.f, 0.f);
  auto load_rows = [&](int x, int n) {
    pq.load(qh, x, n, N);
    pg.load(gh, x, n, N);
    const int i = min(max(x + (int)(threadIdx.x & 63), 0), N - 1);
    const float* sp = rowstat + ((size_t)bh * N + i) * 3;
#pragma unroll
    for (int m = 0; m < 3; ++m) pst[m] = sp[m];
  };
  auto store_rows = [&](int x) {
    auto at = [=](int i) { return (x + i) & (kRingRows - 1); };
    pq.store(sq, ST, 64, at);
    pg.store(sg, ST, 64, at);
    if (threadIdx.x < 64) {
      const int i = at(threadIdx.x);
      const bool ok = x + (int)threadIdx.x >= 0 && x + (int)threadIdx.x < N;
      sm[i] = ok ? pst[0] : 0.f;
      sli[i] = ok ? pst[1] : 0.f;
      sD[i] = ok ? pst[2] : 0.f;
    }
  };
  if constexpr (C::RING) {
    if (ring) {
      const int x0 = new_rows(tile_at(0)) + (CAUSAL ? 64 : -64);
      load_rows(x0, 64);
      store_rows(x0);
    }
  }
  auto prefetch = [&](int tt) {
    const bool on = tt < ntile;
    const int t0 = on ? tile_at(tt) : s0;
    if constexpr (C::RING) load_rows(new_rows(t0), ring && on ? 64 : 0);
    if constexpr (CAUSAL) {
      const int l = min((int)threadIdx.x / TM, R - 1), i = min(t0 + (int)threadIdx.x % TM, N - 1);
      pfar = *reinterpret_cast<const float2*>(rowfar + (((size_t)bh * N + i) * R + l) * 2);
    }
  };
  prefetch(0);
  for (int tt = 0; tt < ntile; ++tt) {
    const int t0 = tile_at(tt);
    const int j0 = t0 + 16 * w, key = j0 + r;
    Q kq[NB], vq[NB];
    f32x4 dka[NB], dva[NB];
    load_q<T, D>(k + base, key, N, kq);
    load_q<T, D>(v + base, key, N, vq);
#pragma unroll
    for (int cb = 0; cb < NB; ++cb) {
      dka[cb] = zero;
      dva[cb] = zero;
    }
    const float2 rf = pfar;
    // ---- near field over the rows whose band holds the strip's keys
    int ra, rb;
    window(t0, ra, rb);
    const bool one_round = ring || rb - ra <= C::WK;
    const int tr = ring ? t0 & (kRingRows - 1) : 0;  // LDS row of the tile's first row (causal)
    for (int rs = ra; rs < rb; rs += C::WK) {
      const int nrow = min(C::WK, rb - rs);
      __syncthreads();
      if (ring) {
        store_rows(new_rows(t0));
      } else {
        stage_pair<T, D>(sq, sg, qh, gh, rs, nrow, N);
        for (int t = threadIdx.x; t < nrow; t += NT) {
          const int i = rs + t;
          const bool ok = i < N;
          const float* sp = rowstat + ((size_t)bh * N + (ok ? i : 0)) * 3;
          sm[t] = ok ? sp[0] : 0.f;
          sli[t] = ok ? sp[1] : 0.f;
          sD[t] = ok ? sp[2] : 0.f;
        }
      }
      if (CAUSAL && rs == ra && (int)threadIdx.x < R * TM) {
        const int l = threadIdx.x / TM, i = threadIdx.x % TM;
        const bool ok = t0 + i < N;
        far[l * 2 * TM + i] = ok ? sfw * rf.x : 0.f;
        far[l * 2 * TM + TM + i] = ok ? rf.y : 0.f;
      }
      __syncthreads();
      if constexpr (CAUSAL)
        if (one_round) stage_phi_rows<T, D, MG>(sq + tr * ST, t0, N, 0, tb);
      // rows of this round that can hold the strip's keys in their band
      const int lo = max(max(0, j0 - (CAUSAL ? 0 : band_k)), rs);
      const int hj = min(min(N - 1, j0 + 15 + band_k), rs + nrow - 1);
      // rows whose band holds this lane's key: [rlo, rhi] (empty past N)
      const int rlo = max(key - (CAUSAL ? 0 : band_k), 0);
      const int rhi = key < N ? min(key + band_k, N - 1) : -1;
      for (int ua = lo >> 5; ua <= (hj >> 5) && lo <= hj; ++ua) {
        const int ur = (ua * 32 - (ring ? 0 : rs)) & mask;  // LDS row of the unit
        const T* qx = sq + ur * ST;
        const T* gx = sg + ur * ST;
        // unit-local row offsets c = 16b + i of this lane group (rows
        // ua*32 + 4g + c) inside the interval
        int ilo = rlo - ua * 32 - 4 * g, ispan = rhi - rlo;
        if (ispan < 0) { ilo = 64; ispan = 0; }
        float pp[2][4], ds[2][4];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          Q qa[NB], ga[NB];
#pragma unroll
          for (int cb = 0; cb < NB; ++cb) {
            qa[cb] = ld_quad(qx, 16 * b + r, 16 * cb + 4 * g, ST);
            ga[cb] = ld_quad(gx, 16 * b + r, 16 * cb + 4 * g, ST);
          }
          const f32x4 s = contract<NB>(qa, kq, zero);
          const f32x4 dp = contract<NB>(ga, vq, zero);
          const int lr0 = ur + 16 * b + 4 * g;  // staged rows lr0 .. lr0+3
          const float4 m4 = *reinterpret_cast<const float4*>(sm + lr0);
          const float4 l4 = *reinterpret_cast<const float4*>(sli + lr0);
          const float4 d4 = *reinterpret_cast<const float4*>(sD + lr0);
          const float mv[4] = {m4.x, m4.y, m4.z, m4.w}, lv[4] = {l4.x, l4.y, l4.z, l4.w},
                      dv4[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const bool ok = (unsigned)(16 * b + i - ilo) <= (unsigned)ispan;
            const float p = ok ? __builtin_amdgcn_exp2f(fmaf(s[i], scale2, -mv[i])) * lv[i] : 0.f;
            pp[b][i] = p * sn;
            ds[b][i] = p * fmaf(sn, dp[i], -dv4[i]) * tau;
          }
        }
        const Q p0 = f32_to_quad<T>(pp[0]), p1 = f32_to_quad<T>(pp[1]);
        const Q d0 = f32_to_quad<T>(ds[0]), d1 = f32_to_quad<T>(ds[1]);
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          dva[cb] = mma_step2(ld_tquad(gx, 0, 16 * cb, ST), ld_tquad(gx, 16, 16 * cb, ST), p0, p1,
                              dva[cb]);
          dka[cb] = mma_step2(ld_tquad(qx, 0, 16 * cb, ST), ld_tquad(qx, 16, 16 * cb, ST), d0, d1,
                              dka[cb]);
        }
      }
      mfma_drain();
    }
    // ---- far field
    const T* gt = sg + tr * ST;  // the tile's dout rows
    // g_i . v_j of the tile's rows
    f32x4 B[2][2];
    if constexpr (CAUSAL) {
      if (!one_round) {
        // the tile's rows again
        __syncthreads();
        stage_pair<T, D>(sq, sg, qh, gh, t0, TM, N);
        __syncthreads();
        stage_phi_rows<T, D, MG>(sq, t0, N, 0, tb);
      }
      __syncthreads();  // the feature rows are in tb
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          Q ga[NB];
#pragma unroll
          for (int eb = 0; eb < NB; ++eb)
            ga[eb] = ld_quad(gt, 32 * u + 16 * b + r, 16 * eb + 4 * g, ST);
          B[u][b] = contract<NB>(ga, vq, zero);
        }
    }
    auto seen = [&](int u, int b, int i) { return 32 * u + 16 * b + 4 * g + i >= 16 * w + r; };
#pragma unroll 1
    for (int l0 = 0; l0 < R; l0 += MG) {
      float W[2][2][4];  // sum_l c E / den of the maps in tb
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) W[u][b][i] = 0.f;
      if constexpr (CAUSAL) {
        if (l0 > 0) {
          __syncthreads();
          stage_phi_rows<T, D, MG>(sq + tr * ST, t0, N, l0, tb);
          __syncthreads();
        }
      }
#pragma unroll C::UL
      for (int m = 0; m < nmap; ++m) {
        const int l = l0 + m;
        const T* px = tb + m * TM * ST;
        Q pk[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          float x[4], p[4];
          quad_to_f32(kq[cb], x);
#pragma unroll
          for (int i = 0; i < 4; ++i) p[i] = PhiX(x[i]).phi(l);
          pk[cb] = f32_to_quad<T>(p);
        }
        // dphi(k) = dS v + dz, dv += dS^T phi(k)
        f32x4 dph[NB];
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          const float4 z = fs.z(l, cb);
          Q a[NB];
#pragma unroll
          for (int eb = 0; eb < NB; ++eb) a[eb] = fs.along_e(l, cb, eb);
          dph[cb] = contract<NB>(a, vq, f32x4{z.x, z.y, z.z, z.w});
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int eb = 0; eb < NB; ++eb) {
          Q a[NB];
#pragma unroll
          for (int cb = 0; cb < NB; ++cb) a[cb] = fs.along_c(l, cb, eb);
          dva[eb] = contract<NB>(a, pk, dva[eb]);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (CAUSAL) {
          const float* cd = far + l * 2 * TM;
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            float cc[2][4];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
              Q fa[NB];
#pragma unroll
              for (int cb = 0; cb < NB; ++cb)
                fa[cb] = ld_quad(px, 32 * u + 16 * b + r, 16 * cb + 4 * g, ST);
              const f32x4 e1 = contract<NB>(fa, pk, zero);
              const int lr = 32 * u + 16 * b + 4 * g;
              float4 c4 = *reinterpret_cast<const float4*>(cd + lr);
              float4 d4 = *reinterpret_cast<const float4*>(cd + TM + lr);
              keep(c4), keep(d4);
              const float cf[4] = {c4.x, c4.y, c4.z, c4.w}, df[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                const bool ok = seen(u, b, i);
                cc[b][i] = ok ? fmaf(cf[i], B[u][b][i], df[i]) : 0.f;
                W[u][b][i] += ok ? e1[i] * cf[i] : 0.f;
              }
            }
            const Q c0q = f32_to_quad<T>(cc[0]), c1q = f32_to_quad<T>(cc[1]);
            const T* pu = px + 32 * max(u, w >> 1) * ST;
#pragma unroll
            for (int cb = 0; cb < NB; ++cb)
              dph[cb] = mma_step2(ld_tquad(pu, 0, 16 * cb, ST), ld_tquad(pu, 16, 16 * cb, ST),
                                  c0q, c1q, dph[cb]);
          }
        }
        mfma_drain();
#pragma unroll
        for (int cb = 0; cb < NB; ++cb) {
          float x[4];
          quad_to_f32(kq[cb], x);
#pragma unroll
          for (int i = 0; i < 4; ++i)
            dka[cb][i] = fmaf(PhiX(x[i]).dphi(l), dph[cb][i], dka[cb][i]);
        }
      }
      if constexpr (CAUSAL) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const Q e0 = f32_to_quad<T>(W[u][0]), e1 = f32_to_quad<T>(W[u][1]);
          const T* gu = gt + 32 * max(u, w >> 1) * ST;
#pragma unroll
          for (int eb = 0; eb < NB; ++eb)
            dva[eb] = mma_step2(ld_tquad(gu, 0, 16 * eb, ST), ld_tquad(gu, 16, 16 * eb, ST), e0,
                                e1, dva[eb]);
        }
        mfma_drain();
        // d = 128: the suffix record takes the tile's rows, unless this is the
        // segment's first tile (the last one walked)
        if constexpr (D > 64) {
          if (tt + 1 < ntile) {
            __syncthreads();  // every wave has read the records
            state_add<T, D, R, true>(fs, tb, gt, far, far + TM, l0, MG, w);
          }
        }
      }
    }
    // (after the far field: issued behind the staging, the loads' registers made
    // the pass spill, 218 us; here 192)
    prefetch(tt + 1);
    store_row<T, D>(dk + base, key, N, dka);
    store_row<T, D>(dv + base, key, N, dva);
    if constexpr (CAUSAL && D <= 64) {
      if (tt + 1 < ntile) {
        state_add<T, D, R, true>(fs, tb, gt, far, far + TM, 0, R, w);
        mfma_drain();
        __syncthreads();  // every wave has read the state's rows
        fs.publish(w);
      }
    }
  }
}

template <typename T, int D, bool CAUSAL, int R, bool TWO>
hipError_t launch_bwd_dcf(const BwdArgs& a, Launcher& L) {
  using C = BwdCfg<T, D, R, TWO>;
  const bool joint = a.far_norm == FMM_FAR_NORM_JOINT;
  static std::atomic<unsigned long long> set_rows{0}, set_rows_j{0}, set_keys{0};
  if (L.note(joint ? lds_limit_once((const void*)k_bwd_rows<T, D, CAUSAL, R, TWO, true>,
                                    C::LDS, set_rows_j)
                   : lds_limit_once((const void*)k_bwd_rows<T, D, CAUSAL, R, TWO, false>,
                                    C::LDS, set_rows)) != hipSuccess ||
      L.note(lds_limit_once((const void*)k_bwd_keys<T, D, CAUSAL, R, TWO>, C::LDS,
                            set_keys)) != hipSuccess)
    return L.err;
  const float scale2 = 1.4426950408889634f / sqrtf((float)D);
  const int BH = a.B * a.H;
  const size_t REC = (size_t)R * D * (D + 1);
  hipStream_t s = (hipStream_t)a.stream;
  const dim3 grid(BH * a.nwalk);
  auto rows = [&](auto kern) {
    L(FMM_KERNEL_BWD_ROWS, kern, grid, dim3(NT), (size_t)C::LDS, s, (const T*)a.q,
      (const T*)a.k, (const T*)a.v, (const T*)a.dout, (T*)a.dq, CAUSAL ? a.part : a.fin,
      a.rowstat, a.rowfar, a.dwpart, a.w_near, a.w_far, a.H, a.N, a.band_k, a.Lwalk, a.nwalk,
      scale2);
  };
  if (joint) rows(k_bwd_rows<T, D, CAUSAL, R, TWO, true>);
  else rows(k_bwd_rows<T, D, CAUSAL, R, TWO, false>);
  L(FMM_KERNEL_BWD_SEG_GRAD, k_seg_grad<T, D, R>, dim3(BH * a.nseg), dim3(SNTB), 0, s,
    (const T*)a.q, (const T*)a.dout, (const float*)a.rowfar, a.w_far, a.dpart, a.H, a.N, a.L,
    a.nseg);
  if constexpr (CAUSAL) {
    (void)launch_state_suffix(L, a.dpart, a.nseg, (int)REC, BH, s);
  } else {
    (void)launch_state_sum(L, a.dpart, a.dfin, a.nseg, (int)REC, BH, s);
  }
  L(FMM_KERNEL_BWD_KEYS, k_bwd_keys<T, D, CAUSAL, R, TWO>, dim3(BH * a.nwalk + a.H), dim3(NT),
    (size_t)C::LDS, s, (const T*)a.q, (const T*)a.k, (const T*)a.v, (const T*)a.dout, (T*)a.dk,
    (T*)a.dv, CAUSAL ? a.dpart : a.dfin, (const float*)a.rowstat, (const float*)a.rowfar, a.w_near,
    a.w_far, a.H, a.N, a.band_k, a.Lwalk, a.nwalk, scale2, (const float*)a.dwpart, a.dw_near,
    a.dw_far, a.B);
  return L.err;
}

template <typename T, int D, int R>
hipError_t launch_bwd_r(const BwdArgs& a, Launcher& L) {
  // at d <= 64 the state leaves room for two workgroups per CU (two waves per
  // SIMD) where a staging round then still holds a tile; not for the causal
  // passes of three maps at d = 64, which spill within 256 registers (194 in the
  // bf16 key pass; forward and backward, 8 slices of 4001 rows: 273 us, 206 with
  // one workgroup; d = 32: 161 against 176)
  constexpr bool two = D <= 64 && BwdCfg<T, D, R, true>::FITS;
  return a.causal ? launch_bwd_dcf<T, D, true, R, two && !(D == 64 && R == 3)>(a, L)
                  : launch_bwd_dcf<T, D, false, R, two>(a, L);
}

template <typename T, int D>
hipError_t launch_bwd_d(const BwdArgs& a, Launcher& L) {
  switch (a.rank) {
    case 1: return launch_bwd_r<T, D, 1>(a, L);
    case 2: return launch_bwd_r<T, D, 2>(a, L);
    default: return launch_bwd_r<T, D, 3>(a, L);
  }
}

}  // namespace

// Three translation units from this file: bf16 and the dispatch; fp32
// (FMM_BWD_F32); fp32 at d = 128 (FMM_BWD_F32_D128), which holds twice the
// operand registers of bf16: its passes run at one workgroup per CU and need
// the accumulation registers beside the 256 vector registers, so that unit is
// compiled without forcing MFMA results into vector registers (with that
// option the compiler fails on the causal key pass).
#if defined(FMM_BWD_F32_D128)
hipError_t launch_backward_f32_d128(const BwdArgs& a, Launcher& L) {
  return launch_bwd_d<float, 128>(a, L);
}
#elif defined(FMM_BWD_F32)
hipError_t launch_backward_f32(const BwdArgs& a, Launcher& L) {
  switch (a.d) {
    case 16: return launch_bwd_d<float, 16>(a, L);
    case 32: return launch_bwd_d<float, 32>(a, L);
    case 64: return launch_bwd_d<float, 64>(a, L);
    case 128: return launch_backward_f32_d128(a, L);
    default: return L.note(hipErrorInvalidValue);
  }
}
#else
hipError_t launch_backward_tail(const BwdArgs& a, Launcher& L) {
  if (a.dtype != FMM_DTYPE_BF16) return launch_backward_f32(a, L);
  switch (a.d) {
    case 16: return launch_bwd_d<bf16_t, 16>(a, L);
    case 32: return launch_bwd_d<bf16_t, 32>(a, L);
    case 64: return launch_bwd_d<bf16_t, 64>(a, L);
    case 128: return launch_bwd_d<bf16_t, 128>(a, L);
    default: return L.note(hipErrorInvalidValue);
  }
}
#endif

}  // namespace fmm
