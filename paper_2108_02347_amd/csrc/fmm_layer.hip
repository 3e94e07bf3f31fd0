// The attention layer around the operator: the Step-1 projections of Sec. 1.1
// ([q | k | v] = x W_qkv per token), the FMMformer operator per head, and the
// output projection (heads concatenated per token, times W_out).
//
//   x [B, N, E] --GEMM--> qkv [B*N, 3E] --k_split_heads--> q, k, v [B, H, N, d]
//     --operator--> o [B, H, N, d] --k_merge_heads--> m [B*N, E] --GEMM--> y [B, N, E]
//
// E a multiple of 32 up to 128 (the long-range models' 64-wide and the language
// model's 128-wide embedding among them): each projection and, in the backward,
// each weight gradient is a kernel of this file that reads and writes the
// layouts of the steps beside it (k_proj, k_wgrad), matrix-core products with
// fp32 accumulation.  Otherwise the projections go to rocBLAS (gemm_ex, fp32
// accumulation, the storage type in and out) with the head split and merge as
// coalesced 16-byte copies.  The operator is this library's either way.
#include <hip/hip_runtime.h>
#include <rocblas/rocblas.h>

#include <atomic>
#include <type_traits>

#include "fmm_apply.h"
#include "fmm_device.h"
#include "fmm_launch.h"

namespace fmm {
namespace {

// One 16-byte chunk per thread.  qkv row t = b*N + n holds [q | k | v], each
// part E = H*d wide with the heads in order; chunk c of the row covers
// columns 8c .. 8c+7 (bf16) or 4c .. 4c+3 (fp32), which never straddle a head
// since d is a multiple of 16.
// (parts = 1: rows of one E-wide part, into q only)
template <typename T>
__global__ __launch_bounds__(256) void k_split_heads(const T* __restrict__ qkv,
                                                     T* __restrict__ q, T* __restrict__ k,
                                                     T* __restrict__ v, long long nchunk, int N,
                                                     int H, int d, int parts) {
  constexpr int EPC = 16 / (int)sizeof(T);
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= nchunk) return;
  const int E = H * d, cpr = parts * E / EPC;
  const long long t = i / cpr;
  const int col = (int)(i - t * cpr) * EPC;
  const int part = col / E, h = (col % E) / d, c = col % d;
  const long long b = t / N, n = t - b * N;
  T* dst = part == 0 ? q : (part == 1 ? k : v);
  const uint4 val = *reinterpret_cast<const uint4*>(qkv + t * parts * E + col);
  *reinterpret_cast<uint4*>(dst + (((b * H + h) * N + n) * d + c)) = val;
}

// o [B, H, N, d] -> m [B*N, E] (the heads of a token side by side), in rows
// of row_len elements from column col0 (E and 0 for the layer's forward).
template <typename T>
__global__ __launch_bounds__(256) void k_merge_heads(const T* __restrict__ o, T* __restrict__ m,
                                                     long long nchunk, int N, int H, int d,
                                                     int row_len, int col0) {
  constexpr int EPC = 16 / (int)sizeof(T);
  const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
  if (i >= nchunk) return;
  const int E = H * d, cpr = E / EPC;
  const long long t = i / cpr;
  const int col = (int)(i - t * cpr) * EPC;
  const int h = col / d, c = col % d;
  const long long b = t / N, n = t - b * N;
  const uint4 val = *reinterpret_cast<const uint4*>(o + (((b * H + h) * N + n) * d + c));
  *reinterpret_cast<uint4*>(m + t * row_len + col0 + col) = val;
}

template <typename T>
void launch_split(Launcher& L, const void* qkv, void* q, void* k, void* v, int B, int N, int H,
                  int d, hipStream_t s, int parts = 3) {
  constexpr int EPC = 16 / (int)sizeof(T);
  const long long nchunk = (long long)B * N * parts * H * d / EPC;
  const long long nb = (nchunk + 255) / 256;
  L(FMM_KERNEL_LAYER_COPY, k_split_heads<T>, dim3((unsigned)std::min<long long>(nb, 0xFFFFFFFFll)),
    dim3(256), 0, s, (const T*)qkv, (T*)q, (T*)k, (T*)v, nchunk, N, H, d, parts);
}

template <typename T>
void launch_merge(Launcher& L, const void* o, void* m, int B, int N, int H, int d,
                  hipStream_t s, int row_len = 0, int col0 = 0) {
  constexpr int EPC = 16 / (int)sizeof(T);
  const long long nchunk = (long long)B * N * H * d / EPC;
  const long long nb = (nchunk + 255) / 256;
  L(FMM_KERNEL_LAYER_COPY, k_merge_heads<T>, dim3((unsigned)std::min<long long>(nb, 0xFFFFFFFFll)),
    dim3(256), 0, s, (const T*)o, (T*)m, nchunk, N, H, d, row_len > 0 ? row_len : H * d, col0);
}

// ------------------------------------------------------------------ k_proj
// The layer's projections for E = 32, 64, 96 or 128, both storage types, each
// in the layouts that the steps beside it use (heads: [B, H, N, d] tensors,
// rows: [T, E]), so that no copy splits or merges heads:
//   kProjQkv   x rows -> q, k, v heads      out[t][c] = sum_e x[t][e] W[e][c], c < 3E
//   kProjOut   heads -> y rows              out[t][c] = sum_e m[t][e] W[e][c]
//   kProjDm    dy rows -> heads             out[t][c] = sum_e dy[t][e] W[c][e]
//   kProjDx    dq, dk, dv heads -> dx rows  out[t][c] = sum_{e < 3E} in[t][e] W[c][e]
// (W row-major with ld columns.)
//
// A workgroup (4 waves) takes 64 tokens (a wave 16) and CC output columns,
// whose part of W is staged in LDS; columns in chunks keep W's part small (fp32
// at E = 128: 35 KB instead of 198) and fill the chip at few tokens.  The
// product is formed transposed, D[c][t], so that a lane ends with four
// consecutive columns of one token, stored together.  4096 tokens, E = 128,
// fp32: 13.9 + 6.2 us, where the two rocBLAS products and the head split and
// merge took 9.4 + 9.4 + 6.4 + 4.3.  fp32 sums in two parts: with one chain of
// up to 384 products dx was up to 1.08 times as far from float64 as rocBLAS's.
enum { kProjQkv, kProjOut, kProjDm, kProjDx };

// Token t as (batch, position), and the offset of its column c of E in a
// tensor of heads (d = 1 << ld).  32-bit and shifts: the compiler's 64-bit
// quotients cost more than the products here.
struct Tok {
  unsigned b, n;
  __device__ __forceinline__ Tok(long long t, int N) {
    b = (unsigned)t / (unsigned)N;
    n = (unsigned)t - b * (unsigned)N;
  }
  __device__ __forceinline__ size_t head(int c, int N, int H, int ld) const {
    const unsigned hh = (unsigned)c >> ld;
    return ((((size_t)b * H + hh) * N + n) << ld) + (c & ((1 << ld) - 1));
  }
};

template <typename T, int E, int MODE, bool WIDE>
struct ProjCfg {
  static constexpr int K = MODE == kProjDx ? 3 * E : E;       // contraction
  static constexpr int OUT = MODE == kProjQkv ? 3 * E : E;    // output columns
  // of a workgroup: all (WIDE) or a part
  static constexpr int CC = WIDE ? OUT : E == 96 ? 96 : (E < 64 ? E : 64);
  static constexpr bool WT = MODE == kProjDm || MODE == kProjDx;  // W used transposed
  static constexpr int ROWS = WT ? CC : K, COLS = WT ? K : CC;    // of its part of W
  static constexpr int ST = COLS + Lay<T>::PAD;
  static constexpr int LDS = ROWS * ST * (int)sizeof(T);
};

template <typename T, int E, int MODE, bool WIDE>
__global__ __launch_bounds__(256) void k_proj(const T* __restrict__ in0,
                                              const T* __restrict__ in1,
                                              const T* __restrict__ in2,
                                              const T* __restrict__ w, T* __restrict__ o0,
                                              T* __restrict__ o1, T* __restrict__ o2, int Tn,
                                              int N, int H, int ld) {
  using C = ProjCfg<T, E, MODE, WIDE>;
  using Q = typename QuadOf<T>::type;
  constexpr int KB = C::K / 16, EPC = Lay<T>::EPC, CPR = C::COLS / EPC;
  constexpr int LDW = MODE == kProjQkv || MODE == kProjDx ? 3 * E : E;
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
  T* wl = reinterpret_cast<T*>(dyn_smem);
  constexpr int NCH = C::OUT / C::CC;
  const int cc0 = (int)(blockIdx.x % NCH) * C::CC;
  const long long tile = blockIdx.x / NCH;
  for (int i = threadIdx.x; i < C::ROWS * CPR; i += 256) {
    const int row = i / CPR, c = (i % CPR) * EPC;
    *reinterpret_cast<uint4*>(wl + row * C::ST + c) = *reinterpret_cast<const uint4*>(
        w + (size_t)(C::WT ? cc0 + row : row) * LDW + (C::WT ? c : cc0 + c));
  }
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const long long tok = tile * 64 + 16 * wv + r;  // this lane's token
  const bool ok = tok < Tn;
  const Tok tk(ok ? tok : 0, N);
  Q x[KB];
#pragma unroll
  for (int kb = 0; kb < KB; ++kb) {
    const int kk = 16 * kb + 4 * g;
    const T* p;
    if constexpr (MODE == kProjQkv || MODE == kProjDm) {
      p = in0 + (ok ? tok : 0) * E + kk;
    } else {
      const int part = kk / E;  // (a 16-wide block lies in one part: E % 16 == 0)
      p = (part == 0 ? in0 : part == 1 ? in1 : in2) + tk.head(kk - part * E, N, H, ld);
    }
    // (tokens past the end read a valid row and are not stored)
    x[kb] = *reinterpret_cast<const Q*>(p);
  }
  __syncthreads();
#pragma unroll 4
  for (int cb = 0; cb < C::CC / 16; ++cb) {
    Q a[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
      a[kb] = C::WT ? ld_quad(wl, 16 * cb + r, 16 * kb + 4 * g, C::ST)
                    : ld_tquad(wl, 16 * kb, 16 * cb, C::ST);
    const f32x4 acc = contract_split<KB, 2>(a, x);
    if (!ok) continue;
    const float f[4] = {acc[0], acc[1], acc[2], acc[3]};
    const int c = cc0 + 16 * cb + 4 * g;
    T* dst;
    if constexpr (MODE == kProjQkv) {
      const int part = c / E;
      dst = (part == 0 ? o0 : part == 1 ? o1 : o2) + tk.head(c - part * E, N, H, ld);
    } else if constexpr (MODE == kProjDm) {
      dst = o0 + tk.head(c, N, H, ld);
    } else {
      dst = o0 + tok * E + c;
    }
    *reinterpret_cast<Q*>(dst) = f32_to_quad<T>(f);
  }
}

template <typename T, int E, int MODE, bool WIDE>
void launch_proj_w(Launcher& L, const void* i0, const void* i1, const void* i2, const void* w,
                   void* o0, void* o1, void* o2, int B, int N, int H, int d, hipStream_t s) {
  using C = ProjCfg<T, E, MODE, WIDE>;
  static std::atomic<unsigned long long> lds_set{0};
  if (L.note(lds_limit_once((const void*)k_proj<T, E, MODE, WIDE>, C::LDS, lds_set)) != hipSuccess)
    return;
  const long long nb = ((long long)B * N + 63) / 64 * (C::OUT / C::CC);
  L(FMM_KERNEL_LAYER_COPY, k_proj<T, E, MODE, WIDE>,
    dim3((unsigned)std::min<long long>(nb, 0xFFFFFFFFll)), dim3(256), (size_t)C::LDS, s,
    (const T*)i0, (const T*)i1, (const T*)i2, (const T*)w, (T*)o0, (T*)o1, (T*)o2,
    (int)((long long)B * N), N, H, __builtin_ctz(d));
}

// All columns in one workgroup where the tokens alone give two per CU and W
// stays small: W is staged and the tokens read once (32768 tokens, E = 64, bf16,
// kProjQkv 10.1 us, 11.5 in parts); else columns in parts.
template <typename T, int E, int MODE>
void launch_proj_k(Launcher& L, const void* i0, const void* i1, const void* i2, const void* w,
                   void* o0, void* o1, void* o2, int B, int N, int H, int d, hipStream_t s) {
  if constexpr (ProjCfg<T, E, MODE, true>::LDS <= 52 * 1024) {
    if ((long long)B * N >= 512 * 64)
      return launch_proj_w<T, E, MODE, true>(L, i0, i1, i2, w, o0, o1, o2, B, N, H, d, s);
  }
  launch_proj_w<T, E, MODE, false>(L, i0, i1, i2, w, o0, o1, o2, B, N, H, d, s);
}

// ------------------------------------------------------------------ k_wgrad
// Weight gradients for the same widths: per chunk of tokens (blockIdx.x) and
// part (blockIdx.y: B one of up to three tensors), C[e][n] = sum_t A[t][e]
// B[t][n] (E x E, fp32) into part[chunk][e][ld]: A rows or heads, B rows or
// heads.  64 tokens of both staged in LDS at a time (the next ones' loads in
// flight), each wave E / 16 tiles of 16 columns n; k_sum_chunks then sums the
// chunks in order.  32768 tokens, E = 64, bf16: 8.4 us for W_qkv, 5.4 for W_out
// (rocBLAS strided batches over merged copies: 15.8 and 8.2, the copies 16).
template <typename T, int E, bool AHEADS, bool BHEADS>
__global__ __launch_bounds__(256) void k_wgrad(const T* __restrict__ A, const T* __restrict__ b0,
                                               const T* __restrict__ b1,
                                               const T* __restrict__ b2,
                                               float* __restrict__ part, int Tn, int chunk, int N,
                                               int H, int ld) {
  using Q = typename QuadOf<T>::type;
  constexpr int EB = E / 16, EPC = Lay<T>::EPC, CPR = E / EPC, ST = E + Lay<T>::PAD;
  constexpr int IT = 64 * CPR / 256;
  constexpr int NBW = (EB + 3) / 4;  // column blocks of a wave
  extern __shared__ __attribute__((aligned(16))) unsigned char dyn_smem[];
  T* sa = reinterpret_cast<T*>(dyn_smem);
  T* sb = sa + 64 * ST;
  const T* Bm = blockIdx.y == 0 ? b0 : blockIdx.y == 1 ? b1 : b2;
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const long long t0 = (long long)blockIdx.x * chunk, t1 = min((long long)Tn, t0 + chunk);
  f32x4 acc[EB][NBW];
#pragma unroll
  for (int e = 0; e < EB; ++e)
#pragma unroll
    for (int x = 0; x < NBW; ++x) acc[e][x] = f32x4{0.f, 0.f, 0.f, 0.f};
  // two 64-token tiles in flight (the loads are what a chunk waits for)
  uint4 ra[2][IT], rb[2][IT];
  auto load = [&](int s, long long ts) {
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int i = threadIdx.x + it * 256, c = (i % CPR) * EPC;
      const long long t = ts + i / CPR;
      const bool ok = t < t1;
      const long long tc = ok ? t : 0;
      const Tok tk(tc, N);
      const uint4 va = *reinterpret_cast<const uint4*>(
          A + (AHEADS ? tk.head(c, N, H, ld) : (size_t)tc * E + c));
      const uint4 vb = *reinterpret_cast<const uint4*>(
          Bm + (BHEADS ? tk.head(c, N, H, ld) : (size_t)tc * E + c));
      // (by component: a choice between two structs would put them in memory)
      ra[s][it] = make_uint4(ok ? va.x : 0u, ok ? va.y : 0u, ok ? va.z : 0u, ok ? va.w : 0u);
      rb[s][it] = make_uint4(ok ? vb.x : 0u, ok ? vb.y : 0u, ok ? vb.z : 0u, ok ? vb.w : 0u);
    }
  };
  load(0, t0);
  load(1, t0 + 64);
  for (long long tp = t0; tp < t1; tp += 128)
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const long long ts = tp + 64 * s;
    if (ts >= t1) break;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int i = threadIdx.x + it * 256, row = i / CPR, c = (i % CPR) * EPC;
      *reinterpret_cast<uint4*>(sa + row * ST + c) = ra[s][it];
      *reinterpret_cast<uint4*>(sb + row * ST + c) = rb[s][it];
    }
    __syncthreads();
    load(s, ts + 128);
#pragma unroll
    for (int x = 0; x < NBW; ++x) {
      const int nb = wv + 4 * x;
      if (nb < EB) {
        Q bq[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) bq[m] = ld_tquad(sb, 16 * m, 16 * nb, ST);
#pragma unroll
        for (int e = 0; e < EB; ++e) {
          Q aq[4];
#pragma unroll
          for (int m = 0; m < 4; ++m) aq[m] = ld_tquad(sa, 16 * m, 16 * e, ST);
          if constexpr (sizeof(T) == 4)
            acc[e][x] += contract<4>(aq, bq, f32x4{0.f, 0.f, 0.f, 0.f});
          else acc[e][x] = contract<4>(aq, bq, acc[e][x]);
        }
      }
    }
  }
  mfma_drain();  // (results read after the loop's branches)
  const int row = E * (int)gridDim.y;
  float* o = part + (size_t)blockIdx.x * E * row + blockIdx.y * E;
#pragma unroll
  for (int x = 0; x < NBW; ++x) {
    const int nb = wv + 4 * x;
    if (nb < EB)
#pragma unroll
      for (int e = 0; e < EB; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          o[(size_t)(16 * e + 4 * g + i) * row + 16 * nb + r] = acc[e][x][i];
  }
}

// f(T of the dtype, E as a compile-time constant)
template <typename F>
hipError_t by_width(Launcher& L, int dtype, int E, F f) {
  auto width = [&](auto t) {
    switch (E) {
      case 32: f(t, std::integral_constant<int, 32>()); break;
      case 64: f(t, std::integral_constant<int, 64>()); break;
      case 96: f(t, std::integral_constant<int, 96>()); break;
      case 128: f(t, std::integral_constant<int, 128>()); break;
      default: return L.note(hipErrorInvalidValue);
    }
    return L.err;
  };
  return dtype == FMM_DTYPE_BF16 ? width(bf16_t()) : width(float());
}

// Row-major C [M, Nc] = A [M, K] B [K, Nc] as the column-major product
// C^T = B^T A^T.
// With ta (tb): A (B) is stored transposed, i.e. A is [K, M] (B is [Nc, K])
// row-major and the product uses its transpose.
hipError_t gemm_rm(rocblas_handle hdl, int dtype, const void* A, const void* Bm, void* C, int M,
                   int K, int Nc, bool ta = false, bool tb = false) {
  const rocblas_datatype t =
      dtype == FMM_DTYPE_BF16 ? rocblas_datatype_bf16_r : rocblas_datatype_f32_r;
  const float one = 1.f, zero = 0.f;
  const rocblas_status st = rocblas_gemm_ex(
      hdl, tb ? rocblas_operation_transpose : rocblas_operation_none,
      ta ? rocblas_operation_transpose : rocblas_operation_none, Nc, M, K, &one, Bm, t,
      tb ? K : Nc, A, t, ta ? M : K, &zero, C, t, Nc, C, t, Nc, rocblas_datatype_f32_r,
      rocblas_gemm_algo_standard, 0, 0);
  return st == rocblas_status_success ? hipSuccess : hipErrorLaunchFailure;
}

}  // namespace

hipError_t launch_layer_copy(Launcher& L, bool split, int dtype, const void* src, void* d0,
                             void* d1, void* d2, int B, int N, int H, int d, hipStream_t s) {
  if (dtype == FMM_DTYPE_BF16) {
    if (split) launch_split<bf16_t>(L, src, d0, d1, d2, B, N, H, d, s);
    else launch_merge<bf16_t>(L, src, d0, B, N, H, d, s);
  } else {
    if (split) launch_split<float>(L, src, d0, d1, d2, B, N, H, d, s);
    else launch_merge<float>(L, src, d0, B, N, H, d, s);
  }
  return L.err;
}

// Any number of tokens (whole causal layer calls, rocBLAS with head copies ->
// these, us: E = 32, 64 tokens fp32 30 -> 20, bf16 20 -> 20; 262144 tokens fp32
// 318 -> 164, bf16 82 -> 77; E = 128 34 -> 22, 23 -> 21; 1194 -> 808, 403 -> 353).
bool layer_proj_applies(int E) { return E == 32 || E == 64 || E == 96 || E == 128; }

hipError_t launch_layer_proj(Launcher& L, LayerProj mode, int dtype, const void* i0,
                             const void* i1, const void* i2, const void* w, void* o0, void* o1,
                             void* o2, int B, int N, int H, int d, hipStream_t s) {
  return by_width(L, dtype, H * d, [&](auto t, auto e) {
    using T = decltype(t);
    constexpr int E = e.value;
    switch (mode) {
      case LayerProj::kQkv:
        launch_proj_k<T, E, kProjQkv>(L, i0, i1, i2, w, o0, o1, o2, B, N, H, d, s);
        break;
      case LayerProj::kOut:
        launch_proj_k<T, E, kProjOut>(L, i0, i1, i2, w, o0, o1, o2, B, N, H, d, s);
        break;
      case LayerProj::kDm:
        launch_proj_k<T, E, kProjDm>(L, i0, i1, i2, w, o0, o1, o2, B, N, H, d, s);
        break;
      case LayerProj::kDx:
        launch_proj_k<T, E, kProjDx>(L, i0, i1, i2, w, o0, o1, o2, B, N, H, d, s);
        break;
    }
  });
}

hipError_t layer_gemm(void* handle, void* stream, int dtype, const void* A, const void* Bm,
                      void* C, int M, int K, int Nc, bool ta, bool tb) {
  rocblas_handle hdl = (rocblas_handle)handle;
  if (rocblas_set_stream(hdl, (hipStream_t)stream) != rocblas_status_success)
    return hipErrorLaunchFailure;
  return gemm_rm(hdl, dtype, A, Bm, C, M, K, Nc, ta, tb);
}

// Weight gradients C [E, Nc] = A^T B with A [M, E] and B [M, Nc] row-major and
// M (the tokens) far larger than E and Nc: one product per chunk of KC tokens
// (a strided batch, fp32 results), then the chunks summed in order into C (the
// storage type).  A single product would leave most of the GPU idle (a few
// output tiles, each walking all M tokens).
namespace {
// 64 elements x 4 ranges of chunks per workgroup, each range in chunk order
// with four loads in flight, the ranges in order (one thread walking all
// chunks of an element: 48 workgroups and 10 us for 12288 elements of 32
// chunks)
template <typename T>
__global__ __launch_bounds__(256) void k_sum_chunks(const float* __restrict__ part,
                                                    T* __restrict__ c, int n, int nchunk) {
  __shared__ float tot[4][64];
  const int el = threadIdx.x & 63, qr = threadIdx.x >> 6;
  const int i = blockIdx.x * 64 + el;
  const int per = (nchunk + 3) / 4, j0 = min(nchunk, qr * per), j1 = min(nchunk, j0 + per);
  float s = 0.f;
  if (i < n) {
    const float* p = part + i;
    int j = j0;
    for (; j + 4 <= j1; j += 4) {
      const float a0 = p[(size_t)j * n], a1 = p[(size_t)(j + 1) * n];
      const float a2 = p[(size_t)(j + 2) * n], a3 = p[(size_t)(j + 3) * n];
      s += (a0 + a1) + (a2 + a3);
    }
    for (; j < j1; ++j) s += p[(size_t)j * n];
  }
  tot[qr][el] = s;
  __syncthreads();
  if (qr != 0 || i >= n) return;
  s = (tot[0][el] + tot[1][el]) + (tot[2][el] + tot[3][el]);
  if constexpr (sizeof(T) == 2) c[i] = (T)f32_to_bf16_bits(s);
  else c[i] = s;
}

hipError_t sum_chunks(Launcher& L, int dtype, const float* part, void* c, int n, int nchunk,
                      hipStream_t s) {
  const dim3 grid((n + 63) / 64);
  if (dtype == FMM_DTYPE_BF16)
    L(FMM_KERNEL_LAYER_COPY, k_sum_chunks<bf16_t>, grid, dim3(256), 0, s, part, (bf16_t*)c, n,
      nchunk);
  else
    L(FMM_KERNEL_LAYER_COPY, k_sum_chunks<float>, grid, dim3(256), 0, s, part, (float*)c, n,
      nchunk);
  return L.err;
}

// Tokens per chunk of k_wgrad: 256, fewer (a multiple of its 64-token tiles)
// where that would be under 32 chunks (forward and backward of 200 to 1000 tokens,
// E = 128, fp32: 143 -> 110 us), more where it would be over 256 (lean: at
// least those of the rocBLAS form).
int own_wgrad_chunk(int M, bool lean) {
  auto tiles = [](long long c) { return (c + 63) / 64 * 64; };
  if (lean) return (int)std::max<long long>(kWgradChunk, tiles(((long long)M + 255) / 256));
  return (int)std::max(std::min<long long>(256, tiles(((long long)M + 31) / 32)),
                       tiles(((long long)M + 255) / 256));
}
}  // namespace

size_t layer_wgrad_scratch_bytes(int M, int E, int Nc, bool lean) {
  const int c = layer_proj_applies(E) ? own_wgrad_chunk(M, lean) : kWgradChunk;
  return (size_t)((M + (long long)c - 1) / c) * E * Nc * sizeof(float);
}

hipError_t launch_layer_wgrad(Launcher& L, int dtype, bool qkv, const void* A, const void* b0,
                              const void* b1, const void* b2, void* C, float* scratch, int B,
                              int N, int H, int d, hipStream_t s, bool lean) {
  const int E = H * d, M = (int)((long long)B * N), chunk = own_wgrad_chunk(M, lean);
  const int nchunk = (int)((M + (long long)chunk - 1) / chunk), parts = qkv ? 3 : 1;
  (void)by_width(L, dtype, E, [&](auto t, auto e) {
    using T = decltype(t);
    constexpr int W = e.value;
    constexpr int lds = 2 * 64 * (W + Lay<T>::PAD) * (int)sizeof(T);
    static std::atomic<unsigned long long> set_q{0}, set_o{0};
    const dim3 grid(nchunk, parts);
    if (qkv) {
      if (L.note(lds_limit_once((const void*)k_wgrad<T, W, false, true>, lds, set_q)) ==
          hipSuccess)
        L(FMM_KERNEL_LAYER_COPY, k_wgrad<T, W, false, true>, grid, dim3(256), (size_t)lds, s,
          (const T*)A, (const T*)b0, (const T*)b1, (const T*)b2, scratch, M, chunk, N, H,
          __builtin_ctz(d));
    } else {
      if (L.note(lds_limit_once((const void*)k_wgrad<T, W, true, false>, lds, set_o)) ==
          hipSuccess)
        L(FMM_KERNEL_LAYER_COPY, k_wgrad<T, W, true, false>, grid, dim3(256), (size_t)lds, s,
          (const T*)A, (const T*)b0, (const T*)nullptr, (const T*)nullptr, scratch, M, chunk, N,
          H, __builtin_ctz(d));
    }
  });
  if (L.err != hipSuccess) return L.err;
  return sum_chunks(L, dtype, scratch, C, E * E * parts, nchunk, s);
}

hipError_t layer_wgrad(void* handle, Launcher& L, void* stream, int dtype, const void* A,
                       const void* Bm, void* C, int M, int E, int Nc, float* scratch) {
  const int nchunk = (M + kWgradChunk - 1) / kWgradChunk;
  const int n = E * Nc;
  hipStream_t s = (hipStream_t)stream;
  if (!L.dry) {
    rocblas_handle hdl = (rocblas_handle)handle;
    if (rocblas_set_stream(hdl, s) != rocblas_status_success) return L.note(hipErrorLaunchFailure);
    const rocblas_datatype t =
        dtype == FMM_DTYPE_BF16 ? rocblas_datatype_bf16_r : rocblas_datatype_f32_r;
    const size_t es = dtype == FMM_DTYPE_BF16 ? 2 : 4;
    const float one = 1.f, zero = 0.f;
    // column-major: C^T [Nc, E] = B^T [Nc, K] A [K, E] per chunk of K tokens;
    // the full chunks as one strided batch, a shorter last chunk as one more
    // product
    const int full = M / kWgradChunk, rem = M - full * kWgradChunk;
    auto batch = [&](int k, int count, const void* a0, const void* b0, float* c0) {
      return rocblas_gemm_strided_batched_ex(
          hdl, rocblas_operation_none, rocblas_operation_transpose, Nc, E, k, &one, b0, t, Nc,
          (rocblas_stride)k * Nc, a0, t, E, (rocblas_stride)k * E, &zero, c0,
          rocblas_datatype_f32_r, Nc, (rocblas_stride)n, c0, rocblas_datatype_f32_r, Nc,
          (rocblas_stride)n, count, rocblas_datatype_f32_r, rocblas_gemm_algo_standard, 0, 0);
    };
    if (full > 0 && batch(kWgradChunk, full, A, Bm, scratch) != rocblas_status_success)
      return L.note(hipErrorLaunchFailure);
    if (rem > 0) {
      const size_t off = (size_t)full * kWgradChunk;
      const void* a1 = static_cast<const unsigned char*>(A) + off * E * es;
      const void* b1 = static_cast<const unsigned char*>(Bm) + off * Nc * es;
      if (batch(rem, 1, a1, b1, scratch + (size_t)full * n) != rocblas_status_success)
        return L.note(hipErrorLaunchFailure);
    }
  }
  return sum_chunks(L, dtype, scratch, C, n, nchunk, s);
}

hipError_t launch_layer_split1(Launcher& L, int dtype, const void* src, void* dst, int B, int N,
                               int H, int d, hipStream_t s) {
  if (dtype == FMM_DTYPE_BF16)
    launch_split<bf16_t>(L, src, dst, nullptr, nullptr, B, N, H, d, s, 1);
  else
    launch_split<float>(L, src, dst, nullptr, nullptr, B, N, H, d, s, 1);
  return L.err;
}

hipError_t launch_layer_merge_part(Launcher& L, int dtype, const void* src, void* dst, int part,
                                   int B, int N, int H, int d, hipStream_t s) {
  if (dtype == FMM_DTYPE_BF16)
    launch_merge<bf16_t>(L, src, dst, B, N, H, d, s, 3 * H * d, part * H * d);
  else
    launch_merge<float>(L, src, dst, B, N, H, d, s, 3 * H * d, part * H * d);
  return L.err;
}

void* layer_blas_handle_create() {
  rocblas_handle h = nullptr;
  if (rocblas_create_handle(&h) != rocblas_status_success) return nullptr;
  return (void*)h;
}

}  // namespace fmm
