// fp32 matrix product with arbitrary element strides and fused bias / GELU / GELU' epilogues, for the fp32 MLP
// (two 256x256 Linear layers, batch 32 / 8, and layers up to about a thousand wide).
//
// At those sizes a product is a few MFLOP: what it takes is a launch, one or two trips to memory and the reduction,
// not arithmetic.  A wavefront therefore owns a 16x16 output tile on v_mfma_f32_16x16x4_f32 (full fp32 products and
// sums) and reads its operands straight from memory into the MFMA's operand registers, eight 16-byte loads in flight
// per lane: four matrix instructions per pair of loads.  An instruction contracts four k, one per 16-lane group; a
// lane loads four consecutive k of its row and hands them to four instructions, so the k an instruction sees are
// {j, 4 + j, 8 + j, 12 + j} of a group of 16 - the same for both operands.
// A block is one output tile of 16 T x 16 T: its four wavefronts take every fourth group of 16 k and the four partial
// tiles are added in a fixed order through LDS (T = 1, 32 x 256 x 256: 32 blocks, a K of 256 is one batch of loads).
// T = 2 halves the operand bytes per product, which is what a larger problem waits for; it is taken as soon as its
// tiles fill the chip.  (32 x 256 x 256 inside a step: 19 us with K staged through LDS 32 at a time, now 5, of which the
// launch and the monitor's prologue and epilogue are 4.)
#include "common.h"
#include "launch.h"

namespace sif {

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Four consecutive k (from k0 on) of row `r` of an operand with element strides sr, sk; rows and k outside read as 0.
// VEC: sk = 1, the address of every fourth k is a multiple of 16 bytes and K is a multiple of 4.
template <bool VEC>
__device__ __forceinline__ floatx4 f32_load4(const float* __restrict__ base, long long sr, long long sk, uint32_t r, uint32_t rows, uint32_t k0, uint32_t k) {
  floatx4 v;
  const bool ok = r < rows;
  const float* p = base + (long long)(ok ? r : 0) * sr;
  if (VEC) {
    const bool in = ok && k0 < k;
    v = *reinterpret_cast<const floatx4*>(p + (in ? k0 : 0));
    if (!in) v = floatx4{0.f, 0.f, 0.f, 0.f};
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool in = ok && k0 + j < k;
      v[j] = p[(long long)(in ? k0 + j : 0) * sk];
      if (!in) v[j] = 0.f;
    }
  }
  return v;
}

template <int T, bool VA, bool VB>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ a, long long a_sm, long long a_sk,
                                                       const float* __restrict__ b, long long b_sk, long long b_sn,
                                                       float* __restrict__ c, long long ldc, uint32_t m, uint32_t n, uint32_t k,
                                                       uint32_t epi, const float* __restrict__ bias, float* __restrict__ aux, KCtl ctl) {
  __shared__ float part[4 * 256 * T * T];
  if (!kernel_begin(ctl)) { kernel_end(ctl, false); return; }
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
  const uint32_t m0 = blockIdx.y * (16 * T), n0 = blockIdx.x * (16 * T);
  constexpr int U = 4 / T;                              // groups of 16 k whose loads (eight per lane) are in flight together
  floatx4 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  for (uint32_t g0 = wave * 16; g0 < k; g0 += 64 * U) {
    floatx4 va[U][T], vb[U][T];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const uint32_t k0 = g0 + u * 64 + 4 * q;
        va[u][t] = f32_load4<VA>(a, a_sm, a_sk, m0 + 16 * t + r, m, k0, k);
        vb[u][t] = f32_load4<VB>(b, b_sn, b_sk, n0 + 16 * t + r, n, k0, k);
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
          for (int j = 0; j < T; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[u][i][e], vb[u][j][e], acc[i][j], 0, 0, 0);
  }
  // accumulator element e of sub-tile (i, j) is row 16 i + 4 q + e, column 16 j + r
  constexpr uint32_t W = 16 * T, TILE = W * W;
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) part[wave * TILE + (16 * i + 4 * q + e) * W + 16 * j + r] = acc[i][j][e];
  __syncthreads();
#pragma unroll
  for (uint32_t o = threadIdx.x; o < TILE; o += 256) {
    const uint32_t row = m0 + o / W, col = n0 + o % W;
    if (row < m && col < n) {
      const long long idx = (long long)row * ldc + col;
      float x = ((part[o] + part[TILE + o]) + part[2 * TILE + o]) + part[3 * TILE + o];
      if (bias != nullptr) x += bias[col];
      if (epi & SIF_EPI_GELU) { if (aux != nullptr) aux[idx] = x; x = gelu_f(x); }
      if (epi & SIF_EPI_GELU_GRAD) x *= gelu_grad_f(aux[idx]);
      c[idx] = x;
    }
  }
  kernel_end(ctl, true);
}

sif_status launch_gemm_f32(const float* a, int64_t a_sm, int64_t a_sk, const float* b, int64_t b_sk, int64_t b_sn,
                           float* c, int64_t ldc, uint32_t m, uint32_t n, uint32_t k, uint32_t epi, const float* bias,
                           float* aux, hipStream_t s, const KCtl& ctl) {
  if (!a || !b || !c) return fail(SIF_E_INVAL, "gemm_f32: null operand");
  if (m == 0 || n == 0 || k == 0) return fail(SIF_E_INVAL, "gemm_f32: empty extent");
  if (ldc < (int64_t)n) return fail(SIF_E_INVAL, "gemm_f32: ldc too small");
  if ((epi & SIF_EPI_GELU_GRAD) && !aux) return fail(SIF_E_INVAL, "gemm_f32: GELU_GRAD needs aux");
  if (epi & ~(uint32_t)(SIF_EPI_BIAS | SIF_EPI_GELU | SIF_EPI_GELU_GRAD)) return fail(SIF_E_INVAL, "gemm_f32: unsupported epilogue");
  // 16-byte loads along K need K contiguous, aligned rows and whole groups of four
  auto vec = [k](const float* p, int64_t sr, int64_t sk) { return sk == 1 && (sr & 3) == 0 && (k & 3) == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  const bool va = vec(a, a_sm, a_sk), vb = vec(b, b_sn, b_sk);
  // The 32x32 tile from one block per CU on (256 x 1024 x 1024: 16.8 -> 11.3 us, 512 x 1024 x 1024: 32.4 -> 18.8 us, where
  // the 32x32 tile of 2x2 outputs per thread that staged K through LDS took 65 and 70); with an operand whose K is strided
  // - four loads in place of one - only from two on (256 x 1024 x 1024: 16.3 against 18.4 us)
  const bool wide = (uint64_t)((m + 31) / 32) * ((n + 31) / 32) >= (va && vb ? 256u : 512u) || (m + 15) / 16 > 65535;
  const uint32_t edge = wide ? 32 : 16;
  const dim3 grid((n + edge - 1) / edge, (m + edge - 1) / edge);
  if (grid.y > 65535) return fail(SIF_E_INVAL, "gemm_f32: grid too large");
  const float* bs = (epi & (SIF_EPI_BIAS | SIF_EPI_GELU)) ? bias : nullptr;
#define F32_LAUNCH(T, VA, VB) hipLaunchKernelGGL((gemm_f32_kernel<T, VA, VB>), grid, dim3(256), 0, s, a, (long long)a_sm, (long long)a_sk, b, (long long)b_sk, \
                                                 (long long)b_sn, c, (long long)ldc, m, n, k, epi, bs, aux, ctl)
#define F32_PICK(T) do { if (va && vb) F32_LAUNCH(T, true, true); else if (va) F32_LAUNCH(T, true, false); else if (vb) F32_LAUNCH(T, false, true); else F32_LAUNCH(T, false, false); } while (0)
  if (wide) F32_PICK(2); else F32_PICK(1);
#undef F32_PICK
#undef F32_LAUNCH
  return check_launch("gemm_f32");
}

}  // namespace sif
