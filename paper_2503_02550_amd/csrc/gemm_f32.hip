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

// What block `tile` of a product does.
template <int T, bool VA, bool VB>
__device__ __forceinline__ void f32_tile(const F32Product& p, uint32_t tile, float* part) {
  const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, q = lane >> 4;
  const uint32_t m0 = tile / p.tiles_n * (16 * T), n0 = tile % p.tiles_n * (16 * T);
  constexpr int U = 4 / T;                              // groups of 16 k whose loads (eight per lane) are in flight together
  floatx4 acc[T][T];
  float rows[T];
#pragma unroll
  for (int i = 0; i < T; ++i) {
    rows[i] = 0.f;
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  for (uint32_t g0 = wave * 16; g0 < p.k; g0 += 64 * U) {
    floatx4 va[U][T], vb[U][T];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const uint32_t k0 = g0 + u * 64 + 4 * q;
        va[u][t] = f32_load4<VA>(p.a, p.a_sm, p.a_sk, m0 + 16 * t + r, p.m, k0, p.k);
        vb[u][t] = f32_load4<VB>(p.b, p.b_sn, p.b_sk, n0 + 16 * t + r, p.n, k0, p.k);
      }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < T; ++i) {
          rows[i] += va[u][i][e];
#pragma unroll
          for (int j = 0; j < T; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(va[u][i][e], vb[u][j][e], acc[i][j], 0, 0, 0);
        }
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
  float sq = 0.f;
#pragma unroll
  for (uint32_t o = threadIdx.x; o < TILE; o += 256) {
    const uint32_t row = m0 + o / W, col = n0 + o % W;
    if (row < p.m && col < p.n) {
      const long long idx = (long long)row * p.ldc + col;
      float x = ((part[o] + part[TILE + o]) + part[2 * TILE + o]) + part[3 * TILE + o];
      if (p.bias != nullptr) x += p.bias[col];
      if (p.epi & SIF_EPI_GELU) { if (p.aux != nullptr) p.aux[idx] = x; x = gelu_f(x); }
      if (p.epi & SIF_EPI_GELU_GRAD) x *= gelu_grad_f(p.aux[idx]);
      p.c[idx] = x;
      if (p.target != nullptr) { const float e = x - p.target[idx]; p.diff[idx] = e * p.inv_n; sq += e * e; }
      if (p.update != nullptr) p.update[idx] -= p.lr * x;
    }
  }
  if (p.target != nullptr) {                            // the tile's part of the loss
    __syncthreads();
    sq = block_sum(sq, part);
    if (threadIdx.x == 0) p.loss_part[tile] = sq;
  }
  if (p.rowsum != nullptr && n0 == 0) {                 // sums of A's rows over k, from the values the products were fed with
    __syncthreads();
#pragma unroll
    for (int i = 0; i < T; ++i) {
      rows[i] += __shfl_xor(rows[i], 16, 64);
      rows[i] += __shfl_xor(rows[i], 32, 64);
      if (q == 0) part[wave * W + 16 * i + r] = rows[i];
    }
    __syncthreads();
    if (threadIdx.x < W && m0 + threadIdx.x < p.m) {
      const float x = ((part[threadIdx.x] + part[W + threadIdx.x]) + part[2 * W + threadIdx.x]) + part[3 * W + threadIdx.x];
      p.rowsum[m0 + threadIdx.x] = x;
      if (p.rowsum_update != nullptr) p.rowsum_update[m0 + threadIdx.x] -= p.lr * x;
    }
  }
}
template <int T>
__device__ __forceinline__ void f32_product(const F32Product& p, uint32_t tile, float* part) {
  if (p.vec == 3u) f32_tile<T, true, true>(p, tile, part);
  else if (p.vec == 1u) f32_tile<T, true, false>(p, tile, part);
  else if (p.vec == 2u) f32_tile<T, false, true>(p, tile, part);
  else f32_tile<T, false, false>(p, tile, part);
}

// One or two products and what of the step can run beside them: the blocks of the first product, those of the second,
// one that adds up the loss, and those of an SGD update (1024 parameters each).
constexpr uint32_t kSgdPerBlock = 1024;
template <int T>
__global__ __launch_bounds__(256) void gemm_f32_kernel(F32Launch l, KCtl ctl) {
  __shared__ float part[4 * 256 * T * T];
  if (!kernel_begin(ctl)) { kernel_end(ctl, false); return; }
  uint32_t b = blockIdx.x;
  if (b < l.blocks[0]) {
    f32_product<T>(l.p[0], b, part);
  } else if ((b -= l.blocks[0]) < l.blocks[1]) {
    f32_product<T>(l.p[1], b, part);
  } else if ((b -= l.blocks[1]) < l.blocks[2]) {
    float s = 0.f;
    for (uint32_t i = threadIdx.x; i < l.loss_parts; i += 256) s += l.loss_part[i];
    s = block_sum(s, part);
    if (threadIdx.x == 0) l.loss[0] = 0.5f * s * l.loss_inv_n;
  } else {
    b -= l.blocks[2];
#pragma unroll
    for (uint32_t u = 0; u < kSgdPerBlock; u += 256) {
      const uint64_t i = (uint64_t)b * kSgdPerBlock + u + threadIdx.x;
      if (i < l.sgd_n) l.sgd_p[i] = l.sgd_p[i] - l.lr * l.sgd_g[i];
    }
  }
  kernel_end(ctl, true);
}

static uint64_t f32_tiles(const F32Product& p, uint32_t edge) { return (uint64_t)((p.m + edge - 1) / edge) * ((p.n + edge - 1) / edge); }

uint32_t f32_loss_parts(uint32_t m, uint32_t n) { return ((m + 15) / 16) * ((n + 15) / 16); }
static uint32_t f32_sgd_blocks(uint64_t n) { return (uint32_t)((n + kSgdPerBlock - 1) / kSgdPerBlock); }

// Checks the products of `l`, chooses the tile and launches.
sif_status launch_f32(F32Launch l, hipStream_t s, const KCtl& ctl) {
  bool wide = true;
  for (uint32_t i = 0; i < 2; ++i) {
    F32Product& p = l.p[i];
    if (i == 1 && p.c == nullptr) continue;
    if (!p.a || !p.b || !p.c) return fail(SIF_E_INVAL, "gemm_f32: null operand");
    if (p.m == 0 || p.n == 0 || p.k == 0) return fail(SIF_E_INVAL, "gemm_f32: empty extent");
    if (p.ldc < (int64_t)p.n) return fail(SIF_E_INVAL, "gemm_f32: ldc too small");
    if ((p.epi & SIF_EPI_GELU_GRAD) && !p.aux) return fail(SIF_E_INVAL, "gemm_f32: GELU_GRAD needs aux");
    if (p.epi & ~(uint32_t)(SIF_EPI_BIAS | SIF_EPI_GELU | SIF_EPI_GELU_GRAD)) return fail(SIF_E_INVAL, "gemm_f32: unsupported epilogue");
    if (!(p.epi & (SIF_EPI_BIAS | SIF_EPI_GELU))) p.bias = nullptr;
    if (f32_tiles(p, 32) > (1u << 29)) return fail(SIF_E_INVAL, "gemm_f32: grid too large");
    // 16-byte loads along K need K contiguous, aligned rows and whole groups of four
    auto vec = [&](const float* q, int64_t sr, int64_t sk) { return sk == 1 && (sr & 3) == 0 && (p.k & 3) == 0 && (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
    p.vec = (vec(p.a, p.a_sm, p.a_sk) ? 1u : 0u) | (vec(p.b, p.b_sn, p.b_sk) ? 2u : 0u);
    // The 32x32 tile from one block per CU on (256 x 1024 x 1024: 16.8 -> 11.3 us, 512 x 1024 x 1024: 32.4 -> 18.8 us, where
    // the 32x32 tile of 2x2 outputs per thread that staged K through LDS took 65 and 70); with an operand whose K is strided
    // - four loads in place of one - only from two on (256 x 1024 x 1024: 16.3 against 18.4 us)
    wide = wide && f32_tiles(p, 32) >= (p.vec == 3u ? 256u : 512u);
  }
  uint64_t grid = (uint64_t)(l.blocks[2] = l.loss != nullptr ? 1u : 0u) + (l.sgd_p != nullptr ? f32_sgd_blocks(l.sgd_n) : 0u);
  for (uint32_t i = 0; i < 2; ++i) {
    if (l.p[i].c == nullptr) { l.blocks[i] = 0; continue; }
    wide = wide || f32_tiles(l.p[i], 16) > (1u << 30);
  }
  const uint32_t edge = wide ? 32 : 16;
  for (uint32_t i = 0; i < 2; ++i) {
    if (l.p[i].c == nullptr) continue;
    l.p[i].tiles_n = (l.p[i].n + edge - 1) / edge;
    l.blocks[i] = (uint32_t)f32_tiles(l.p[i], edge);
    grid += l.blocks[i];
  }
  if (grid > 0x7FFFFFFFull) return fail(SIF_E_INVAL, "gemm_f32: grid too large");
  if (wide) hipLaunchKernelGGL(gemm_f32_kernel<2>, dim3((uint32_t)grid), dim3(256), 0, s, l, ctl);
  else hipLaunchKernelGGL(gemm_f32_kernel<1>, dim3((uint32_t)grid), dim3(256), 0, s, l, ctl);
  return check_launch("gemm_f32");
}

F32Product f32_product_of(const float* a, int64_t a_sm, int64_t a_sk, const float* b, int64_t b_sk, int64_t b_sn, float* c, int64_t ldc,
                          uint32_t m, uint32_t n, uint32_t k, uint32_t epi, const float* bias, float* aux) {
  F32Product p{};
  p.a = a; p.a_sm = a_sm; p.a_sk = a_sk; p.b = b; p.b_sk = b_sk; p.b_sn = b_sn; p.c = c; p.ldc = ldc;
  p.m = m; p.n = n; p.k = k; p.epi = epi; p.bias = bias; p.aux = aux;
  return p;
}

sif_status launch_gemm_f32(const float* a, int64_t a_sm, int64_t a_sk, const float* b, int64_t b_sk, int64_t b_sn,
                           float* c, int64_t ldc, uint32_t m, uint32_t n, uint32_t k, uint32_t epi, const float* bias,
                           float* aux, hipStream_t s, const KCtl& ctl) {
  F32Launch l{};
  l.p[0] = f32_product_of(a, a_sm, a_sk, b, b_sk, b_sn, c, ldc, m, n, k, epi, bias, aux);
  return launch_f32(l, s, ctl);
}

}  // namespace sif
