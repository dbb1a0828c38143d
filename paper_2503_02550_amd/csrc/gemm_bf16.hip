// bf16 matrix product on the gfx950 MFMA units, fp32 accumulation, fused epilogues.
//
//   C[M,N] = alpha * sum_k A(m,k) B(k,n)   (+ bias, GELU, residual, GELU' multiply)
//
// These kernels serve every dense contraction of the training step and of the inference forward pass (the
// "kernels issued by the training instance" and the inference kernels the Kernel Barrier releases, Sec. 3.1):
// forward products (A [M][K], B [N][K]), data gradients (B [K][N]), weight gradients (A [K][M], B [K][N]) and
// the per-head attention products via two batch strides.
//
// Every wavefront owns a grid of v_mfma_f32_16x16x32_bf16 accumulators; operand tiles, 64 k deep, travel from global
// memory straight into LDS (buffer_load_dwordx4 ... lds) and from there into MFMA operand registers.  LDS holds an
// operand as it lies in memory: rows of 64 k (128 bytes, XOR-swizzled in 16-byte chunks so that reads spread over the
// banks) or, where the other dimension is contiguous, k-rows that the LDS read itself transposes (ds_read_b64_tr_b16).
//
// Three kernels, chosen by a model of their times (gemm_choose, gemm_kernel), each compiled for the common epilogues and for the
// rare ones (gemm_rare):
//   gemm_fed_kernel    the smaller tiles where no CU gets more than one: wavefronts of their own for the fetches.
//   gemm_ring_kernel   one tile per block, a ring of two to four K steps in LDS.  Tiles from 32x64 (a handful of rows)
//                      over 64x64, 128x64 and 128x128 to 256x128, so that a product of any size finds one that
//                      spreads it over the chip.
//   gemm_pp_kernel     256x256 tiles, persistent blocks, the two wavefronts of a SIMD alternate between memory phases
//                      and matrix phases: the fewest bytes per product, for what fills the chip with such tiles.
//
// What a K step costs, measured: a compute unit takes in about 65 bytes/ns of fetches when its wavefronts wait for all
// of them at a barrier and 100 when fetches stay in flight across it; a wavefront issues in order, so everything that
// is not an MFMA - LDS reads, fetches, address arithmetic, branches - delays the MFMAs behind it unless it stands
// between them.  Hence: no branch and no address arithmetic in the steady part of a loop (the ring's slots are constants
// of an unrolled body), fragments of the next K step read between the MFMAs of this one, fetches waited for by count.
// (Two K steps in LDS, waited for as a whole, were 4096 x 768 x 3072: 36 us, 77 x 768 x 3072: 23 us, 8192 x 768 x 3072:
// 44 us, 2048 x 4096 x 8192 as a weight gradient: 130 us; now 23.5, 8.2, 38.6 and 112, launches back to back.)
//
// Which MFMA: with operands in registers and every CU busy the chip sustains 2.03 PFLOP/s of 16x16x32 and 1.82 of 32x32x16 (the
// clock follows the power: per flop the narrower shape moves half the accumulator words), reading each operand from LDS 1.63 and
// 1.54; both give the same bits.  8192^3 769 -> 715 us with it, 131072 x 768 x 3072 with bias and residual 522 -> 498, 131072 x
// 3072 x 768 with GELU 598 -> 574.
//
// Results depend neither on the grid nor on the tile: each output element is reduced over K in one fixed order
// (ascending, 32 at a time) by one wavefront, so launching a row range of the same problem, or another configuration,
// gives bit-identical values.
#include <algorithm>
#include <math.h>

#include "common.h"
#include "specinf.h"
#include "launch.h"

namespace sif {

constexpr int BK = 64;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

struct GemmP {
  const bf16_t* a; const bf16_t* b; void* c; const bf16_t* bias; const void* res; bf16_t* aux;
  uint32_t m, n, k, lda, ldb, ldc, epi, k_causal, batch_inner, tiles_m, tiles_n, k_limit;
  long long a_so, a_si, b_so, b_si, c_so, c_si;
  float alpha;
  // a launch over several products at once (no batch): `group` points to their records in device memory, each with the
  // number of the launch's first block that works on it (a multiple of 8)
  const GemmP* group;
  uint32_t group_n, tile_base;
};

// ---------------------------------------------------------------------------------------------- operands in LDS
// LDS tile: rows x 64 k (bf16), 128 bytes per row = eight 16-byte chunks, no padding.  Chunk c of row r lives at chunk
// position c ^ key(r).  An MFMA operand is 16 rows of four consecutive chunks, lane l's row l%16 and chunk l/16.  A read takes
// 16 lanes per cycle over 64 banks, and not consecutive ones: 0-3, 12-15 and 20-27 go together, and 4-11, 16-19 and 28-31 (rows
// 0-3 and 12-15 of one chunk with rows 4-11 of the next).  With row % 8 as the key these are 16 different (row parity, position)
// pairs: 4.2 cycles a read with eight wavefronts at it, where (row % 8) ^ (row / 8 % 2), as good for 32 rows of two chunks,
// takes 8.0.
__device__ __forceinline__ uint32_t swz_key(uint32_t row) { return row & 7u; }
__device__ __forceinline__ uint32_t lds_off(uint32_t row, uint32_t chunk) { return row * BK + ((chunk ^ swz_key(row)) << 3); }

// A K-major operand (memory [k][row]) is staged as it lies in memory: LDS tile [64 k][ROWS], 2*ROWS bytes per k, the
// 32-byte units (16 rows) of k-row k stored at unit position unit ^ key(k).  The MFMA operand - eight consecutive k for
// one row per lane - is then fetched with the transposing LDS read of gfx950 (ds_read_b64_tr_b16): within each group of
// 16 lanes, source lane s supplies the address of four consecutive rows at k = k0 + s/4, rows r0 + 4*(s%4).., and lane i
// receives rows r0 + i at k0..k0+3.  Two such reads make one operand, the four groups of lanes reading 8 k each.  The key makes
// the eight pieces of 32 bytes that half a wavefront reads (k-rows k0..k0+3 and k0+8..k0+11) lie in different banks.
typedef short short4_lds __attribute__((ext_vector_type(4)));
template <int ROWS>
__device__ __forceinline__ uint32_t kmajor_key(uint32_t k) {
  const uint32_t far = (k >> 3) & 1u;
  return ROWS >= 128 ? ((k & 3u) << 1) | far : ROWS == 64 ? (k & 2u) | far : far;
}
// element offset in such a tile of the address that this lane supplies for 16 rows from unit `unit`, first k = 0
template <int ROWS>
__device__ __forceinline__ uint32_t kmajor_off(uint32_t unit) {
  const uint32_t lane = threadIdx.x & 63, s = lane & 15, k = (lane >> 4) * 8 + (s >> 2);
  return k * ROWS + ((unit ^ kmajor_key<ROWS>(k)) << 4) + 4 * (s & 3u);
}
typedef __attribute__((address_space(3))) short4_lds* kmajor_ptr;
template <int ROWS>
__device__ __forceinline__ bf16x8 kmajor_frag(uint32_t lds) {                // (LDS byte address)
  const short4_lds lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((kmajor_ptr)(uintptr_t)lds);
  const short4_lds hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((kmajor_ptr)(uintptr_t)(lds + 4 * ROWS * 2));
  typedef short short8_v __attribute__((ext_vector_type(8)));
  const short8_v v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  return __builtin_bit_cast(bf16x8, v);
}
// 16 rows from `rowbase16` (a multiple of 16), k slice ks of 32, as an MFMA operand
template <int LAYOUT, int ROWS>
__device__ __forceinline__ bf16x8 operand_frag(const bf16_t* tile, uint32_t rowbase16, int ks) {
  const uint32_t lane = threadIdx.x & 63;
  if (LAYOUT == 0) return *reinterpret_cast<const bf16x8*>(tile + lds_off(rowbase16 + (lane & 15), ks * 4 + (lane >> 4)));
  return kmajor_frag<ROWS>((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const bf16_t*)tile + 2 * (kmajor_off<ROWS>(rowbase16 >> 4) + ks * (32 * ROWS)));
}
// The same for a ring of such tiles: T operands 16 rows apart, read from slot after slot with the distance as the read's
// immediate offset (16 bits).  The registers that hold the lane's addresses are few - one per k slice, or per operand where
// the LDS read transposes, and again per 64 KB of ring - and opaque to the compiler, which otherwise keeps an address for
// nearly every read (256x128 tiles, both operands k-major: 41 of them, 23 spilled, reloaded inside the loop).
template <int LAYOUT, int ROWS, int T, int ST>
struct RingFrags {
  static constexpr uint32_t TILE = ROWS * BK * 2, PER = 65536 / TILE;      // bytes of a slot, slots within reach
  static constexpr int N = LAYOUT == 0 ? 2 : T, WINDOWS = (ST + PER - 1) / PER;
  uint32_t at[WINDOWS][N];
  __device__ __forceinline__ void init(uint32_t ring, uint32_t rowbase16) {      // `ring`: LDS byte address of slot 0
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (int w = 0; w < WINDOWS; ++w)
#pragma unroll
      for (int q = 0; q < N; ++q) {
        at[w][q] = ring + w * (PER * TILE) + 2 * (LAYOUT == 0 ? lds_off(rowbase16 + (lane & 15), q * 4 + (lane >> 4)) : kmajor_off<ROWS>((rowbase16 >> 4) + q));
        asm("" : "+v"(at[w][q]));
      }
  }
  // operand i, k slice ks of a slot; `beyond` = where it starts past the slots of window w
  __device__ __forceinline__ bf16x8 read(int w, uint32_t beyond, int i, int ks) const {
    typedef __attribute__((address_space(3))) const bf16x8* row_ptr;
    if (LAYOUT == 0) return *(row_ptr)(uintptr_t)(at[w][ks] + beyond + i * (16 * BK * 2));
    return kmajor_frag<ROWS>(at[w][i] + beyond + ks * (32 * ROWS * 2));
  }
  __device__ __forceinline__ bf16x8 read_tile(int slot, int i, int ks) const { return read(slot / PER, slot % PER * TILE, i, ks); }      // (slot a constant)
  template <int SLOT>
  __device__ __forceinline__ bf16x8 read_slot(int i, int ks) const { return read(SLOT / PER, SLOT % PER * TILE, i, ks); }
};

// ---------------------------------------------------------------------------------------------- fetches
// One fetch instruction writes the 64 lanes' 16 bytes to consecutive LDS addresses from the scalar M0 on, 1 KB per
// wavefront, so a lane's place in the tile is fixed and the swizzle is applied to what it fetches.  The instruction is
// written as assembly: the compiler would otherwise make every LDS read wait for every fetch in flight.  `volatile` and
// "memory" keep it in its place between the barriers.  (M0 is reserved: the compiler keeps nothing in it, and naming it as
// clobbered is no help, so nothing else in these kernels may use it; a test looks through the built instructions.)
constexpr uint32_t kOutside = 0x80000000u;      // an offset beyond the resource's extent: the lane's 16 bytes are zeros
__device__ __forceinline__ void fetch16(const i32x4& rsrc, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc) : "memory");
}
// a buffer resource over the operand from `base` on: raw bytes, extent 2 GB (what a lane's offset within a tile can be,
// see gemm_fill), so that only a 32-bit offset per lane travels to the memory pipeline
__device__ __forceinline__ i32x4 operand_rsrc(uint64_t base) {
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((uint32_t)base);
  r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(base >> 32));
  r[2] = (int)kOutside;
  r[3] = 0x00020000;
  return r;
}
// What the threads of a block fetch of one operand tile of ROWS rows and 64 k; instruction i, thread t covers
//   LAYOUT 0 (memory [row][k]): LDS row (i*THREADS + t) / 8, chunk position t % 8 = logical chunk (t % 8) ^ key(row)
//   LAYOUT 1 (memory [k][row]): k-row (i*THREADS + t) / (ROWS/8), 16 bytes t % (ROWS/8) of it, units swizzled with k
// The tile may be part PART of a larger one: LDS row r is row (r / G) * GS + PART * G + r % G of it.  Rows past the
// operand's last one read as zeros, and so does what lies past the end of K in a last, ragged step (issue_last).
template <int LAYOUT, int ROWS, int THREADS, int G, int GS, int PART>
struct TileFetch {
  static_assert(ROWS * 8 % THREADS == 0, "whole 16-byte vectors per thread and tile");
  static constexpr int NV = ROWS * 8 / THREADS;
  uint32_t voff[NV];
  __device__ __forceinline__ static uint32_t unit(int i, uint32_t tid) { return i * THREADS + tid; }
  __device__ __forceinline__ static uint32_t row_of(uint32_t r) { return (r / G) * GS + PART * G + r % G; }
  __device__ __forceinline__ static uint32_t k_of(int i, uint32_t tid) {      // first k of the 16 bytes
    const uint32_t u = unit(i, tid);
    return LAYOUT == 0 ? ((u & 7u) ^ swz_key(u >> 3)) * 8 : u / (ROWS / 8);
  }
  __device__ __forceinline__ void init(uint32_t ld, uint32_t rows_left, uint32_t tid) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const uint32_t u = unit(i, tid), k = k_of(i, tid);
      if (LAYOUT == 0) {
        const uint32_t r = row_of(u >> 3);
        voff[i] = r < rows_left ? (r * ld + k) * 2u : kOutside;
      } else {
        const uint32_t q = u % (ROWS / 8), r = row_of(((q >> 1) ^ kmajor_key<ROWS>(k)) * 16 + (q & 1u) * 8);
        voff[i] = r < rows_left ? (k * ld + r) * 2u : kOutside;
      }
    }
  }
  __device__ __forceinline__ void issue(const i32x4& rsrc, uint32_t lds, uint32_t wave, int i) const {
    fetch16(rsrc, voff[i], lds + i * (THREADS * 16) + wave * 1024);
  }
  __device__ __forceinline__ void issue_last(const i32x4& rsrc, uint32_t lds, uint32_t wave, int i, uint32_t k_left, uint32_t tid) const {
    fetch16(rsrc, k_of(i, tid) < k_left ? voff[i] : kOutside, lds + i * (THREADS * 16) + wave * 1024);
  }
};
// waits until at most N vector memory operations of this wavefront are outstanding (they complete in order)
template <int N>
__device__ __forceinline__ void wait_vm() { __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14)); }
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }
// a block barrier that waits for nothing by itself (the fences only keep the compiler from moving accesses across it)
__device__ __forceinline__ void barrier_only() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// ---------------------------------------------------------------------------------------------- epilogue
// What one wavefront stores is its (TI*32) x (TJ*32) part of an output tile, first row mw, first column nw.  Accumulator
// element r of lane l is row (l/16)*4 + r, column l%16 of its 16x16 tile.  The values pass through kStage bytes of LDS of the
// wavefront's own, as many at a time as give each lane one vector, so that every global access - residual, auxiliary tensor,
// result - is a 16-byte vector along a row; no block-wide barrier is needed.
//
// Straight-line code: which tensors are read and written is decided once per tile (a variant each), and what lies past the
// last row or column is left out by the range check of the buffer resources, not by branches; LDS operations of a wavefront
// complete in order, so the next pass is written while the last one's reads are under way.  (What bounds it: with little
// on the chip a wavefront's own instructions, with a tile on every CU the rate at which memory takes 32 MB at once.  With
// the decisions taken element by element and a wait per pass, an eighth of a 256x256 tile took 5800 cycles plain and 13900
// with a residual, nothing else on the chip; now 3300 and 5700.  131072 x 768 x 3072 with bias and residual 549 -> 539 us,
// x 3072 x 768 with GELU 679 -> 650, 131072 x 768 x 768 with residual 200 -> 187, 4096 x 4096 x 512 with residual 29.4 -> 26.8;
// six layers of d 2048 18.2 -> 17.0 ms a step, a batch of 4096 tokens through twelve of d 768 1.61 -> 1.54 ms.)

// `bytes` from `base` on as a buffer resource, at most 2 GB: offsets beyond it read as zeros and are not written
__device__ __forceinline__ __amdgpu_buffer_rsrc_t result_rsrc(const void* base, uint64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)(bytes < kOutside ? bytes : kOutside), 0x00020000);
}
__device__ __forceinline__ uint4 read16(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
// 16 bytes of a result, stored with the non-temporal hint (2).  A product's output is written once and read by a later
// kernel, and the chip's CUs write their tiles in bursts that exceed what the L2 takes in at once: stores that do not
// claim L2 lines are acknowledged sooner (the wavefront waits for them at its next wait for a fetch), and they leave
// the operand panels, which the tiles of an XCD share, in the L2.
__device__ __forceinline__ void write16(__amdgpu_buffer_rsrc_t r, uint32_t off, const uint4& v, bool streamed = true) {
  if (streamed) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)off, 0, 2);
  else __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, (int)off, 0, 0);
}
// LDS accesses of a wavefront's lanes to each other's data stay in order: for the compiler, the hardware keeps it anyway
__device__ __forceinline__ void lanes_in_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Where the values of a pass lie in the staging LDS: `t` numbers its rows from the top, W columns each (W = 64 or 32); the keys
// make the groups of 16 lanes that write at the same time, in different rows, and what 16 lanes read in a cycle (see swz_key) fall
// on different banks.  (With the MFMAs' operands exchanged a lane holds four columns of a row instead, and a write is four words
// wide; that is as fast, 1 % slower where a residual or an auxiliary tensor has to come into that layout.)
constexpr uint32_t kStage = 2048;
constexpr int gemm_room(uint32_t bytes, uint32_t wavefronts) { return bytes >= 4 * wavefronts * kStage ? 4 : bytes >= 2 * wavefronts * kStage ? 2 : 1; }      // areas for each
template <int TJ>
struct Staging {
  static_assert(TJ == 1 || TJ == 2, "the keys below");
  static constexpr int W = TJ * 32, CPR = W / 8;                     // columns, 8-column chunks per row
  // fp32 words: a pass takes RPG of a lane's four rows of a 16x16 tile, PASSES of them a tile
  static constexpr int RPG = TJ == 2 ? 2 : 4, PASSES = 4 / RPG, ROWS = 4 * RPG;
  __device__ __forceinline__ static uint32_t row_of(uint32_t t) { return t / RPG * 4 + t % RPG; }                    // (in the first pass of a tile)
  __device__ __forceinline__ static uint32_t key(uint32_t t) { return TJ == 2 ? ((t >> 1) & 3u) << 2 | ((t >> 1) & 1u) : ((t >> 2) & 1u) << 2; }      // of chunks of four words
  __device__ __forceinline__ static uint32_t at(uint32_t t, uint32_t col) { return t * W + ((((col >> 2) ^ key(t)) << 2) | (col & 3u)); }
  // pass `ps` of a row of tiles
  __device__ __forceinline__ static void put(float* sW, const floatx4 (&acc)[2 * TJ], int ps, uint32_t lane) {
#pragma unroll
    for (int j = 0; j < 2 * TJ; ++j)
#pragma unroll
      for (int e = 0; e < RPG; ++e) sW[at((lane >> 4) * RPG + e, j * 16 + (lane & 15))] = acc[j][ps * RPG + e];
  }
  // a lane's chunk: columns (lane % CPR) * 8 of row t = lane / CPR
  __device__ __forceinline__ static void get(const float* sW, uint32_t lane, float4 (&q)[2]) {
    const uint32_t t = lane / CPR, c = (lane % CPR * 2) ^ key(t);
    q[0] = *reinterpret_cast<const float4*>(sW + t * W + (c << 2));
    q[1] = *reinterpret_cast<const float4*>(sW + t * W + ((c ^ 1u) << 2));
  }
  // all passes of a tile in areas that follow each other: its rows in their order
  __device__ __forceinline__ static uint32_t tile_key(uint32_t t) { return TJ == 2 ? ((t >> 2) & 3u) << 2 | ((t >> 1) & 1u) : key(t); }
  __device__ __forceinline__ static void put_tile(float* sW, const floatx4 (&acc)[2 * TJ], uint32_t lane) {
#pragma unroll
    for (int j = 0; j < 2 * TJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t t = (lane >> 4) * 4 + e;
        sW[t * W + ((j * 16 + (lane & 15)) ^ (tile_key(t) << 2))] = acc[j][e];
      }
  }
  // a lane's chunk in the k-th pass' share of them: rows k * ROWS + lane / CPR
  __device__ __forceinline__ static void get_tile(const float* sW, int k, uint32_t lane, float4 (&q)[2]) {
    const uint32_t t = k * ROWS + lane / CPR, c = (lane % CPR * 2) ^ tile_key(t);
    q[0] = *reinterpret_cast<const float4*>(sW + t * W + (c << 2));
    q[1] = *reinterpret_cast<const float4*>(sW + t * W + ((c ^ 1u) << 2));
  }
  // pairs of vertically adjacent bf16 results as words: a pass takes PAIRED rows of tiles
  static constexpr int PAIRED = TJ == 2 ? 1 : 2;
  __device__ __forceinline__ static uint32_t pair_key(uint32_t t) { return TJ == 2 ? ((t >> 1) & 3u) << 4 | ((t >> 1) & 1u) << 2 : ((t >> 1) & 1u) << 4; }
};
__device__ __forceinline__ uint4 pack_bf8(const float (&v)[8]) { return make_uint4(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])); }
__device__ __forceinline__ void unpack_bf8(const uint4& q, float (&v)[8]) {
  v[0] = bflo(q.x); v[1] = bfhi(q.x); v[2] = bflo(q.y); v[3] = bfhi(q.y); v[4] = bflo(q.z); v[5] = bfhi(q.z); v[6] = bflo(q.w); v[7] = bfhi(q.w);
}

// bf16 variants that read nothing but the bias (plain, bias, bias + GELU without the pre-activation output) are finished in the
// accumulator layout, where a lane's column is fixed, and staged as bf16: two vertically adjacent results share a 32-bit
// word, half the LDS traffic of the fp32 staging below.  A lane then reads eight words = eight columns of two rows,
// separates the rows with byte permutes and stores two 16-byte row vectors.
template <int TI, int TJ, bool GELU>
__device__ __forceinline__ void gemm_store_packed(const GemmP& p, floatx4 (&acc)[2 * TI][2 * TJ], float* sW, uint32_t mw, uint32_t nw, size_t c_off, uint32_t lane,
                                                  const bf16_t* bias_s) {
  typedef Staging<TJ> S;
  constexpr int PASSES = 2 * TI / S::PAIRED;
  uint32_t* const sP = reinterpret_cast<uint32_t*>(sW);
  const uint32_t g = lane >> 4, pitch = p.ldc * 2;        // pitch: bytes from row to row
  const uint32_t tl = lane / S::CPR, c8 = lane % S::CPR;
  const auto c = result_rsrc(reinterpret_cast<bf16_t*>(p.c) + c_off + (size_t)mw * p.ldc + nw, mw < p.m ? (uint64_t)(p.m - mw) * pitch : 0);
  const uint32_t off = nw + c8 * 8 < p.n ? tl * 2 * pitch + c8 * 16 : kOutside;
  float bcol[2 * TJ];
#pragma unroll
  for (int j = 0; j < 2 * TJ; ++j) bcol[j] = p.bias != nullptr ? bf2f(bias_s[j * 16 + (lane & 15)]) : 0.f;
  uint4 w[2][2];
  auto finish = [&](int pass) {
    const uint4 &w0 = w[pass & 1][0], &w1 = w[pass & 1][1];
    const uint32_t o = off + (uint32_t)(pass * S::PAIRED * 16) * pitch;
    write16(c, o, make_uint4(__builtin_amdgcn_perm(w0.y, w0.x, 0x05040100), __builtin_amdgcn_perm(w0.w, w0.z, 0x05040100),
                             __builtin_amdgcn_perm(w1.y, w1.x, 0x05040100), __builtin_amdgcn_perm(w1.w, w1.z, 0x05040100)));
    write16(c, o + pitch, make_uint4(__builtin_amdgcn_perm(w0.y, w0.x, 0x07060302), __builtin_amdgcn_perm(w0.w, w0.z, 0x07060302),
                                     __builtin_amdgcn_perm(w1.y, w1.x, 0x07060302), __builtin_amdgcn_perm(w1.w, w1.z, 0x07060302)));
  };
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
#pragma unroll
    for (int i = 0; i < S::PAIRED; ++i)
#pragma unroll
      for (int j = 0; j < 2 * TJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; r += 2) {
          const floatx4& v = acc[pass * S::PAIRED + i][j];
          float x0 = v[r] * p.alpha + bcol[j], x1 = v[r + 1] * p.alpha + bcol[j];
          if (GELU) { x0 = gelu_fast(x0); x1 = gelu_fast(x1); }
          const uint32_t t = i * 8 + g * 2 + (r >> 1);
          sP[t * S::W + ((j * 16 + (lane & 15)) ^ S::pair_key(t))] = pack_bf2(x0, x1);
        }
    lanes_in_order();
    const uint32_t pos = (c8 * 8) ^ S::pair_key(tl);
    w[pass & 1][0] = *reinterpret_cast<const uint4*>(sP + tl * S::W + pos);
    w[pass & 1][1] = *reinterpret_cast<const uint4*>(sP + tl * S::W + (pos ^ 4u));
    lanes_in_order();
    if (pass > 0) finish(pass - 1);
    __builtin_amdgcn_sched_barrier(0);                    // (no more than two passes in registers)
  }
  finish(PASSES - 1);
}

// bf16 variants that read a tensor of the result's shape or write the pre-activation too: staged as fp32, a chunk of eight columns
// per lane and pass.  What is read is requested for 64 rows ahead: a wait for it also waits for the stores before it.  Those that read
// are staged by whole tiles, 32 rows at once, where the wavefront has the areas for it (not on 256x256 tiles), so that a request
// or a store covers rows that follow each other: 8192 x 2304 x 768 with a residual 39.5 -> 37.7 us, 16384 x 768 x 256 with GELU' 17.7 ->
// 16.7, fourteen shapes 0.5 to 5 % less.  (The variant with the pre-activation, which only writes, takes up to 2 % more that way.)
enum { kRowsResidual, kRowsGeluAux, kRowsGeluGrad };
template <int TI, int TJ, int KIND, int ROOM>
__device__ __forceinline__ void gemm_store_rows(const GemmP& p, floatx4 (&acc)[2 * TI][2 * TJ], float* sW, uint32_t mw, uint32_t nw, size_t c_off, uint32_t lane,
                                                const bf16_t* bias_s) {
  typedef Staging<TJ> S;
  constexpr int PER = 2 * S::PASSES;                      // passes, and vectors per lane, of 32 rows
  constexpr bool READS = KIND == kRowsResidual || KIND == kRowsGeluGrad;
  constexpr int AHEAD = TI < 2 ? TI : 2, TURN = !READS ? 1 : ROOM >= PER ? PER : ROOM >= S::PASSES ? S::PASSES : 1;      // passes of a turn
  const uint32_t pitch = p.ldc * 2, c8 = lane % S::CPR;
  const size_t first = c_off + (size_t)mw * p.ldc + nw;
  const uint64_t extent = mw < p.m ? (uint64_t)(p.m - mw) * pitch : 0;
  const auto c = result_rsrc(reinterpret_cast<bf16_t*>(p.c) + first, extent);
  const auto other = result_rsrc(KIND == kRowsResidual ? reinterpret_cast<const bf16_t*>(p.res) + first : p.aux + first, extent);
  constexpr bool IN_ORDER = TURN >= S::PASSES;                       // whole tiles, their rows in their order
  const uint32_t off0 = nw + c8 * 8 < p.n ? (IN_ORDER ? lane / S::CPR : S::row_of(lane / S::CPR)) * pitch + c8 * 16 : kOutside;
  auto off = [&](int pass) { return off0 + (uint32_t)(IN_ORDER ? pass * S::ROWS : pass / S::PASSES * 16 + pass % S::PASSES * S::RPG) * pitch; };
  uint4 q[AHEAD][PER];
  auto request = [&](int i) {
    if constexpr (READS) {
#pragma unroll
      for (int k = 0; k < PER; ++k) q[i % AHEAD][k] = read16(other, off(i * PER + k));
    }
  };
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) request(i);
  float bias[8];
  unpack_bf8(p.bias != nullptr ? *reinterpret_cast<const uint4*>(bias_s + c8 * 8) : make_uint4(0, 0, 0, 0), bias);
  float4 s[2][TURN][2];
  auto finish = [&](int pass) {
    const float4 (&q01)[2] = s[pass / TURN & 1][pass % TURN];
    float v[8] = {q01[0].x, q01[0].y, q01[0].z, q01[0].w, q01[1].x, q01[1].y, q01[1].z, q01[1].w};
    const uint32_t o = off(pass);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] * p.alpha + bias[e];
    if constexpr (READS) {
      float x[8];
      unpack_bf8(q[pass / PER % AHEAD][pass % PER], x);
#pragma unroll
      for (int e = 0; e < 8; ++e) { if (KIND == kRowsResidual) v[e] += x[e]; else v[e] *= gelu_grad_fast(x[e]); }
    }
    if constexpr (KIND == kRowsGeluAux) {
      write16(other, o, pack_bf8(v), false);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = gelu_fast(v[e]);
    }
    write16(c, o, pack_bf8(v));
  };
  auto finish_turn = [&](int turn) {
#pragma unroll
    for (int k = 0; k < TURN; ++k) finish(turn * TURN + k);
  };
#pragma unroll
  for (int turn = 0; turn < TI * PER / TURN; ++turn) {
    if constexpr (IN_ORDER) {
#pragma unroll
      for (int k = 0; k < TURN; k += S::PASSES) S::put_tile(sW + k * (kStage / 4), acc[(turn * TURN + k) / S::PASSES], lane);
    } else {
      S::put(sW, acc[turn / S::PASSES], turn % S::PASSES, lane);
    }
    lanes_in_order();
#pragma unroll
    for (int k = 0; k < TURN; ++k) {
      if constexpr (IN_ORDER) S::get_tile(sW + k / S::PASSES * (S::PASSES * kStage / 4), k % S::PASSES, lane, s[turn & 1][k]);
      else S::get(sW, lane, s[turn & 1][k]);
    }
    lanes_in_order();
    if (turn > 0) {
      finish_turn(turn - 1);
      const int done = turn * TURN;
      if (done % PER == 0 && done / PER - 1 + AHEAD < TI) request(done / PER - 1 + AHEAD);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  finish_turn(TI * PER / TURN - 1);
}

// fp32 results, four columns per lane, so that one store writes rows of the wavefront's part whole.  (4096 x 4096 x 512 on 256x256
// tiles 26 us, with eight columns per lane in two stores 30.)
template <int TI, int TJ>
__device__ __forceinline__ void gemm_store_f32(const GemmP& p, floatx4 (&acc)[2 * TI][2 * TJ], float* sW, uint32_t mw, uint32_t nw, size_t c_off, uint32_t lane,
                                               const bf16_t* bias_s) {
  typedef Staging<TJ> S;
  constexpr int CPR = S::W / 4;
  const uint32_t t = lane / CPR, c4 = lane % CPR, n = nw + c4 * 4, pitch = p.ldc * 4;
  const auto c = result_rsrc(reinterpret_cast<float*>(p.c) + c_off + (size_t)mw * p.ldc + nw, mw < p.m ? (uint64_t)(p.m - mw) * pitch : 0);
  const uint32_t off = n < p.n ? S::row_of(t) * pitch + c4 * 16 : kOutside;
  const uint2 bq = p.bias != nullptr ? *reinterpret_cast<const uint2*>(bias_s + c4 * 4) : make_uint2(0, 0);
  const float bias[4] = {bflo(bq.x), bfhi(bq.x), bflo(bq.y), bfhi(bq.y)};
  float4 s[2][2];                              // rows t and t + ROWS/2, which is eight rows of the tile further down
  auto finish = [&](int pass) {
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const float4 q = s[pass & 1][it];
      write16(c, off + (uint32_t)(pass / S::PASSES * 16 + pass % S::PASSES * S::RPG + it * 8) * pitch,
              make_uint4(__float_as_uint(q.x * p.alpha + bias[0]), __float_as_uint(q.y * p.alpha + bias[1]), __float_as_uint(q.z * p.alpha + bias[2]), __float_as_uint(q.w * p.alpha + bias[3])),
              false);
    }
  };
#pragma unroll
  for (int pass = 0; pass < 2 * TI * S::PASSES; ++pass) {
    S::put(sW, acc[pass / S::PASSES], pass % S::PASSES, lane);
    lanes_in_order();
#pragma unroll
    for (int it = 0; it < 2; ++it) s[pass & 1][it] = *reinterpret_cast<const float4*>(sW + S::at(t + it * (S::ROWS / 2), c4 * 4));
    lanes_in_order();
    if (pass > 0) finish(pass - 1);
    __builtin_amdgcn_sched_barrier(0);
  }
  finish(2 * TI * S::PASSES - 1);
}

// bf16 results of the other combinations - a residual together with GELU or GELU' - and of rows further apart than the offsets
// above reach: vectors too, but 64-bit addresses and decisions while it runs.  The first tensor that is read is requested 32
// rows ahead (64 where a wavefront has as many), the residual beside an auxiliary tensor for 32 rows at once (16 on 256x256 tiles, which
// have no registers for more): a wait for it also waits for the stores before it.  (One element at a time 4096 x 4096 x 512 on
// 256x256 tiles took 115 us with GELU and a residual, 148 with GELU' and a residual, 75 with both of GELU and GELU'; now 27, 39 and
// 36, with the residual alone 25.5; 77 x 768 x 768 with rows of 2 M elements 6.8 and now 5.6.  With a request for every 8 rows, and
// 32 ahead everywhere, 28, 43 and 38; on 128x128 tiles GELU and a residual 31, now 28, with the pre-activation 42 and 37.)
template <int TI, int TJ>
__device__ __forceinline__ void gemm_store_mixed(const GemmP& p, floatx4 (&acc)[2 * TI][2 * TJ], float* sW, uint32_t mw, uint32_t nw, size_t c_off, uint32_t lane,
                                                 const bf16_t* bias_s) {
  typedef Staging<TJ> S;
  constexpr int PER = 2 * S::PASSES, AHEAD = TI == 2 ? 2 : 1, LATE = TI > 2 ? PER / 2 : PER;
  const uint32_t c8 = lane % S::CPR, n = nw + c8 * 8, row0 = mw + S::row_of(lane / S::CPR);
  const bool grad = (p.epi & SIF_EPI_GELU_GRAD) != 0, gelu = (p.epi & SIF_EPI_GELU) != 0, residual = (p.epi & SIF_EPI_RESIDUAL) != 0;
  const bf16_t* const res = reinterpret_cast<const bf16_t*>(p.res);
  const bf16_t* const first = grad ? p.aux : residual ? res : nullptr;      // the tensor that is requested ahead
  // a lane's row in a pass, and where what is read for it lies: beyond the last row or column, in these
  auto row_of = [&](int pass) { return row0 + pass / S::PASSES * 16 + pass % S::PASSES * S::RPG; };
  auto read_at = [&](int pass) { return c_off + (size_t)min(row_of(pass), p.m - 1) * p.ldc + min(n, p.n - 8); };
  uint4 ahead[AHEAD][PER], late[LATE];          // late: the residual where it is not the tensor requested ahead
  auto request = [&](int i) {
    if (first == nullptr) return;
#pragma unroll
    for (int k = 0; k < PER; ++k) ahead[i % AHEAD][k] = *reinterpret_cast<const uint4*>(first + read_at(i * PER + k));
  };
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) request(i);
  float bias[8];
  unpack_bf8(p.bias != nullptr ? *reinterpret_cast<const uint4*>(bias_s + c8 * 8) : make_uint4(0, 0, 0, 0), bias);
#pragma unroll
  for (int pass = 0; pass < TI * PER; ++pass) {
    if (residual && grad && pass % LATE == 0) {
#pragma unroll
      for (int k = 0; k < LATE; ++k) late[k] = *reinterpret_cast<const uint4*>(res + read_at(pass + k));
    }
    S::put(sW, acc[pass / S::PASSES], pass % S::PASSES, lane);
    lanes_in_order();
    float4 q[2];
    S::get(sW, lane, q);
    const uint32_t m = row_of(pass);
    float v[8] = {q[0].x, q[0].y, q[0].z, q[0].w, q[1].x, q[1].y, q[1].z, q[1].w};
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = v[e] * p.alpha + bias[e];
    const bool inside = m < p.m && n < p.n;
    const size_t idx = c_off + (size_t)m * p.ldc + n;
    if (gelu) {
      if (p.aux != nullptr && inside) *reinterpret_cast<uint4*>(p.aux + idx) = pack_bf8(v);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] = gelu_fast(v[e]);
    }
    const uint4 a = ahead[pass / PER % AHEAD][pass % PER];
    float x[8];
    if (grad) {
      unpack_bf8(a, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] *= gelu_grad_fast(x[e]);
    }
    if (residual) {
      unpack_bf8(grad ? late[pass % LATE] : a, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) v[e] += x[e];
    }
    const uint4 w = pack_bf8(v);
    const u32x4 y = {w.x, w.y, w.z, w.w};
    if (inside) __builtin_nontemporal_store(y, reinterpret_cast<u32x4*>(reinterpret_cast<bf16_t*>(p.c) + idx));
    lanes_in_order();
    if (pass % PER == PER - 1 && pass / PER + AHEAD < TI) request(pass / PER + AHEAD);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// fp32 results with anything else, the auxiliary tensor and the residual requested as above.  (4096 x 4096 x 512 on 256x256 tiles with a
// residual 41 us, with GELU' 41, with both GELU and a residual 48; with a request for every 8 rows 50, 45 and 60, one element at a
// time 98, 101 and 134.  On 128x128 tiles 43, 40 and 51; with a request for every 8 rows 53, 47 and 63.)
template <int TI, int TJ>
__device__ __forceinline__ void gemm_store_f32_mixed(const GemmP& p, floatx4 (&acc)[2 * TI][2 * TJ], float* sW, uint32_t mw, uint32_t nw, size_t c_off, uint32_t lane,
                                                     const bf16_t* bias_s) {
  typedef Staging<TJ> S;
  constexpr int CPR = S::W / 4, PER = 2 * S::PASSES, AHEAD = TI == 2 ? 2 : 1, LATE = TI > 2 ? PER / 2 : PER;
  const uint32_t t = lane / CPR, c4 = lane % CPR, n = nw + c4 * 4, row0 = mw + S::row_of(t);
  const bool grad = (p.epi & SIF_EPI_GELU_GRAD) != 0, gelu = (p.epi & SIF_EPI_GELU) != 0, residual = (p.epi & SIF_EPI_RESIDUAL) != 0;
  const float* const res = reinterpret_cast<const float*>(p.res);
  auto row_of = [&](int pass, int it) { return row0 + pass / S::PASSES * 16 + pass % S::PASSES * S::RPG + it * 8; };      // (it: as in gemm_store_f32)
  auto read_at = [&](int pass, int it) { return c_off + (size_t)min(row_of(pass, it), p.m - 1) * p.ldc + min(n, p.n - 4); };
  uint2 z[AHEAD][PER][2];
  float4 r[LATE][2];
  auto request = [&](int i) {
    if (!grad) return;
#pragma unroll
    for (int k = 0; k < PER; ++k)
#pragma unroll
      for (int it = 0; it < 2; ++it) z[i % AHEAD][k][it] = *reinterpret_cast<const uint2*>(p.aux + read_at(i * PER + k, it));
  };
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) request(i);
  const uint2 bq = p.bias != nullptr ? *reinterpret_cast<const uint2*>(bias_s + c4 * 4) : make_uint2(0, 0);
  const float bias[4] = {bflo(bq.x), bfhi(bq.x), bflo(bq.y), bfhi(bq.y)};
#pragma unroll
  for (int pass = 0; pass < TI * PER; ++pass) {
    if (residual && pass % LATE == 0) {
#pragma unroll
      for (int k = 0; k < LATE; ++k)
#pragma unroll
        for (int it = 0; it < 2; ++it) r[k][it] = *reinterpret_cast<const float4*>(res + read_at(pass + k, it));
    }
    S::put(sW, acc[pass / S::PASSES], pass % S::PASSES, lane);
    lanes_in_order();
    float4 s[2];
#pragma unroll
    for (int it = 0; it < 2; ++it) s[it] = *reinterpret_cast<const float4*>(sW + S::at(t + it * (S::ROWS / 2), c4 * 4));
    lanes_in_order();
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const uint32_t m = row_of(pass, it);
      const bool inside = m < p.m && n < p.n;
      const size_t idx = c_off + (size_t)m * p.ldc + n;
      float v[4] = {s[it].x, s[it].y, s[it].z, s[it].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = v[e] * p.alpha + bias[e];
      if (gelu) {
        if (p.aux != nullptr && inside) *reinterpret_cast<uint2*>(p.aux + idx) = make_uint2(pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]));
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu_fast(v[e]);
      }
      if (grad) {
        const uint2 q = z[pass / PER % AHEAD][pass % PER][it];
        const float x[4] = {bflo(q.x), bfhi(q.x), bflo(q.y), bfhi(q.y)};
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] *= gelu_grad_fast(x[e]);
      }
      if (residual) {
        const float4 x = r[pass % LATE][it];
        v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
      }
      if (inside) *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.c) + idx) = make_float4(v[0], v[1], v[2], v[3]);
    }
    if (pass % PER == PER - 1 && pass / PER + AHEAD < TI) request(pass / PER + AHEAD);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A column count that is no multiple of eight: one element at a time, consecutive ones in consecutive lanes, what is read for a pass'
// eight of them at once (four on 256x256 tiles: unrolled for eight the passes are more than the compiler keeps in registers, and take
// four times as long).  (4096 x 4093 x 512 with a residual: 92 us with a wait for each element, now 41; plain 38, now 33.  4096 x
// 777 x 512, on smaller tiles, takes 0.89 to 0.93 of its time with four at once.)
template <int TI, int TJ>
__device__ __forceinline__ void gemm_store_single(const GemmP& p, floatx4 (&acc)[2 * TI][2 * TJ], float* sW, uint32_t mw, uint32_t nw, size_t c_off, uint32_t lane) {
  typedef Staging<TJ> S;
  constexpr int W = S::W, PER_ITEM = 64 / W, AT_ONCE = S::ROWS / PER_ITEM / (TI > 2 ? 2 : 1);      // PER_ITEM: rows of the staging that the lanes cover
  const bool grad = (p.epi & SIF_EPI_GELU_GRAD) != 0, gelu = (p.epi & SIF_EPI_GELU) != 0, residual = (p.epi & SIF_EPI_RESIDUAL) != 0, f32 = (p.epi & SIF_EPI_OUT_F32) != 0;
  const uint32_t col = lane % W, n = nw + col, n_read = min(n, p.n - 1);
  const float bias = p.bias != nullptr ? bf2f(p.bias[n_read]) : 0.f;
#pragma unroll
  for (int pass = 0; pass < 2 * TI * S::PASSES; ++pass) {
    S::put(sW, acc[pass / S::PASSES], pass % S::PASSES, lane);
    lanes_in_order();
#pragma clang loop unroll(disable)
    for (uint32_t t0 = W == 64 ? 0u : lane / W; t0 < (uint32_t)S::ROWS; t0 += PER_ITEM * AT_ONCE) {
      const uint32_t m = mw + pass / S::PASSES * 16 + pass % S::PASSES * S::RPG;
      auto t = [&](int e) { return t0 + e * PER_ITEM; };
      auto row = [&](int e) { return m + S::row_of(t(e)); };
      auto inside = [&](int e) { return row(e) < p.m && n < p.n; };
      auto at = [&](auto* base, int e) { return base + (c_off + (size_t)row(e) * p.ldc) + n; };      // (a row is the same for all lanes, or for half of them)
      auto read = [&](const auto* base, int e) { return (base + (c_off + (size_t)min(row(e), p.m - 1) * p.ldc))[n_read]; };
      float x[AT_ONCE], z[AT_ONCE], res[AT_ONCE];
      if (grad) {
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) z[e] = bf2f(read(p.aux, e));
      }
      if (residual && f32) {
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) res[e] = read(reinterpret_cast<const float*>(p.res), e);
      } else if (residual) {
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) res[e] = bf2f(read(reinterpret_cast<const bf16_t*>(p.res), e));
      }
#pragma unroll
      for (int e = 0; e < AT_ONCE; ++e) x[e] = sW[t(e) * W + (col ^ (S::key(t(e)) << 2))] * p.alpha + bias;      // (S::at, the key of the whole row)
      if (gelu) {
        if (p.aux != nullptr) {
#pragma unroll
          for (int e = 0; e < AT_ONCE; ++e) {
            z[e] = grad ? bf2f(f2bf(x[e])) : z[e];       // (GELU' of what is written)
            if (inside(e)) *at(p.aux, e) = f2bf(x[e]);
          }
        }
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) x[e] = gelu_fast(x[e]);
      }
      if (grad) {
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) x[e] *= gelu_grad_fast(z[e]);
      }
      if (residual) {
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) x[e] += res[e];
      }
      if (f32) {
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) { if (inside(e)) *at(reinterpret_cast<float*>(p.c), e) = x[e]; }
      } else {
#pragma unroll
        for (int e = 0; e < AT_ONCE; ++e) { if (inside(e)) *at(reinterpret_cast<bf16_t*>(p.c), e) = f2bf(x[e]); }
      }
    }
    lanes_in_order();
  }
}

// An epilogue that is not one of the common ones: ragged columns, two of GELU, GELU', a residual and fp32, rows so far apart that
// 32-bit offsets do not reach over the 128 of a wavefront.  They have kernels of their own.  (With all variants in one kernel the
// main loops beside the common ones came out slower: six layers of d 2048 16.6 -> 17.4 ms a step, a batch of 4096 tokens through
// twelve of d 768 1.55 -> 1.62.  Plain fp32 among the rare ones, decided element by element, made 8192 x 768 x 50304 in eight slices
// of K 6 % slower.)  A launch over several products that has both takes one with all of them.
__host__ __device__ __forceinline__ bool gemm_rare(uint32_t epilogue, uint32_t n, uint32_t ldc) {
  const uint32_t what = epilogue & (SIF_EPI_GELU | SIF_EPI_GELU_GRAD | SIF_EPI_RESIDUAL | SIF_EPI_OUT_F32);
  return (n & 7) != 0 || ldc > (1u << 21) || (what & (what - 1)) != 0;
}
enum { kEpiCommon, kEpiRare, kEpiAll };
// bias_s: the bias of the columns nw.. in LDS (gemm_fetch_bias)
template <int TI, int TJ, int EPI, int ROOM>
__device__ __forceinline__ void gemm_store_tile(const GemmP& p, floatx4 (&acc)[2 * TI][2 * TJ], float* sW, uint32_t mw, uint32_t nw, size_t c_off, uint32_t lane,
                                                const bf16_t* bias_s) {
  if constexpr (EPI != kEpiCommon) {
    if (EPI == kEpiRare || gemm_rare(p.epi, p.n, p.ldc)) {
      if ((p.n & 7) != 0) gemm_store_single<TI, TJ>(p, acc, sW, mw, nw, c_off, lane);
      else if (p.epi & SIF_EPI_OUT_F32) gemm_store_f32_mixed<TI, TJ>(p, acc, sW, mw, nw, c_off, lane, bias_s);
      else gemm_store_mixed<TI, TJ>(p, acc, sW, mw, nw, c_off, lane, bias_s);
      return;
    }
  }
  if constexpr (EPI != kEpiRare) {
    if (p.epi & SIF_EPI_RESIDUAL) gemm_store_rows<TI, TJ, kRowsResidual, ROOM>(p, acc, sW, mw, nw, c_off, lane, bias_s);
    else if (p.epi & SIF_EPI_GELU_GRAD) gemm_store_rows<TI, TJ, kRowsGeluGrad, ROOM>(p, acc, sW, mw, nw, c_off, lane, bias_s);
    else if (p.epi & SIF_EPI_OUT_F32) gemm_store_f32<TI, TJ>(p, acc, sW, mw, nw, c_off, lane, bias_s);
    else if (!(p.epi & SIF_EPI_GELU)) gemm_store_packed<TI, TJ, false>(p, acc, sW, mw, nw, c_off, lane, bias_s);
    else if (p.aux == nullptr) gemm_store_packed<TI, TJ, true>(p, acc, sW, mw, nw, c_off, lane, bias_s);
    else gemm_store_rows<TI, TJ, kRowsGeluAux, ROOM>(p, acc, sW, mw, nw, c_off, lane, bias_s);
  }
}

// The bias of a wavefront's columns nw.. into 1 KB of LDS of its own, by one fetch (which writes zeros behind them)
__device__ __forceinline__ void gemm_fetch_bias(const GemmP& p, uint32_t nw, uint32_t width, uint32_t lane, uint32_t lds) {
  if (p.bias != nullptr && (p.n & 7) == 0) fetch16(operand_rsrc((uint64_t)(p.bias + nw)), lane * 8 < width && nw + lane * 8 < p.n ? lane * 16 : kOutside, lds);
}

// ---------------------------------------------------------------------------------------------- tiles
template <int V> struct Int { static constexpr int value = V; };

template <int I, int J>
__device__ __forceinline__ void gemm_clear(floatx4 (&acc)[I][J]) {
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int j = 0; j < J; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
}

// Block -> tile.  Consecutive workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2.  Every XCD
// gets a contiguous run of tiles (tile number pid belongs to XCD pid % 8 and is the (pid / 8)-th of its run), and each
// run is walked in bands of 8 tile rows, so that the tiles an XCD works on at one time share their A and B panels in
// that XCD's L2.
__device__ __forceinline__ void gemm_tile_of(const GemmP& p, uint32_t total_tiles, uint32_t pid, uint32_t& tm, uint32_t& tn) {
  const uint32_t per = (total_tiles + 7) / 8, tall = (total_tiles % 8) ? (total_tiles % 8) : 8, xcd = pid % 8, local = pid / 8;
  const uint32_t logical = xcd < tall ? xcd * per + local : tall * per + (xcd - tall) * (per - 1) + local;
  const uint32_t width = 8 * p.tiles_n, group = logical / width, first = group * 8;
  const uint32_t gsz = min(p.tiles_m - first, 8u), in = logical % width;
  tm = first + in % gsz;
  tn = in / gsz;
}
__device__ __forceinline__ uint32_t gemm_tiles_of_xcd(uint32_t total_tiles, uint32_t x) { return x < total_tiles ? (total_tiles - x + 7u) / 8u : 0u; }
// One thread: takes a tile from the per-XCD counters of the stream's record, own XCD first: a tile number, else kNone.
__device__ __forceinline__ uint32_t gemm_steal_tile(StreamRec* rec, uint32_t total_tiles, uint32_t my_x) {
  for (uint32_t r = 0; r < 8; ++r) {
    const uint32_t x = (my_x + r) & 7u, cnt = gemm_tiles_of_xcd(total_tiles, x);
    uint32_t* ctr = &rec->tile_next[x * 32u];
    if (ld_relaxed(ctr) >= cnt) continue;
    const uint32_t l = atomicAdd(ctr, 1u);
    if (l < cnt) return l * 8u + x;
  }
  return kNone;
}

// A product's record where it lies in memory that no kernel writes: the launch's own arguments, or its entry in the list of a
// launch over several.  Read through the scalar cache where it is needed; the pointer is made opaque so that the words are
// read again instead of being kept in (or spilled from) scalar registers through a main loop.
typedef __attribute__((address_space(4))) const GemmP* gemm_record_ptr;
__device__ __forceinline__ gemm_record_ptr gemm_record_of_launch() { return (gemm_record_ptr)__builtin_amdgcn_kernarg_segment_ptr(); }
// (of a launch over several: the entry that block `pid` works on)
__device__ __forceinline__ gemm_record_ptr gemm_record_of_block(gemm_record_ptr group, uint32_t group_n, uint32_t pid) {
  uint32_t g = 0;
  while (g + 1 < group_n && pid >= group[g + 1].tile_base) ++g;
  return group + g;
}
__device__ __forceinline__ GemmP gemm_read_record(gemm_record_ptr p) {
  asm volatile("" : "+s"(p));
  static_assert(sizeof(GemmP) % 4 == 0, "copied as 32-bit words");
  typedef __attribute__((address_space(4))) const uint32_t* word_ptr;
  uint32_t words[sizeof(GemmP) / 4];
#pragma unroll
  for (uint32_t w = 0; w < sizeof(GemmP) / 4; ++w) words[w] = ((word_ptr)p)[w];
  GemmP q;
  __builtin_memcpy(&q, words, sizeof(GemmP));
  return q;
}

// One tile per block.  A ring of ST K steps in LDS; a wavefront keeps the fragments of two steps in registers, so that
// those of step t+1 are read, slice by slice, between the MFMAs of step t.  The steady part is a body of whole turns of
// the ring (every LDS address a constant); what is left - the last ST and a few steps, a ragged last step among them -
// runs through the same step with the ring's position and its conditions worked out.
//   LAG = 0: step t's slot is fetched into again in step t, once all wavefronts have their fragments of t in registers
//            (they wait for these before the barrier): ST steps in flight.
//   LAG = 1: one step later; nothing is waited for before the barrier but the fetches of step t+1: ST - 1 in flight.
// Registers: at most 248 of the 256 that two wavefronts of a SIMD may take (the attribute counts in pairs), so that a
// one-wavefront kernel that sits on a CU for the length of a bubble (the training stream's wait) fits beside a block of the
// 256x128 tiles, which otherwise stays off that CU until it ends.
template <int ALAY, int BLAY, int BM, int BN, int WM, int WN, int ST, int LAG, int OCC, int EPI, bool GROUPED = false>
__global__ __launch_bounds__(64 * WM * WN, OCC) __attribute__((amdgpu_num_vgpr(124))) void gemm_ring_kernel(GemmP p_in, KCtl ctl) {
  // (a launch over several products has an instantiation of its own: in the others the product's record stays the
  // kernel argument, in scalar registers)
  GemmP p = p_in;
  constexpr int THREADS = 64 * WM * WN, TI = BM / (WM * 32), TJ = BN / (WN * 32), AHEAD = LAG ? ST - 1 : ST;
  constexpr uint32_t SA = BM * BK, SB = BN * BK, STAGE = SA + SB;      // elements
  typedef TileFetch<ALAY, BM, THREADS, BM, BM, 0> FetchA;
  typedef TileFetch<BLAY, BN, THREADS, BN, BN, 0> FetchB;
  constexpr int FA = FetchA::NV, F = FA + FetchB::NV;                  // fetches per thread and K step
  constexpr int ROOM = gemm_room(ST * STAGE * 2, WM * WN);            // the epilogue is staged in the ring
  static_assert(F * (AHEAD - 1) < 64, "the wait counts 63 operations");
  __shared__ __align__(1024) bf16_t lds[ST * STAGE];
  __shared__ __align__(1024) bf16_t s_bias[WM * WN * 512];
  if (!kernel_begin(ctl)) { kernel_end(ctl, false); return; }
  if constexpr (GROUPED) p = gemm_read_record(gemm_record_of_block((gemm_record_ptr)p_in.group, p_in.group_n, blockIdx.x));

  const uint32_t total_tiles = p.tiles_m * p.tiles_n, pid = blockIdx.x - p.tile_base;
  const uint32_t bo = blockIdx.z / p.batch_inner, bi = blockIdx.z % p.batch_inner;
  uint32_t tile_m = 0, tile_n = 0;
  if (pid < total_tiles) gemm_tile_of(p, total_tiles, pid, tile_m, tile_n);
  const uint32_t m0 = tile_m * BM, n0 = tile_n * BN;
  // (blocks of a group beyond their product's tiles have nothing to do, and of a causal product those whose 128x128 tile
  // lies above the diagonal)
  if (pid >= total_tiles || ((p.epi & SIF_EPI_CAUSAL_SKIP) && n0 / 128 > (m0 + BM - 1) / 128)) { kernel_end(ctl, true); return; }

  uint32_t k_begin = 0, k_end = p.k;
  if (p.k_limit != 0) k_end = min(p.k, p.k_limit - bi * p.k);      // slices of one long K: the last may be shorter
  if (p.k_causal == 1) k_end = min(p.k, m0 + BM);
  if (p.k_causal == 2) k_begin = (m0 / BK) * BK;
  const uint32_t nt = (k_end - k_begin + BK - 1) / BK, full = (k_end - k_begin) / BK, k_rest = (k_end - k_begin) % BK;

  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave / WN, wn = wave % WN;
  floatx4 acc[2 * TI][2 * TJ];
  gemm_clear(acc);
  const size_t c_off = (size_t)(bo * p.c_so + bi * p.c_si);
  FetchA ta;
  FetchB tb;
  ta.init(p.lda, p.m - m0, threadIdx.x);
  tb.init(p.ldb, p.n - n0, threadIdx.x);
  const bf16_t* A = p.a + bo * p.a_so + bi * p.a_si;
  const bf16_t* B = p.b + bo * p.b_so + bi * p.b_si;
  uint64_t base_a = (uint64_t)(ALAY == 0 ? A + (size_t)m0 * p.lda + k_begin : A + (size_t)k_begin * p.lda + m0);
  uint64_t base_b = (uint64_t)(BLAY == 0 ? B + (size_t)n0 * p.ldb + k_begin : B + (size_t)k_begin * p.ldb + n0);
  const uint64_t step_a = ALAY == 0 ? BK * 2 : (uint64_t)BK * p.lda * 2, step_b = BLAY == 0 ? BK * 2 : (uint64_t)BK * p.ldb * 2;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)lds;

  bf16x8 fa[2][2][2 * TI], fb[2][2][2 * TJ];
  RingFrags<ALAY, BM, 2 * TI, ST> ra_frags;
  RingFrags<BLAY, BN, 2 * TJ, ST> rb_frags;
  ra_frags.init(lds0, wm * (TI * 32));
  rb_frags.init(lds0 + ST * SA * 2, wn * (TJ * 32));
  // a step in four quarters: two slices of 32 k, half of the operands to read and of the MFMAs each
  auto read_quarter = [&](auto SLOT, int h, bf16x8 (&a)[2 * TI], bf16x8 (&b)[2 * TJ]) {
#pragma unroll
    for (int i = (h & 1) * TI; i < (h & 1) * TI + TI; ++i) a[i] = ra_frags.template read_slot<decltype(SLOT)::value>(i, h >> 1);
#pragma unroll
    for (int j = (h & 1) * TJ; j < (h & 1) * TJ + TJ; ++j) b[j] = rb_frags.template read_slot<decltype(SLOT)::value>(j, h >> 1);
  };
  auto mfma_quarter = [&](int h, bf16x8 (&a)[2 * TI], bf16x8 (&b)[2 * TJ]) {
#pragma unroll
    for (int i = (h & 1) * TI; i < (h & 1) * TI + TI; ++i)
#pragma unroll
      for (int j = 0; j < 2 * TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
  };
  // the next K step into a slot; `last`: the ragged one
  auto fetch_step = [&](uint32_t slot, bool last) {
    const uint32_t oa = lds0 + slot * (SA * 2), ob = lds0 + ST * (SA * 2) + slot * (SB * 2);
    const i32x4 ra = operand_rsrc(base_a), rb = operand_rsrc(base_b);
    if (last) {
#pragma unroll
      for (int d = 0; d < F; ++d) { if (d < FA) ta.issue_last(ra, oa, wave, d, k_rest, threadIdx.x); else tb.issue_last(rb, ob, wave, d - FA, k_rest, threadIdx.x); }
    } else {
#pragma unroll
      for (int d = 0; d < F; ++d) { if (d < FA) ta.issue(ra, oa, wave, d); else tb.issue(rb, ob, wave, d - FA); }
    }
    base_a += step_a; base_b += step_b;
  };
  gemm_fetch_bias(p, n0 + wn * (TJ * 32), TJ * 32, lane, (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)s_bias + wave * 1024);
  for (uint32_t s = 0; s < (uint32_t)AHEAD && s < nt; ++s) fetch_step(s, s >= full);
  if (nt >= (uint32_t)AHEAD) wait_vm<F * (AHEAD - 1)>(); else wait_vm<0>();
  barrier_only();
#pragma unroll
  for (int h = 0; h < 4; ++h) read_quarter(Int<0>(), h, fa[0][h >> 1], fb[0][h >> 1]);

  auto steady = [&](auto S, auto P) {          // step in slot S with its fragments in register set P
    constexpr int s = decltype(S)::value, cur = decltype(P)::value, nx = (s + 1) % ST, fs = (s + AHEAD) % ST;
    wait_vm<F * (AHEAD - 2)>();                 // the next step has landed
    if (!LAG) wait_lds();
    barrier_only();
    const uint32_t oa = lds0 + fs * (SA * 2), ob = lds0 + ST * (SA * 2) + fs * (SB * 2);
    const i32x4 ra = operand_rsrc(base_a), rb = operand_rsrc(base_b);
    base_a += step_a; base_b += step_b;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      read_quarter(Int<nx>(), h, fa[cur ^ 1][h >> 1], fb[cur ^ 1][h >> 1]);
#pragma unroll
      for (int d = h * F / 4; d < (h + 1) * F / 4; ++d) { if (d < FA) ta.issue(ra, oa, wave, d); else tb.issue(rb, ob, wave, d - FA); }
      __builtin_amdgcn_sched_barrier(0);
      mfma_quarter(h, fa[cur][h >> 1], fb[cur][h >> 1]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  uint32_t t = 0;
  constexpr uint32_t TURN = ST == 3 ? 6 : ST;      // an even number of steps: the register sets alternate too
  static_assert(ST >= 2 && ST <= 4, "the turns written out below");
  while (t + AHEAD + TURN - 1 < full) {
    if constexpr (ST == 2) { steady(Int<0>(), Int<0>()); steady(Int<1>(), Int<1>()); }
    if constexpr (ST == 3) {
      steady(Int<0>(), Int<0>()); steady(Int<1>(), Int<1>()); steady(Int<2>(), Int<0>());
      steady(Int<0>(), Int<1>()); steady(Int<1>(), Int<0>()); steady(Int<2>(), Int<1>());
    }
    if constexpr (ST == 4) { steady(Int<0>(), Int<0>()); steady(Int<1>(), Int<1>()); steady(Int<2>(), Int<0>()); steady(Int<3>(), Int<1>()); }
    t += TURN;
  }
  uint32_t slot = 0;
  auto step = [&](auto P) {                    // (where no step follows, what is read is not used: see the kernel below)
    constexpr int cur = decltype(P)::value;
    const uint32_t nx = slot + 1 == ST ? 0 : slot + 1;
    if (t + 1 < nt) {
      if (t + AHEAD - 1 < nt) wait_vm<F * (AHEAD - 2)>(); else wait_vm<0>();
      if (!LAG) wait_lds();
      barrier_only();
    }
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
      for (int i = 0; i < 2 * TI; ++i) fa[cur ^ 1][ks][i] = ra_frags.read(0, nx * (SA * 2), i, ks);
#pragma unroll
      for (int j = 0; j < 2 * TJ; ++j) fb[cur ^ 1][ks][j] = rb_frags.read(0, nx * (SB * 2), j, ks);
      if (ks == 0 && t + AHEAD < nt) fetch_step(LAG ? (slot == 0 ? ST - 1 : slot - 1) : slot, t + AHEAD >= full);
      __builtin_amdgcn_sched_barrier(0);
      mfma_quarter(2 * ks, fa[cur][ks], fb[cur][ks]);
      mfma_quarter(2 * ks + 1, fa[cur][ks], fb[cur][ks]);
      __builtin_amdgcn_sched_barrier(0);
    }
    slot = nx;
    ++t;
  };
  while (t + 1 < nt) { step(Int<0>()); step(Int<1>()); }
  if (t < nt) step(Int<0>());

  __syncthreads();                             // nobody reads the ring any more: it stages the results
  const Arrival arrival = kernel_arrive(ctl, !GROUPED && !(p.epi & SIF_EPI_CAUSAL_SKIP));
  gemm_store_tile<TI, TJ, EPI, ROOM>(p, acc, reinterpret_cast<float*>(lds) + wave * (ROOM * kStage / 4), m0 + wm * (TI * 32), n0 + wn * (TJ * 32), c_off, lane, s_bias + wave * 512);
  kernel_finish(ctl, arrival);
}

// Tiles of a launch with at most one per CU, with wavefronts that only fetch.  A fetch of 1 KB holds its wavefront for some 70
// cycles (a wavefront by itself takes in 33 bytes/ns, two 70, four 120 to 155), and in the ring above it stands in front of the
// same wavefront's MFMAs: with 8 to 24 KB per 64 k and few MFMAs to them that was what a step waited for.  Here FW wavefronts
// fetch and wait for what has landed, the other WM x WN read fragments and multiply; a barrier per step, of KB times 64 k,
// keeps them together (with one per 64 k the smallest tiles spend more than half of a step in it).  Weights as they come from
// twelve layers' 170 MB, launches back to back: 77 x 768 x 3072 13.0 -> 8.1 us, 77 x 768 x 768 5.8 -> 4.8, 512 x 768 x 3072
// 13.3 -> 10.0, 1100 x 768 x 3072 15.2 -> 12.7, 2008 x 768 x 3072 22.1 -> 20.5.  With several tiles on a CU these hide each
// other's fetches and the ring above is as fast.  (So it is with 128x128 tiles, one per
// CU or fewer: eight wavefronts' MFMAs cover the fetches, and with four more that fetch it took 0.96 to 1.04 of the time.)
//   Apart: one request of 77 tokens through twelve layers takes 860 us on the ring, 761 with these wavefronts, 32x64 tiles and a
// barrier per 64 k, 723 with one per 128 k, 662 with 32x32 tiles; 77 x 768 x 3072 17.0, 12.2, 11.4, 8.7.  Their 97 to 148 KB of LDS
// leave less room for another stream's blocks than the ring's 50 to 70; beside training that costs nothing (online requests p95 5.4
// ms on either, the training step +2.4 % and on the ring +3.2 %).
//   ST - 1 steps are in flight: the slot of the step before the current one is free for fetches when all wavefronts have
// passed the barrier in front of the current one's products, which used that step's fragments before it.
template <int I, int N, typename F>
__device__ __forceinline__ void gemm_unrolled(F&& f) {
  if constexpr (I < N) { f(Int<I>()); gemm_unrolled<I + 1, N>(f); }
}
// (each behind the one before it and nothing else, so that the compiler knows which of its reads are on their way)
template <int I, int N, typename F>
__device__ __forceinline__ void gemm_while(uint32_t n, F&& f) {
  if constexpr (I < N) {
    if (n > (uint32_t)I) { f(Int<I>()); gemm_while<I + 1, N>(n, f); }
  }
}
// waits until at most `steps` steps of F fetches, of no more than MOST, are outstanding
template <int F, int MOST>
__device__ __forceinline__ void gemm_wait_steps(uint32_t steps) {
  if constexpr (MOST == 0) { wait_vm<0>(); }
  else { if (steps >= (uint32_t)MOST) wait_vm<F * MOST>(); else gemm_wait_steps<F, MOST - 1>(steps); }
}
template <int ALAY, int BLAY, int BM, int BN, int WM, int WN, int FW, int ST, int KB, int EPI>
__global__ __launch_bounds__(64 * (WM * WN + FW), 2) void gemm_fed_kernel(GemmP p, KCtl ctl) {
  constexpr int MW = WM * WN, FT = 64 * FW, TI = BM / (WM * 32), TJ = BN / (WN * 32), AHEAD = ST - 1;
  constexpr uint32_t SA = BM * BK, SB = BN * BK, STAGE = SA + SB;      // elements of 64 k
  typedef TileFetch<ALAY, BM, FT, BM, BM, 0> FetchA;
  typedef TileFetch<BLAY, BN, FT, BN, BN, 0> FetchB;
  constexpr int FA = FetchA::NV, F1 = FA + FetchB::NV, F = F1 * KB;    // fetches per thread: of 64 k, of a step
  constexpr int ROOM = gemm_room(ST * KB * STAGE * 2, MW);             // the epilogue is staged in the ring
  static_assert(F * AHEAD < 64, "the waits count 63 operations");
  static_assert(ST % 2 == 0, "the register sets alternate with the slots");
  __shared__ __align__(1024) bf16_t lds[ST * KB * STAGE];
  __shared__ __align__(1024) bf16_t s_bias[MW * 512];
  if (!kernel_begin(ctl)) { kernel_end(ctl, false); return; }

  const uint32_t bo = blockIdx.z / p.batch_inner, bi = blockIdx.z % p.batch_inner;
  uint32_t tile_m, tile_n;
  gemm_tile_of(p, p.tiles_m * p.tiles_n, blockIdx.x, tile_m, tile_n);
  const uint32_t m0 = tile_m * BM, n0 = tile_n * BN;
  if ((p.epi & SIF_EPI_CAUSAL_SKIP) && n0 / 128 > (m0 + BM - 1) / 128) { kernel_end(ctl, true); return; }      // (as in the ring)
  uint32_t k_begin = 0, k_end = p.k;
  if (p.k_limit != 0) k_end = min(p.k, p.k_limit - bi * p.k);
  if (p.k_causal == 1) k_end = min(p.k, m0 + BM);
  if (p.k_causal == 2) k_begin = (m0 / BK) * BK;
  const uint32_t nt = (k_end - k_begin + BK * KB - 1) / (BK * KB), full = (k_end - k_begin) / BK, k_rest = (k_end - k_begin) % BK;
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)lds;
  Arrival arrival = {Arrival::kNotCounted, 0};

  if (wave >= MW) {
    const uint32_t tid = threadIdx.x - MW * 64, fw = wave - MW;
    FetchA ta;
    FetchB tb;
    ta.init(p.lda, p.m - m0, tid);
    tb.init(p.ldb, p.n - n0, tid);
    const bf16_t* A = p.a + bo * p.a_so + bi * p.a_si;
    const bf16_t* B = p.b + bo * p.b_so + bi * p.b_si;
    uint64_t base_a = (uint64_t)(ALAY == 0 ? A + (size_t)m0 * p.lda + k_begin : A + (size_t)k_begin * p.lda + m0);
    uint64_t base_b = (uint64_t)(BLAY == 0 ? B + (size_t)n0 * p.ldb + k_begin : B + (size_t)k_begin * p.ldb + n0);
    const uint64_t step_a = ALAY == 0 ? BK * 2 : (uint64_t)BK * p.lda * 2, step_b = BLAY == 0 ? BK * 2 : (uint64_t)BK * p.ldb * 2;
    uint32_t slot = 0;                         // of the next step to be fetched
    auto fetch_step = [&](uint32_t step) {
#pragma unroll
      for (int u = 0; u < KB; ++u) {
        const uint32_t oa = lds0 + (slot * KB + u) * (SA * 2), ob = lds0 + ST * KB * (SA * 2) + (slot * KB + u) * (SB * 2), at = step * KB + u;
        const i32x4 ra = operand_rsrc(base_a), rb = operand_rsrc(base_b);
        if (at >= full) {                      // the ragged end of K, and zeros for what a step has beyond it
          const uint32_t left = at == full ? k_rest : 0;
#pragma unroll
          for (int d = 0; d < F1; ++d) { if (d < FA) ta.issue_last(ra, oa, fw, d, left, tid); else tb.issue_last(rb, ob, fw, d - FA, left, tid); }
        } else {
#pragma unroll
          for (int d = 0; d < F1; ++d) { if (d < FA) ta.issue(ra, oa, fw, d); else tb.issue(rb, ob, fw, d - FA); }
        }
        base_a += step_a; base_b += step_b;
      }
      slot = slot + 1 == ST ? 0 : slot + 1;
    };
    uint32_t s = 0;                            // steps asked for
    for (; s < (uint32_t)AHEAD && s < nt; ++s) fetch_step(s);
    gemm_wait_steps<F, AHEAD - 1>(s - 1);
    barrier_only();
    for (uint32_t t = 1; t < nt; ++t) {        // step t has landed: it is read behind the barrier
      gemm_wait_steps<F, AHEAD - 2>(s - t - 1);
      barrier_only();
      if (s < nt) { fetch_step(s); ++s; }
    }
    __syncthreads();
    // the tile is counted by a wavefront that has nothing else left to do (block 0 behind the wait for the bias in its others)
    arrival = kernel_arrive(ctl, !(p.epi & SIF_EPI_CAUSAL_SKIP), tid == 0);
    kernel_answer(ctl, arrival, tid == 0);
  } else {
    const uint32_t wm = wave / WN, wn = wave % WN;
    floatx4 acc[2 * TI][2 * TJ];
    gemm_clear(acc);
    bf16x8 fa[2][2 * KB][2 * TI], fb[2][2 * KB][2 * TJ];
    RingFrags<ALAY, BM, 2 * TI, ST * KB> ra_frags;
    RingFrags<BLAY, BN, 2 * TJ, ST * KB> rb_frags;
    ra_frags.init(lds0, wm * (TI * 32));
    rb_frags.init(lds0 + ST * KB * SA * 2, wn * (TJ * 32));
    auto read_slice = [&](int slot, int ks, bf16x8 (&a)[2 * TI], bf16x8 (&b)[2 * TJ]) {
#pragma unroll
      for (int i = 0; i < 2 * TI; ++i) a[i] = ra_frags.read_tile(slot * KB + ks / 2, i, ks % 2);
#pragma unroll
      for (int j = 0; j < 2 * TJ; ++j) b[j] = rb_frags.read_tile(slot * KB + ks / 2, j, ks % 2);
    };
    gemm_fetch_bias(p, n0 + wn * (TJ * 32), TJ * 32, lane, (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)s_bias + wave * 1024);
    barrier_only();
#pragma unroll
    for (int ks = 0; ks < 2 * KB; ++ks) read_slice(0, ks, fa[0][ks], fb[0][ks]);
    // the step in slot S, its fragments in register set S % 2; more: another one follows (where none does, what is read is not
    // used: behind a branch around the reads the compiler would wait for all of them in front of the MFMAs)
    auto step = [&](auto S, bool more) {
      constexpr int s = decltype(S)::value, cur = s & 1, nx = (s + 1) % ST;
      if (more) barrier_only();
#pragma unroll
      for (int ks = 0; ks < 2 * KB; ++ks) {
        read_slice(nx, ks, fa[cur ^ 1][ks], fb[cur ^ 1][ks]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2 * TI; ++i)
#pragma unroll
          for (int j = 0; j < 2 * TJ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[cur][ks][i], fb[cur][ks][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    uint32_t t = 0;
#pragma clang loop unroll(disable)
    for (; t + ST < nt; t += ST) gemm_unrolled<0, ST>([&](auto S) { step(S, true); });
    gemm_while<0, ST>(nt - t, [&](auto S) { step(S, t + decltype(S)::value + 1 < nt); });
    wait_vm<0>();                              // the bias
    __syncthreads();                           // nobody reads the ring any more: it stages the results
    gemm_store_tile<TI, TJ, EPI, ROOM>(p, acc, reinterpret_cast<float*>(lds) + wave * (ROOM * kStage / 4), m0 + wm * (TI * 32), n0 + wn * (TJ * 32),
                                (size_t)(bo * p.c_so + bi * p.c_si), lane, s_bias + wave * 512);
  }
  kernel_finish(ctl, arrival, threadIdx.x == MW * 64);
}

// 256x256 tiles, eight wavefronts of 128x64, whole K steps.  The wavefronts of the tile's upper and of its lower half -
// one of each per SIMD - take turns: while one half multiplies (32 MFMAs, nothing else in its instruction stream), the
// other reads the fragments of its next 32 from LDS and issues fetches, then a barrier swaps them.  Per K step a
// wavefront has two memory phases: B (kept in registers for both) with the first half of its A rows, then the second
// half of its A rows.  The parts of a step are therefore read, and free for the fetch of two steps later, at different
// times: the first halves of A and half of B are fetched in one phase, the rest of B and the second halves of A in the next, and
// every fetch has four to six phases (1 to 1.5 us) to arrive; the counts waited for leave six to eight younger fetches per
// wavefront in flight.  (All of B with the first halves of A: six fetches in that phase and two in the other, and a phase is as
// long as its memory half: 8192^3 719 us, now 705, with both operands k-major 778 and 737; on zeros, which leave the clock at its
// limit, 549 and 516.)  Two buffers of each part are 128 KB of LDS; the epilogue has 16 KB of its own for staging.
// (One phase is 512 cycles of MFMA.  With a few tiles on the chip a step takes 0.96 us where it was 1.18 with a barrier per
// step and everything in one stream; with a tile on every CU the clock falls to what the power allows: 1.47 us against
// 1.51, 8192^3 795 -> 767 us.)
//
// Persistent: a block works through tiles one after the other; the first operand tiles of the next output tile are
// fetched while the current one's epilogue runs.  Which tile comes next: a monitored launch hands its tiles out through
// counters in the stream's record, one per XCD (a block takes the tiles of its own XCD's run in order and, when that
// run is exhausted, helps the others), so that a block that starts late - its CU was held by a kernel of the other
// stream - simply takes fewer tiles; with a fixed share per block the whole launch would wait for the late one.  An
// unmonitored launch has no record: every block takes each gridDim.x-th tile (a stride that is a multiple of 8 keeps it
// on its XCD's run).
// Registers: held to 248 for the same reason as the ring kernel.
template <int ALAY, int BLAY, int EPI, bool GROUPED = false>
__global__ __launch_bounds__(512, 1) __attribute__((amdgpu_num_vgpr(124))) void gemm_pp_kernel(GemmP p_in, KCtl ctl) {
  constexpr int BM = 256, BN = 256, WM = 2, WN = 4, THREADS = 512, TI = 4, TJ = 2, HI = TI;      // HI: 16-row operands of a half of A
  constexpr uint32_t HA = BM / 2 * BK, STAGE = 2 * HA + BN * BK;       // elements: two halves of A, then B
  typedef TileFetch<ALAY, BM / 2, THREADS, BM / WM / 2, BM / WM, 0> FetchA0;
  typedef TileFetch<ALAY, BM / 2, THREADS, BM / WM / 2, BM / WM, 1> FetchA1;
  typedef TileFetch<BLAY, BN, THREADS, BN, BN, 0> FetchB;
  constexpr int FA = FetchA0::NV, FB = FetchB::NV / 2;                 // fetches of a half of A; of a half of B
  static_assert(FetchA1::NV == FA, "two equal halves");
  __shared__ __align__(1024) bf16_t lds[2 * STAGE];
  __shared__ __align__(16) float stage[WM * WN * (kStage / 4)];
  __shared__ __align__(1024) bf16_t s_bias[WM * WN * 512];
  __shared__ uint32_t s_next;
  if (!kernel_begin(ctl)) { kernel_end(ctl, false); return; }
  gemm_record_ptr fetched = gemm_record_of_launch();       // the product whose operands are fetched
  // (the record of a group's launch says how many blocks' worth of tiles it has in all)
  const uint32_t all_tiles = GROUPED ? p_in.tiles_m : p_in.tiles_m * p_in.tiles_n;
  const uint32_t bo = blockIdx.z / p_in.batch_inner, bi = blockIdx.z % p_in.batch_inner;
  const bool dynamic = ctl.rec != nullptr && gridDim.z == 1 && gridDim.x < all_tiles;
  const uint32_t my_x = blockIdx.x & 7u;
  uint32_t pid = blockIdx.x;
  if (dynamic) {
    if (threadIdx.x == 0) s_next = gemm_steal_tile(ctl.rec, all_tiles, my_x);
    __syncthreads();
    pid = s_next;
  }
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wm = wave / WN, wn = wave % WN;
  const bool second = wm != 0;                 // the half that is one phase behind
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)lds;

  FetchA0 ta0;
  FetchA1 ta1;
  FetchB tb;
  uint64_t base_a = 0, base_b = 0, step_a = 0, step_b = 0;
  uint32_t m0 = 0, n0 = 0, nt = 0;
  // of step t, whose operands begin at base_a and base_b
  auto fetch_a0 = [&](uint32_t t) {
    const i32x4 r = operand_rsrc(base_a);
#pragma unroll
    for (int i = 0; i < FA; ++i) ta0.issue(r, lds0 + (t & 1u) * (STAGE * 2), wave, i);
  };
  auto fetch_a1 = [&](uint32_t t) {
    const i32x4 r = operand_rsrc(base_a);
#pragma unroll
    for (int i = 0; i < FA; ++i) ta1.issue(r, lds0 + (t & 1u) * (STAGE * 2) + HA * 2, wave, i);
  };
  auto fetch_b = [&](uint32_t t, auto PART) {
    const i32x4 r = operand_rsrc(base_b);
#pragma unroll
    for (int i = decltype(PART)::value * FB; i < (decltype(PART)::value + 1) * FB; ++i) tb.issue(r, lds0 + (t & 1u) * (STAGE * 2) + HA * 4, wave, i);
  };
  // sets up tile `id` and fetches what its first two memory phases read, and one part more
  auto open_tile = [&](uint32_t id) {
    uint32_t local = id, tile_m, tile_n, tid = threadIdx.x;
    asm volatile("" : "+v"(tid));              // (what follows from it is worked out here, not kept in registers through the main loop)
    if constexpr (GROUPED) fetched = gemm_record_of_block((gemm_record_ptr)p_in.group, p_in.group_n, id);
    const GemmP p = gemm_read_record(fetched);
    if constexpr (GROUPED) {
      local = id - p.tile_base;
      // (a group pads every product to a multiple of eight tiles: what is beyond has no K steps and stores nothing)
      if (local >= p.tiles_m * p.tiles_n) { nt = 0; return; }
    }
    gemm_tile_of(p, p.tiles_m * p.tiles_n, local, tile_m, tile_n);
    m0 = tile_m * BM;
    n0 = tile_n * BN;
    uint32_t k_end = p.k;
    if (p.k_limit != 0) k_end = min(p.k, p.k_limit - bi * p.k);      // slices of one long K: the last may be shorter
    nt = k_end / BK;
    ta0.init(p.lda, p.m - m0, tid);
    ta1.init(p.lda, p.m - m0, tid);
    tb.init(p.ldb, p.n - n0, tid);
    const bf16_t* A = p.a + bo * p.a_so + bi * p.a_si;
    const bf16_t* B = p.b + bo * p.b_so + bi * p.b_si;
    base_a = (uint64_t)(ALAY == 0 ? A + (size_t)m0 * p.lda : A + m0);
    base_b = (uint64_t)(BLAY == 0 ? B + (size_t)n0 * p.ldb : B + n0);
    step_a = ALAY == 0 ? BK * 2 : (uint64_t)BK * p.lda * 2;
    step_b = BLAY == 0 ? BK * 2 : (uint64_t)BK * p.ldb * 2;
    fetch_a0(0);
    fetch_b(0, Int<0>());
    fetch_b(0, Int<1>());
    fetch_a1(0);
    base_a += step_a; base_b += step_b;
    if (nt > 1) { fetch_a0(1); fetch_b(1, Int<0>()); }
  };
  Arrival arrival = {Arrival::kNotCounted, 0};
  if (pid < all_tiles) open_tile(pid);
  while (pid < all_tiles) {
    const uint32_t cm0 = m0, cn0 = n0, cnt = nt;
    const gemm_record_ptr current = fetched;   // (of a group: the next tile may belong to another product)
    floatx4 acc[2 * TI][2 * TJ];
    gemm_clear(acc);
    bf16x8 fa[2][HI], fb[2][2 * TJ];
    auto read_a = [&](const bf16_t* half) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int i = 0; i < HI; ++i) fa[ks][i] = operand_frag<ALAY, BM / 2>(half, (wm * HI + i) * 16, ks);
    };
    auto read_b = [&](const bf16_t* tile) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int j = 0; j < 2 * TJ; ++j) fb[ks][j] = operand_frag<BLAY, BN>(tile, (wn * 2 * TJ + j) * 16, ks);
    };
    auto multiply = [&](auto H) {
      constexpr int h = decltype(H)::value;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int e = 0; e < HI * 2 * TJ; ++e) {      // (blocks of 2 x 2: 0.5 % faster than row by row)
          const int i = e / (4 * TJ) * 2 + (e >> 1 & 1), j = e / 4 % TJ * 2 + (e & 1);
          acc[h * HI + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[ks][i], fb[ks][j], acc[h * HI + i][j], 0, 0, 0);
        }
      __builtin_amdgcn_sched_barrier(0);
    };
    if (nt > 1) wait_vm<2 * FA + FB>(); else wait_vm<FA>();      // B and the first halves of A of step 0
    barrier_only();
    gemm_fetch_bias(gemm_read_record(current), cn0 + wn * 64, 64, lane, (uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t*)s_bias + wave * 1024);
    uint32_t own = 0;
    if (dynamic && threadIdx.x == 0) own = atomicAdd(&ctl.rec->tile_next[my_x * 32u], 1u);      // the block's next tile is asked for now
    // A step, of the half SECOND; MORE: another one follows, MORE2: and one more (all known when compiling: scalar code between the
    // MFMAs and the barriers, and between the barriers and the fetches, is in the way of both halves).  The waits stand before the
    // barrier behind which the first half reads what they wait for: at the end of its own matrix phase, at the end of the second
    // half's memory phase.
    auto step = [&](uint32_t t, auto SECOND, auto MORE, auto MORE2) {
      constexpr bool late = decltype(SECOND)::value != 0, more = decltype(MORE)::value != 0, more2 = decltype(MORE2)::value != 0;
      const bf16_t* cur = lds + (t & 1u) * STAGE;
      auto second_halves = [&] { wait_vm<more ? 2 * FA + 2 * FB : 0>(); };                        // of A, step t
      auto next_step = [&] { if (more) wait_vm<FA + (more2 ? FA + FB : 0)>(); };                  // B and first halves of A, step t + 1
      read_b(cur + 2 * HA);
      read_a(cur);
      if (more) { fetch_b(t + 1, Int<1>()); fetch_a1(t + 1); }
      wait_lds();
      if (late) second_halves();
      barrier_only();
      multiply(Int<0>());
      if (!late) second_halves();
      barrier_only();
      read_a(cur + HA);
      base_a += step_a; base_b += step_b;
      if (more2) { fetch_a0(t + 2); fetch_b(t + 2, Int<0>()); }
      wait_lds();
      if (late) next_step();
      barrier_only();
      multiply(Int<1>());
      if (!late) next_step();
      barrier_only();
    };
    auto steps = [&](auto SECOND) {
      uint32_t t = 0;
      for (; t + 2 < nt; ++t) step(t, SECOND, Int<1>(), Int<1>());
      if (t + 1 < nt) { step(t, SECOND, Int<1>(), Int<0>()); ++t; }
      if (t < nt) step(t, SECOND, Int<0>(), Int<0>());
    };
    if (second) { barrier_only(); steps(Int<1>()); } else { steps(Int<0>()); barrier_only(); }

    if (threadIdx.x == 0) {
      uint32_t np = kNone;
      if (dynamic) np = own < gemm_tiles_of_xcd(all_tiles, my_x) ? own * 8u + my_x : gemm_steal_tile(ctl.rec, all_tiles, my_x);
      else if (pid + gridDim.x < all_tiles) np = pid + gridDim.x;
      s_next = np;
    }
    __syncthreads();
    pid = s_next;
    if (pid < all_tiles) open_tile(pid);
    else arrival = kernel_arrive(ctl, !GROUPED, threadIdx.x == 0);
    if (cnt != 0) {
      const GemmP cp = gemm_read_record(current);
      uint32_t l = lane;
      asm volatile("" : "+v"(l));              // (as in open_tile)
      gemm_store_tile<TI, TJ, EPI, 1>(cp, acc, stage + wave * (kStage / 4), cm0 + wm * (TI * 32), cn0 + wn * 64, (size_t)(bo * cp.c_so + bi * cp.c_si), l, s_bias + wave * 512);
    }
  }
  kernel_finish(ctl, arrival, threadIdx.x == 0, true);
}

static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// ---------------------------------------------------------------------------------------------- configurations
// What a launch costs, per configuration: 2 us, and per round of tiles `fixed` + `step` * (K steps of 64) us with `slots`
// tiles on a CU at a time, `step1` with one.  Least squares over 37 shapes from 77 x 768 x 3072 to 8192^3, three operand
// layouts and three epilogues, of kernels on 32x32x16 MFMAs.  Checked against every configuration's time on the present ones at 638
// other shapes, plain products launched back to back: the modelled times are 0.65 to 1.4 of the measured ones (the two largest tiles
// are 1.25 times as fast as modelled, the small ones as modelled), the choice is on average 0.9 % slower than the best
// configuration, 6 % in the 95th percentile, and at worst 54 % (1299 x 3000 x 7296: 110 us on 64x64, 71 on 256x128).  8192 x 3072 x
// 768 takes 44 us on 256x128 and 40 on 256x256; inside the training step, with its epilogues and with operands that come from
// memory, it took 67.6 on 256x128 and 71.2 on 128x128 with the kernels before.  Over 477 products of 32 to 4096 rows with
// weights from memory the choice was 0.4 % above the best on average, as it was with constants fitted to those.
struct GemmTiles { uint32_t bm, bn, slots; double fixed, step, step1; };
enum { kT32x64, kT64x64, kT128x64, kT128x128x1, kT128x128, kT256x128, kT256x256, kNTiles };
static const GemmTiles kGemmTiles[kNTiles] = {
    {32, 64, 3, 1.75, 0.380, 0.114}, {64, 64, 2, 1.80, 0.369, 0.171},   {128, 64, 2, 2.40, 0.616, 0.261},  {128, 128, 1, 2.94, 0.436, 0.436},
    {128, 128, 2, 2.69, 0.958, 0.525}, {256, 128, 1, 4.99, 0.735, 0.735}, {256, 256, 1, 6.68, 1.233, 1.233},
};

// whole K steps - also in the last, shorter slice of a K cut into slices - and no causal variant: what the 256x256 tiles
// need
static bool gemm_causal(const sif_gemm_args& a) { return a.k_causal != 0 || (a.epilogue & SIF_EPI_CAUSAL_SKIP); }
static bool gemm_whole_steps(const sif_gemm_args& a) {
  if (gemm_causal(a) || (a.k % BK) != 0) return false;
  if (a.k_limit == 0) return true;
  const uint64_t before_last = (uint64_t)(a.batch_inner - 1) * a.k;
  return a.k_limit > before_last && ((a.k_limit - before_last) % BK) == 0;
}

// A causal product stops at the end of its row's (and skips what lies beyond its column's) 128-wide tile: what is past it
// need not have been written, so tiles more than 128 rows tall are not for it.
static bool gemm_tiles_fit(const sif_gemm_args& a, int cfg) {
  if (cfg == kT256x256) return gemm_whole_steps(a);
  return cfg != kT256x128 || !gemm_causal(a);
}

static uint64_t gemm_tiles_of(const sif_gemm_args& a, int cfg) {
  const GemmTiles& t = kGemmTiles[cfg];
  return (uint64_t)((a.m + t.bm - 1) / t.bm) * ((a.n + t.bn - 1) / t.bn) * a.batch_outer * a.batch_inner;
}
static double gemm_steps_of(const sif_gemm_args& a) { return (double)((a.k + BK - 1) / BK); }

static double gemm_time_us(uint64_t tiles, double steps, int cfg) {
  const GemmTiles& t = kGemmTiles[cfg];
  const uint64_t round = 256ull * t.slots, whole = tiles / round, rest = tiles % round;
  double us = 2.0 + (double)whole * (t.fixed + t.step * steps);
  if (rest > 0) {
    // a last round goes by the CU that holds the most of its tiles
    const double share = rest <= 256 ? 0.0 : (double)((rest - 1) / 256) / (double)(t.slots - 1);
    us += t.fixed + (t.step1 + (t.step - t.step1) * share) * steps;
  }
  return us;
}

static int gemm_choose(const sif_gemm_args& a) {
  if (a.tile == 256) return kT256x256;
  if (a.tile == 128) return kT128x128;
  int best = kT128x128;
  double best_us = gemm_time_us(gemm_tiles_of(a, best), gemm_steps_of(a), best);
  for (int c = 0; c < kNTiles; ++c) {
    if (!gemm_tiles_fit(a, c)) continue;
    const double us = gemm_time_us(gemm_tiles_of(a, c), gemm_steps_of(a), c);
    if (us < best_us) { best = c; best_us = us; }
  }
  return best;
}

uint32_t gemm_round_rows(const sif_gemm_args& a) {
  const GemmTiles& t = kGemmTiles[gemm_choose(a)];
  return t.bm * std::max(1u, 256u * t.slots / ((a.n + t.bn - 1) / t.bn));
}

// checks one product's arguments and fills its kernel record for configuration `cfg` (kAuto: the one gemm_choose takes)
constexpr int kAuto = -1;
static sif_status gemm_fill(const sif_gemm_args* a, GemmP& p, int cfg, int* cfg_out) {
  if (a == nullptr || a->struct_size != sizeof(sif_gemm_args)) return fail(SIF_E_INVAL, "gemm: bad args struct");
  if (a->m == 0 || a->n == 0 || a->k == 0) return fail(SIF_E_INVAL, "gemm: empty extent");
  if (a->a_layout > 1 || a->b_layout > 1) return fail(SIF_E_INVAL, "gemm: bad layout");
  if (!a->a_dev || !a->b_dev || !a->c_dev) return fail(SIF_E_INVAL, "gemm: null operand");
  if (!aligned16(a->a_dev) || !aligned16(a->b_dev) || !aligned16(a->c_dev)) return fail(SIF_E_INVAL, "gemm: operands must be 16-byte aligned");
  if ((a->lda & 7) || (a->ldb & 7)) return fail(SIF_E_INVAL, "gemm: lda/ldb must be multiples of 8");
  // a lane's offset within an operand tile (up to 255 rows of ld elements) is kept in 32 bits
  if (a->lda > (1u << 22) || a->ldb > (1u << 22)) return fail(SIF_E_INVAL, "gemm: lda/ldb above 4194304 elements are not supported");
  if ((a->a_stride_outer | a->a_stride_inner | a->b_stride_outer | a->b_stride_inner) & 7) return fail(SIF_E_INVAL, "gemm: batch strides must be multiples of 8");
  const uint32_t a_contig = a->a_layout == SIF_A_ROW_K ? a->k : a->m;
  const uint32_t b_contig = a->b_layout == SIF_B_ROW_K ? a->k : a->n;
  if (a->lda < ((a_contig + 7) & ~7u) || a->ldb < ((b_contig + 7) & ~7u) || a->ldc < a->n) return fail(SIF_E_INVAL, "gemm: leading dimension too small");
  if (a->batch_outer == 0 || a->batch_inner == 0) return fail(SIF_E_INVAL, "gemm: batch counts must be >= 1");
  if ((a->epilogue & SIF_EPI_GELU_GRAD) && !a->aux_dev) return fail(SIF_E_INVAL, "gemm: GELU_GRAD needs aux");
  if ((a->epilogue & SIF_EPI_RESIDUAL) && !a->res_dev) return fail(SIF_E_INVAL, "gemm: RESIDUAL needs res");
  if ((a->epilogue & (SIF_EPI_BIAS | SIF_EPI_GELU)) == SIF_EPI_BIAS && !a->bias_dev) return fail(SIF_E_INVAL, "gemm: BIAS needs bias");
  if (a->k_causal > 2) return fail(SIF_E_INVAL, "gemm: bad k_causal");
  if (a->k_limit != 0 && (a->k_causal != 0 || (uint64_t)(a->batch_inner - 1) * a->k >= a->k_limit || a->k_limit > (uint64_t)a->batch_inner * a->k))
    return fail(SIF_E_INVAL, "gemm: k_limit must lie in the last of the batch_inner slices of k (no k_causal)");
  if ((a->n & 7) == 0) {
    // vector epilogue: rows of C, the residual and the auxiliary tensor are accessed 8 elements at a time
    if ((a->ldc & 7) || ((a->c_stride_outer | a->c_stride_inner) & 7)) return fail(SIF_E_INVAL, "gemm: ldc and the output batch strides must be multiples of 8 when n is");
    if ((a->bias_dev && !aligned16(a->bias_dev)) || (a->res_dev && !aligned16(a->res_dev)) || (a->aux_dev && !aligned16(a->aux_dev))) return fail(SIF_E_INVAL, "gemm: bias, residual and aux must be 16-byte aligned");
  }
  if (a->tile != 0 && a->tile != 128 && a->tile != 256) return fail(SIF_E_INVAL, "gemm: tile must be 0, 128 or 256");
  if (a->tile == 256 && !gemm_whole_steps(*a)) return fail(SIF_E_INVAL, "gemm: 256-wide tiles need k (and the last slice under k_limit) to be a multiple of 64 and no causal variant");
  const uint64_t batches = (uint64_t)a->batch_outer * a->batch_inner;
  if (cfg == kAuto) cfg = gemm_choose(*a);
  const uint32_t bm = kGemmTiles[cfg].bm, bn = kGemmTiles[cfg].bn;
  p.a = (const bf16_t*)a->a_dev; p.b = (const bf16_t*)a->b_dev; p.c = a->c_dev;
  p.bias = (a->epilogue & (SIF_EPI_BIAS | SIF_EPI_GELU)) ? (const bf16_t*)a->bias_dev : nullptr;
  p.res = a->res_dev; p.aux = (bf16_t*)a->aux_dev;
  p.m = a->m; p.n = a->n; p.k = a->k; p.lda = a->lda; p.ldb = a->ldb; p.ldc = a->ldc;
  p.epi = a->epilogue; p.k_causal = a->k_causal; p.batch_inner = a->batch_inner; p.k_limit = a->k_limit;
  p.a_so = a->a_stride_outer; p.a_si = a->a_stride_inner; p.b_so = a->b_stride_outer; p.b_si = a->b_stride_inner;
  p.c_so = a->c_stride_outer; p.c_si = a->c_stride_inner; p.alpha = a->alpha;
  p.tiles_n = (a->n + bn - 1) / bn; p.tiles_m = (a->m + bm - 1) / bm;
  p.group = nullptr; p.group_n = 0; p.tile_base = 0;
  if (batches > 65535) return fail(SIF_E_INVAL, "gemm: grid too large");
  *cfg_out = cfg;
  return SIF_OK;
}

typedef void (*gemm_kern_fn)(GemmP, KCtl);
#define OF_LAYOUTS(KERNEL, EPI, ...)                                                                                              \
  {{KERNEL<0, 0, __VA_ARGS__ EPI>, KERNEL<0, 1, __VA_ARGS__ EPI>}, {KERNEL<1, 0, __VA_ARGS__ EPI>, KERNEL<1, 1, __VA_ARGS__ EPI>}}
#define OF_EPILOGUES(KERNEL, ...) {OF_LAYOUTS(KERNEL, kEpiCommon, __VA_ARGS__), OF_LAYOUTS(KERNEL, kEpiRare, __VA_ARGS__)}
#define RING(...) OF_EPILOGUES(gemm_ring_kernel, __VA_ARGS__, )
#define FED(...) OF_EPILOGUES(gemm_fed_kernel, __VA_ARGS__, )
// The kernels: one per configuration, and behind them those with wavefronts that only fetch.
enum { kFed32x64 = kNTiles, kFed64x64, kFed128x64, kFed32x32, kNKernels };
static const struct { gemm_kern_fn kern[2][2][2]; uint32_t threads; } kGemmKernels[kNKernels] = {      // [common or rare epilogue][layout of A][layout of B]
    {RING(32, 64, 1, 2, 4, 1, 2), 128},    {RING(64, 64, 2, 2, 4, 1, 2), 256},    {RING(128, 64, 2, 2, 3, 0, 2), 256}, {RING(128, 128, 4, 2, 4, 1, 1), 512},
    {RING(128, 128, 2, 2, 2, 0, 2), 256},  {RING(256, 128, 4, 2, 3, 0, 1), 512},  {OF_EPILOGUES(gemm_pp_kernel, ), 512},
    {FED(32, 64, 1, 2, 4, 6, 2), 384},     {FED(64, 64, 2, 2, 4, 8, 1), 512},     {FED(128, 64, 2, 2, 4, 6, 1), 512},  {FED(32, 32, 1, 1, 4, 6, 2), 320}};
#undef RING
#undef FED
#undef OF_LAYOUTS
#undef OF_EPILOGUES

static uint32_t gemm_cus() {
  static const uint32_t cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = 256;
    return (uint32_t)(n / 8 * 8);
  }();
  return cus;
}

// The kernel of a product on configuration cfg's tiles: where no CU gets more than one of the smaller tiles the one with
// wavefronts that only fetch, and 32x32 tiles instead of 32x64 where that is still one per CU (a third less to fetch for each;
// 77 x 768 x 3072: 8.1 us, on 32x64 9.5).  A single K step has no fetches to keep in flight, and the ring's smaller blocks start
// sooner: with K 8 and 64 twelve shapes from 32 x 768 to 1024 x 1024 take 3.3 to 3.9 us on it, 3.4 to 4.2 on the others.  (From
// K 128 to 1024 the others take 0.63 to 0.98 of the ring's time with weights from memory, with operands that stay in the L2 0.93
// to 1.01, but 64x64 tiles from K 512 on 1.03 to 1.07.)
static int gemm_kernel(const sif_gemm_args& a, int cfg) {
  if (cfg > kT128x64 || a.k <= BK || gemm_tiles_of(a, cfg) > gemm_cus()) return cfg;
  const uint64_t narrow = (uint64_t)((a.m + 31) / 32) * ((a.n + 31) / 32) * a.batch_outer * a.batch_inner;
  return cfg == kT32x64 && narrow <= gemm_cus() ? (int)kFed32x32 : kFed32x64 + cfg;
}
int gemm_kernel_of(const sif_gemm_args& a) { return gemm_kernel(a, gemm_choose(a)); }

sif_status launch_gemm_bf16(const sif_gemm_args* a, hipStream_t stream, const KCtl& ctl) {
  GemmP p;
  int cfg = kAuto;
  if (sif_status st = gemm_fill(a, p, kAuto, &cfg)) return st;
  const uint64_t batches = (uint64_t)a->batch_outer * a->batch_inner;
  const int kernel = gemm_kernel(*a, cfg);
  if (kernel == kFed32x32) p.tiles_n = (a->n + 31) / 32;
  // 256x256 tiles: one block per CU, each working through every (number of CUs)-th tile; a stride that is a multiple of
  // 8 keeps a block on the tiles of its own XCD
  uint32_t grid_x = p.tiles_m * p.tiles_n;
  if (cfg == kT256x256 && batches == 1) grid_x = std::min(grid_x, gemm_cus());
  const auto kern = kGemmKernels[kernel].kern[gemm_rare(a->epilogue, a->n, a->ldc)][a->a_layout][a->b_layout];
  hipLaunchKernelGGL(kern, dim3(grid_x, 1, (uint32_t)batches), dim3(kGemmKernels[kernel].threads), 0, stream, p, ctl);
  return check_launch("gemm_bf16");
}

// Several products of the same operand layouts as ONE launch (the weight gradients of a layer: each by itself has too
// few tiles for the chip and would have to be cut along K, with fp32 partial results written, read again and summed;
// together they fill it).  gemm_group_fill checks the products, chooses the tiles and writes the kernel records, to be
// copied to `gemm_group_bytes(n)` bytes of device memory once; launch_gemm_bf16_group then takes that copy.
uint64_t gemm_group_bytes(uint32_t n) { return (uint64_t)n * sizeof(GemmP); }

// Which tiles: the model's time for all products' tiles together, the longest K deciding.  A small layer's gradients (21
// tiles of 128x128 at 128 x 512) are a chain of K steps on few CUs: 128x128 with four steps in the ring of a CU's only
// block, as long as that is one round (2048 tokens of 128 x 512: 16 us, with two steps in the ring 20, on 256x128 27;
// two rounds, 8192 tokens of 768 x 3072: 131 us, where two blocks of a CU hide each other's ends 125).
//   Every product begins at a multiple of eight blocks, so the first XCD gets an eighth of each product's tiles, rounded up, and
// with one tile per CU that is what makes a round (256x256 too: a block asks for its next tile when it begins one, so an XCD's
// 33rd is taken there).  (85 + 85 + 20 + 60 tiles of 128x128 are 250, but 33 on each of four XCDs, whose 32 CUs begin a second
// round: steps of four layers of 520 x 2056 on 8192 tokens 2.91 ms, on 256x128 2.65; 704 x 2816 on 8192 3.24 -> 3.05, 856 x 7176 on
// 8192 5.88 -> 5.49.  Over 48 layers and token counts at such borders a step takes 0.98 of the time, at most 1.02.  With
// two tiles per CU these hide it: counted so for them, nine of 110 launches got slower by up to 11 %.)
static int gemm_group_choose(const sif_gemm_args* list, uint32_t n, double* us_out) {
  int cfg = -1;
  double best = 0.0;
  for (int c : {(int)kT128x128, (int)kT128x128x1, (int)kT256x128, (int)kT256x256}) {
    uint64_t tiles = 0;
    double steps = 0.0;
    bool ok = true;
    for (uint32_t i = 0; i < n; ++i) {
      const uint64_t own = gemm_tiles_of(list[i], c);
      tiles += kGemmTiles[c].slots == 1 ? (own + 7) / 8 * 8 : own;
      steps = std::max(steps, gemm_steps_of(list[i]));
      ok = ok && gemm_tiles_fit(list[i], c);
    }
    ok = ok && (c != kT128x128x1 || tiles <= 256);
    const double us = gemm_time_us(tiles, steps, c);
    if (ok && (cfg < 0 || us < best)) { cfg = c; best = us; }
  }
  *us_out = best;
  return cfg;
}

// How many of a launch's n products it should hold, where the ones from `first` on could be launches of their own: all, or the
// first ones.  By themselves these take small tiles that the whole chip shares; in the group a row of them is a chain over
// the whole K on a few big tiles, which costs nothing in a round that is not full and a whole round where it begins one.
// (4096 tokens of 2048 columns: 768 tiles of 256x256 are three rounds, with two one-row products more a fourth.  Modelled
// 344 us against 259 and twice 11; a step of six such layers, two micro-batches: 17.0 -> 16.5 ms.)
//   The model has to see a tenth and 5 us for each launch that follows: its error is of that size, and a one-row product takes 13 us
// where it says 11, and a gap to the next launch.  (Steps of four layers of random widths, apart against the group whole: where the
// model sees less than that 0.99 to 1.04 of the time, on average 1.02; where it sees more 0.95 to 1.01, on average 0.985.)
uint32_t gemm_group_part(const sif_gemm_args* list, uint32_t first, uint32_t n) {
  if (first == 0 || first >= n) return n;
  double all = 0.0, apart = 0.0;
  if (gemm_group_choose(list, n, &all) < 0 || gemm_group_choose(list, first, &apart) < 0) return n;
  for (uint32_t i = first; i < n; ++i) {
    const int cfg = gemm_choose(list[i]);
    apart += gemm_time_us(gemm_tiles_of(list[i], cfg), gemm_steps_of(list[i]), cfg);
  }
  return apart < 0.91 * all && apart + 5.0 * (n - first) < all ? first : n;
}

sif_status gemm_group_fill(const sif_gemm_args* list, uint32_t n, void* host_records, GemmGroup* out) {
  if (list == nullptr || n == 0 || n > 16 || host_records == nullptr || out == nullptr) return fail(SIF_E_INVAL, "gemm group: bad arguments");
  double us = 0.0;
  const int cfg = gemm_group_choose(list, n, &us);
  GemmP* rec = static_cast<GemmP*>(host_records);
  uint32_t base = 0;
  out->rare = 0;
  for (uint32_t i = 0; i < n; ++i) {
    sif_gemm_args a = list[i];
    if (a.a_layout != list[0].a_layout || a.b_layout != list[0].b_layout) return fail(SIF_E_INVAL, "gemm group: the products must share their operand layouts");
    if ((uint64_t)a.batch_outer * a.batch_inner != 1) return fail(SIF_E_INVAL, "gemm group: no batched products");
    a.tile = 0;
    int got = 0;
    if (sif_status st = gemm_fill(&a, rec[i], cfg, &got)) return st;
    out->rare |= gemm_rare(a.epilogue, a.n, a.ldc);
    rec[i].tile_base = base;
    base += (rec[i].tiles_m * rec[i].tiles_n + 7u) & ~7u;       // a multiple of 8 keeps the tile order's idea of the XCDs
  }
  out->tiles = base;
  out->cfg = cfg;
  return SIF_OK;
}

sif_status launch_gemm_bf16_group(const void* dev_records, uint32_t n, const GemmGroup& g, uint32_t a_layout, uint32_t b_layout, hipStream_t stream, const KCtl& ctl) {
  if (dev_records == nullptr || n == 0 || g.tiles == 0 || a_layout > 1 || b_layout > 1) return fail(SIF_E_INVAL, "gemm group: bad arguments");
  GemmP head = {};
  head.group = static_cast<const GemmP*>(dev_records);
  head.group_n = n;
  head.batch_inner = 1;
  head.tiles_m = g.tiles;
  // (instantiated for the layouts of weight gradients, A [K][M] and B [K][N]; other layouts would need their own)
  if (a_layout != SIF_A_ROW_M || b_layout != SIF_B_ROW_N) return fail(SIF_E_INVAL, "gemm group: only A stored [K][M] with B stored [K][N]");
#define GROUPED(KERNEL, ...) (g.rare ? KERNEL<1, 1, __VA_ARGS__ kEpiAll, true> : KERNEL<1, 1, __VA_ARGS__ kEpiCommon, true>)
  gemm_kern_fn kern = GROUPED(gemm_ring_kernel, 128, 128, 2, 2, 2, 0, 2, );
  if (g.cfg == kT256x256) kern = GROUPED(gemm_pp_kernel, );
  if (g.cfg == kT128x128x1) kern = GROUPED(gemm_ring_kernel, 128, 128, 4, 2, 4, 1, 1, );
  if (g.cfg == kT256x128) kern = GROUPED(gemm_ring_kernel, 256, 128, 4, 2, 3, 0, 1, );
#undef GROUPED
  hipLaunchKernelGGL(kern, dim3(g.cfg == kT256x256 ? std::min(g.tiles, gemm_cus()) : g.tiles), dim3(kGemmKernels[g.cfg].threads), 0, stream, head, ctl);
  return check_launch("gemm_bf16_group");
}

}  // namespace sif
