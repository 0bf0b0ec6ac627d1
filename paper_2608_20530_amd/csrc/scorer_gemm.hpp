// Matrix products of the scoring-Transformer stand-in on the bf16 matrix cores: C[M][N] = A[M][K] .
// B[K][N] with the epilogue of its mode. Both operands are kept in fragment order, 16 rows of A (or
// 16 columns of B) x 32 k-values per 1 KB fragment:
//   [k-block][row block][lane 64][8 bf16], lane l holding row (column) l % 16, k (l / 16) * 8 ..
// so one 16-byte-per-lane load is one operand of v_mfma_f32_16x16x32_bf16, a fragment is one
// contiguous kilobyte wherever it is read from, and LDS reads of it have no bank conflicts and
// need no swizzle. The producers of A (RMSNorm, attention, the SiLU epilogue) write that order
// directly; B is packed into it once. Rows past M inside the last row block hold whatever the
// buffer held: they only reach output rows that are not stored.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "common.hpp"

namespace lilicorr {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) void* lds_ptr_t;

constexpr uint32_t kFragBytes = 1024;  // one fragment
constexpr int kGemmThreads = 512;      // eight waves
constexpr int kNormMaxK = 1024;        // widest rows that a product normalises itself
constexpr float kEps = 1e-6f;          // of RMSNorm
constexpr int kGroup = 8;              // row blocks per tile group (L2 blocking of the grid)

// fp32 -> bf16, round to nearest even: one v_cvt_pk_bf16_f32 per pair of values on gfx950
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

__device__ __forceinline__ uint32_t bf16_rne(float x) {
  return __builtin_bit_cast(uint16_t, (__bf16)x);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}

// Byte offset, in an A operand of row_blocks row blocks, of columns col .. col + 3 of token row
// `row` (col % 4 == 0).
__device__ __forceinline__ size_t frag_offset(int64_t row, int col, int64_t row_blocks) {
  return ((size_t)(col / 32) * row_blocks + (row >> 4)) * kFragBytes +
         (((col >> 3) & 3) * 16 + (int)(row & 15)) * 16 + (col & 4) * 2;
}

enum { kModeQKV = 0, kModeResid = 1, kModeSilu = 2 };

struct GemmArgs {
  const uint16_t* A;   // fragment order, ceil(M / 16) row blocks
  const uint16_t* B;   // fragment order, N / 16 column blocks
  int64_t M;
  int K, N;            // multiples of 128
  float* X;            // resid: X[M][N] += A . B
  uint16_t* Y;         // silu: bf16(silu(A . B)) in fragment order; qkv: Q and K, Y[M][2H]
  uint16_t* Vt;        // qkv: V columns transposed per request, Vt[M / L][H][Lv]
  int H, L, Lv;
  const float* Xn;     // where the kernel normalises its own rows: A = rms norm of Xn[M][K] ...
  const float* g;      // ... times g[K], rounded to bf16
};

// One accumulator tile of the products (weights x activations): lane holds columns
// col .. col + 3 of token row `row`.
template <int MODE>
__device__ __forceinline__ void store_row_quad(const GemmArgs& p, const f32x4& v, int64_t row,
                                               int col) {
  if (row >= p.M) return;
  if constexpr (MODE == kModeResid) {
    f32x4* x = reinterpret_cast<f32x4*>(p.X + row * p.N + col);
    *x = *x + v;
  } else if constexpr (MODE == kModeSilu) {
    // silu(v) = v / (1 + e^-v), the reciprocal on the hardware unit (the result is rounded to
    // bf16 next)
    float s[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) s[i] = v[i] * __builtin_amdgcn_rcpf(1.0f + __expf(-v[i]));
    *reinterpret_cast<u32x2*>(reinterpret_cast<unsigned char*>(p.Y) + frag_offset(row, col, (p.M + 15) / 16)) =
        u32x2{pack_bf16x2(s[0], s[1]), pack_bf16x2(s[2], s[3])};
  } else {
    *reinterpret_cast<u32x2*>(p.Y + row * (2 * p.H) + col) =
        u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  }
}

// A tile rounded to bf16 and transposed by 4 x 4 blocks within each lane quad (four tokens, four
// columns): the lane then holds four consecutive tokens, (lane & 12) .. + 3, of column
// 4 (lane / 16) + (lane & 3).
__device__ __forceinline__ u32x2 transpose_quad(const f32x4& v, int lane) {
  const uint32_t w0 = pack_bf16x2(v[0], v[1]), w1 = pack_bf16x2(v[2], v[3]);
  auto quad = [](uint32_t x, auto ctrl) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, decltype(ctrl)::value, 0xf, 0xf, false);
  };
  typedef std::integral_constant<int, 0xB1> Xor1;  // quad_perm 1,0,3,2
  typedef std::integral_constant<int, 0x4E> Xor2;  // quad_perm 2,3,0,1
  const uint32_t o0 = quad(w0, Xor1{}), o1 = quad(w1, Xor1{});
  // even lanes take the low halves (columns 0, 2) of both tokens, odd lanes the high halves
  const uint32_t sel = (lane & 1) ? 0x03020706u : 0x05040100u;  // v_perm: bytes 0-3 are w's
  const uint32_t n0 = __builtin_amdgcn_perm(o0, w0, sel), n1 = __builtin_amdgcn_perm(o1, w1, sel);
  const uint32_t q0 = quad(n0, Xor2{}), q1 = quad(n1, Xor2{});
  return (lane & 2) ? u32x2{q1, n1} : u32x2{n0, q0};
}

// The V columns' output, transposed: the tile of token rows row0 .. row0 + 15 (row0 % 16 == 0) and
// columns col0 .. col0 + 15. Each lane stores four consecutive positions of one dimension of V^T;
// where a request may end among them (L % 4 != 0), value by value instead.
__device__ __forceinline__ void store_v_tile(const GemmArgs& p, const f32x4& v, int64_t row0,
                                             int col0, int lane) {
  const int g = lane >> 4, c16 = lane & 15;
  if (p.L % 4 == 0) {
    const u32x2 t = transpose_quad(v, lane);
    const int64_t row = row0 + (c16 & 12);
    if (row < p.M) {
      const int rq = (int)row / p.L, l = (int)row - rq * p.L;
      const int dim = col0 + 4 * g + (c16 & 3) - 2 * p.H;
      *reinterpret_cast<u32x2*>(p.Vt + ((int64_t)rq * p.H + dim) * p.Lv + l) = t;
    }
    return;
  }
  const int64_t row = row0 + c16;
  if (row >= p.M) return;
  const int rq = (int)row / p.L, l = (int)row - rq * p.L;
  uint16_t* o = p.Vt + ((int64_t)rq * p.H + (col0 + 4 * g - 2 * p.H)) * p.Lv + l;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[(size_t)i * p.Lv] = (uint16_t)bf16_rne(v[i]);
}

// Tile t of the grid. Workgroups are dealt to the eight XCDs round robin; when the grid divides
// evenly, each XCD takes a contiguous run of tile numbers. Tile numbers run over groups of kGroup
// row tiles, column tiles outer, so the workgroups an XCD holds at once share A rows and B columns
// in its L2.
__device__ __forceinline__ void tile_of(int64_t M, int ntn, int BM, int64_t& tm, int& tn) {
  const uint32_t nt = gridDim.x;
  const uint32_t t = (nt % 8u == 0u) ? (blockIdx.x % 8u) * (nt / 8u) + blockIdx.x / 8u
                                     : blockIdx.x;
  const int64_t ntm = (M + BM - 1) / BM;
  const int64_t per_group = (int64_t)kGroup * ntn;
  const int64_t grp = t / per_group;
  const int64_t rows_in = (ntm - grp * kGroup) < kGroup ? (ntm - grp * kGroup) : kGroup;
  const int64_t r = t - grp * per_group;
  tm = grp * kGroup + r % rows_in;
  tn = (int)(r / rows_in);
}

// ---- 128 x 256 tiles ----------------------------------------------------------------------------
// Four waves, each a 128 x 64 block of 8 x 4 accumulator tiles in ordinary registers, two workgroups
// per compute unit (one's prologue and epilogue run beside the other's products). The A tile goes
// through LDS (DMA: buffer loads with an LDS destination), in a ring of four 64-deep stages of
// 16 KB, shared by the four waves; each wave reads the four B fragments of a k-block straight from
// the L1/L2 into one of four register buffers, three k-blocks ahead. Only A in LDS: with both
// operands there, 12 KB of LDS reads per 32 MFMAs and wave plus the copies ask for more than the
// 128 bytes a cycle that LDS gives (the four products at M = 15360, H = 1024, F = 2048 took 112,
// 47, 76 and 88 us that way and take 90, 47, 64 and 70 now; the loop alone runs at 1.6 PFLOP/s,
// and what is left is the first loads, the output and, for the residual, 126 MB of X that no
// product runs beside: one round of tiles). 256 x 256 tiles of eight waves, one workgroup per
// compute unit, took 112, 48, 67 and 69 us with the products alone.
constexpr int kBigThreads = 256;
constexpr int kBigStages = 4;
constexpr int kBigRows = 8;  // row blocks of a tile
constexpr uint32_t kBigStageBytes = kBigRows * 2 * kFragBytes;  // x 2 k-blocks
constexpr size_t kBigLds = (size_t)kBigStages * kBigStageBytes;
constexpr uint32_t kWaveLds = kBigLds / 4;  // a wave's share of it, for the epilogue

template <int MODE>
__global__ __launch_bounds__(kBigThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_big_kernel(GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char big_smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  int64_t tm;
  int tn;
  tile_of(p.M, (p.N + 255) / 256, 16 * kBigRows, tm, tn);
  const int KB = p.K / 32;
  const uint32_t row_blocks = (uint32_t)((p.M + 15) / 16);
  const uint32_t col_blocks = (uint32_t)(p.N / 16);
  const uint32_t stepA = row_blocks * kFragBytes, stepB = col_blocks * kFragBytes;  // one k-block
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.A, (uint32_t)KB * stepA);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.B, (uint32_t)KB * stepB);
  // lane offsets of the two row blocks this wave copies and of its four column blocks (kOut where
  // they lie past M or N: such loads return zeros and fetch nothing); the k-block displacement is
  // scalar, and loads past the last k-block get kOut added
  constexpr uint32_t kOut = 0x80000000u;
  const uint32_t voff = (uint32_t)lane * 16u;
  uint32_t offA[2], offB[4];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const uint32_t rb16 = (uint32_t)tm * kBigRows + (uint32_t)(wave * 2 + r);
    offA[r] = rb16 < row_blocks ? rb16 * kFragBytes + voff : kOut;
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t cb16 = (uint32_t)tn * 16u + (uint32_t)(wave * 4 + j);
    offB[j] = cb16 < col_blocks ? cb16 * kFragBytes + voff : kOut;
  }

  // stage s of the A tile: wave w copies row blocks 2w and 2w + 1, two k-blocks each; in LDS
  // [k-block][row block]
  const int ns = KB / 2;  // even: K is a multiple of 128
  auto dma = [&](int s) {
    unsigned char* dst = big_smem + (uint32_t)(s % kBigStages) * kBigStageBytes +
                         (uint32_t)wave * 2u * kFragBytes;
    const uint32_t past = s < ns ? 0u : kOut;
    const uint32_t k = s < ns ? (uint32_t)(s * 2) * stepA : 0u;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_ptr_t)(dst + (kb * kBigRows + r) * kFragBytes),
                                                 16, offA[r] | past, (int)(k + (uint32_t)kb * stepA),
                                                 0, 0);
  };
  bf16x8 b[4][4];
  auto load_b = [&](bf16x8 (&d)[4], int kb) {
    const uint32_t past = kb < KB ? 0u : kOut;
    const uint32_t k = kb < KB ? (uint32_t)kb * stepB : 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j)
      d[j] = __builtin_bit_cast(
          bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rb, offB[j] | past, (int)k, 0));
  };
  f32x4 acc[8][4];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // in this order, which the first wait's count relies on: the copies of stage 0, then the 20 loads
  // of the later stages' copies and the first weights
  dma(0);
  __builtin_amdgcn_sched_barrier(0);
  dma(1);
  dma(2);
  __builtin_amdgcn_sched_barrier(0);
  load_b(b[0], 0);
  load_b(b[1], 1);
  load_b(b[2], 2);
  __builtin_amdgcn_sched_barrier(0);
  for (int s = 0; s < ns; s += 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      // this wave's copies of stage s + u have landed once at most 20 of its loads are in flight
      // (20 are issued after the first stage's copies, 28 and more after later ones'). The barrier
      // then covers every wave's copies, and says that all waves are done with the slot that the
      // next copies overwrite.
      __asm__ volatile("s_waitcnt vmcnt(20)\n\ts_barrier" ::: "memory");
      dma(s + u + 3);
      const unsigned char* as = big_smem + (uint32_t)((s + u) % kBigStages) * kBigStageBytes + voff;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const int t = 2 * u + ks;  // k-block 2 s + t, in register buffer t
        load_b(b[(t + 3) & 3], 2 * s + t + 3);
        bf16x8 a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i)
          a[i] = *reinterpret_cast<const bf16x8*>(as + (uint32_t)(ks * kBigRows + i) * kFragBytes);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j)
            acc[i][j] =
                __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[t][j], a[i], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // no copy into this workgroup's LDS outlives it
  __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory");
  const int64_t row0 = tm * (16 * kBigRows);
  const int col0 = tn * 256 + wave * 64;
  const int g = lane >> 4, c16 = lane & 15;
  if constexpr (MODE == kModeQKV) {
    // through this wave's quarter of the ring, free once every wave is past its last stage, so that
    // each store instruction writes whole 128-byte lines (32-byte pieces of 16 rows per
    // instruction took 107 instead of 90 us for the whole product at M = 15360, H = 1024)
    __syncthreads();
    unsigned char* st = big_smem + (uint32_t)wave * kWaveLds;
    if (col0 < 2 * p.H) {  // uniform: H is a multiple of 256, a tile is all Q/K or all V
      constexpr uint32_t kStride = 64 * 2 + 16;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const f32x4& v = acc[h * 4 + i][j];
            *reinterpret_cast<u32x2*>(st + (i * 16 + c16) * kStride + (j * 16 + 4 * g) * 2) =
                u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
          }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int r = k * 8 + (lane >> 3), c = lane & 7;
          const u32x4 w = *reinterpret_cast<const u32x4*>(st + r * kStride + c * 16);
          const int64_t row = row0 + h * 64 + r;
          if (row < p.M) *reinterpret_cast<u32x4*>(p.Y + row * (2 * p.H) + col0 + c * 8) = w;
        }
      }
    } else if (p.L % 8 == 0) {  // eight consecutive positions of V^T at a time
      constexpr uint32_t kStride = 128 * 2 + 16;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            *reinterpret_cast<u32x2*>(st + (j * 16 + 4 * g + (c16 & 3)) * kStride +
                                      (i * 16 + (c16 & 12)) * 2) =
                transpose_quad(acc[i][h * 2 + j], lane);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int d = k * 4 + (lane >> 4);
          const u32x4 w = *reinterpret_cast<const u32x4*>(st + d * kStride + c16 * 16);
          const int64_t row = row0 + c16 * 8;
          if (row < p.M) {
            const int rq = (int)row / p.L, l = (int)row - rq * p.L;
            *reinterpret_cast<u32x4*>(
                p.Vt + ((int64_t)rq * p.H + col0 - 2 * p.H + h * 32 + d) * p.Lv + l) = w;
          }
        }
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          store_v_tile(p, acc[i][j], row0 + i * 16, col0 + j * 16, lane);
    }
    return;
  }
  if (col0 >= p.N) return;  // the last tile of an N that is an odd multiple of 128
  if constexpr (MODE == kModeResid) {
    // X += acc, the loads of row block i + 1 (rows past M clamped and not stored) issued before
    // block i is stored
    f32x4 xv[2][4];
    auto load = [&](int i, f32x4 (&d)[4]) {
      int64_t row = row0 + i * 16 + c16;
      row = row < p.M ? row : p.M - 1;
      const f32x4* x = reinterpret_cast<const f32x4*>(p.X + row * p.N + col0 + 4 * g);
#pragma unroll
      for (int j = 0; j < 4; ++j) d[j] = x[j * 4];
    };
    load(0, xv[0]);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i + 1 < 8) load(i + 1, xv[(i + 1) & 1]);
      const int64_t row = row0 + i * 16 + c16;
      if (row < p.M) {
        f32x4* x = reinterpret_cast<f32x4*>(p.X + row * p.N + col0 + 4 * g);
#pragma unroll
        for (int j = 0; j < 4; ++j) x[j * 4] = xv[i & 1][j] + acc[i][j];
      }
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        store_row_quad<MODE>(p, acc[i][j], row0 + i * 16 + c16, col0 + j * 16 + 4 * g);
  }
}

// ---- few tiles: the contraction split over the waves --------------------------------------------
// Eight waves on a (16 TM WM) x (16 TN WN) tile: WM x WN blocks of TM x TN accumulator tiles, and
// KS = 8 / (WM WN) waves per block that take every KS-th k-block. Both operands are read straight
// into registers (RING k-blocks in flight, no barrier in the loop); the partial sums meet in LDS,
// where wave by wave, in order, they are added and stored. What bounds these sizes is the latency
// of a few hundred KB through each compute unit and how many compute units have any work, so the
// contraction is cut rather than left to few workgroups (M = 120, H = 1024, F = 2048: 6.2, 3.3,
// 5.0 and 5 us for the four products against 21, 18, 18.5 and 26 us from 128 x 256 tiles).
//
// NORM (QKV and SiLU products of few rows, gemm_norms): the workgroup makes its own A rows,
// the bf16 rounding of their RMSNorm (the same operations in the same order as
// rmsnorm_bf16_kernel), in LDS while its first weights are on their way, and reads A from there.
template <int MODE, bool NORM, int TM, int TN, int WM, int WN, int RING>
__global__ __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_split_kernel(GemmArgs p) {
  constexpr int KS = 8 / (WM * WN), BM = 16 * TM * WM, BN = 16 * TN * WN;
  extern __shared__ __attribute__((aligned(16))) unsigned char split_smem[];
  f32x4* part = reinterpret_cast<f32x4*>(split_smem);  // [KS][WM * WN][TM * TN][64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = (int)__builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave / (WM * WN), blk = wave % (WM * WN), wm = blk / WN, wn = blk % WN;
  int64_t tm;
  int tn;
  tile_of(p.M, p.N / BN, BM, tm, tn);
  const int KB = p.K / 32;
  const uint32_t row_blocks = (uint32_t)((p.M + 15) / 16), col_blocks = (uint32_t)(p.N / 16);
  const uint32_t stepA = row_blocks * kFragBytes, stepB = col_blocks * kFragBytes;  // one k-block
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(p.A, (uint32_t)KB * stepA);
  const __amdgpu_buffer_rsrc_t rb = make_rsrc(p.B, (uint32_t)KB * stepB);
  constexpr uint32_t kOut = 0x80000000u;  // past every descriptor: the load returns zeros
  const uint32_t voff = (uint32_t)lane * 16u;
  const uint32_t a0 = (uint32_t)tm * (TM * WM) + (uint32_t)wm * TM;
  const uint32_t b0 = (uint32_t)tn * (TN * WN) + (uint32_t)wn * TN;
  uint32_t offA[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i)
    offA[i] = a0 + i < row_blocks ? (a0 + i) * kFragBytes + voff : kOut;

  // NORM: this wave's rows wave, wave + 8, .. of the tile, 256 columns a step, all in flight
  constexpr int NR = BM / 8, NV = kNormMaxK / 256;
  f32x4 x[NORM ? NR : 1][NV], gv[NV];
  if constexpr (NORM) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      int64_t row = tm * BM + wave + r * 8;
      row = row < p.M ? row : p.M - 1;  // such rows reach no output that is stored
#pragma unroll
      for (int j = 0; j < NV; ++j)
        x[r][j] = j * 256 < p.K ? *reinterpret_cast<const f32x4*>(p.Xn + row * p.K + (j * 64 + lane) * 4)
                                : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < NV; ++j)
      gv[j] = j * 256 < p.K ? *reinterpret_cast<const f32x4*>(p.g + (j * 64 + lane) * 4)
                            : f32x4{0.f, 0.f, 0.f, 0.f};
  }
  bf16x8 a[RING][TM], b[RING][TN];
  auto load = [&](int r, int step) {
    const int kb = ks + step * KS;
    // uniform; steps past the end multiply zeros
    const uint32_t past = kb < KB ? 0u : kOut;
    const uint32_t k = kb < KB ? (uint32_t)kb : 0u;
    if constexpr (!NORM)
#pragma unroll
      for (int i = 0; i < TM; ++i)
        a[r][i] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                                 ra, offA[i] | past, (int)(k * stepA), 0));
#pragma unroll
    for (int j = 0; j < TN; ++j)
      b[r][j] = __builtin_bit_cast(
          bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                      rb, (voff + (b0 + (uint32_t)j) * kFragBytes) | past, (int)(k * stepB), 0));
  };
  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int col0 = tn * BN;
  const bool vpart = MODE == kModeQKV && col0 >= 2 * p.H;  // uniform (BN divides H)
  const int nsteps = (KB + KS - 1) / KS;
#pragma unroll
  for (int r = 0; r < RING; ++r) load(r, r);
  __builtin_amdgcn_sched_barrier(0);
  // A in LDS: fragment (kb, row block) as everywhere, its 16-byte piece (row r, quarter q) at
  // q * 16 + (r ^ (4 kb + q) % 16), so that the pieces that one row's write covers lie in distinct
  // banks
  if constexpr (NORM) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      float ss = 0.f;
#pragma unroll
      for (int j = 0; j < NV; ++j)
        ss += x[r][j][0] * x[r][j][0] + x[r][j][1] * x[r][j][1] + x[r][j][2] * x[r][j][2] +
              x[r][j][3] * x[r][j][3];
      ss = wave_sum(ss);
      const float inv = 1.0f / sqrtf(ss / (float)p.K + kEps);
      const int rl = wave + r * 8;
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int col = (j * 64 + lane) * 4, kb = col >> 5, q = (col >> 3) & 3;
        if (col < p.K)
          *reinterpret_cast<u32x2*>(split_smem + (uint32_t)(kb * (TM * WM) + (rl >> 4)) * kFragBytes +
                                    (q * 16 + ((rl & 15) ^ ((kb * 4 + q) & 15))) * 16 + (col & 4) * 2) =
              u32x2{pack_bf16x2(x[r][j][0] * inv * gv[j][0], x[r][j][1] * inv * gv[j][1]),
                    pack_bf16x2(x[r][j][2] * inv * gv[j][2], x[r][j][3] * inv * gv[j][3])};
      }
    }
    __syncthreads();
  }
  for (int s = 0; s < nsteps; s += RING) {
#pragma unroll
    for (int r = 0; r < RING; ++r) {
      if constexpr (NORM) {
        const int kb = ks + (s + r) * KS, q = lane >> 4;  // zeros past the end
        const uint32_t at = (uint32_t)(q * 16 + ((lane & 15) ^ ((kb * 4 + q) & 15))) * 16u;
#pragma unroll
        for (int i = 0; i < TM; ++i)
          a[r][i] = kb < KB ? *reinterpret_cast<const bf16x8*>(
                                  split_smem + (uint32_t)(kb * (TM * WM) + wm * TM + i) * kFragBytes + at)
                            : bf16x8{};
      }
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[r][j], a[r][i], acc[i][j], 0, 0, 0);
      load(r, s + r + RING);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  if constexpr (NORM) __syncthreads();  // the partial sums take the place of A
  constexpr int F = TM * TN;
  f32x4* mine = part + (size_t)(ks * WM * WN + blk) * F * 64 + lane;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) mine[(i * TN + j) * 64] = acc[i][j];
  __syncthreads();
  const int g = lane >> 4, c16 = lane & 15;
  // the KS waves of a block share its accumulator tiles
  for (int f = ks; f < F; f += KS) {
    const f32x4* q = part + ((size_t)blk * F + f) * 64 + lane;
    f32x4 v = q[0];
#pragma unroll
    for (int k = 1; k < KS; ++k) v = v + q[(size_t)k * WM * WN * F * 64];
    const int64_t row = tm * BM + (wm * TM + f / TN) * 16;
    const int col = col0 + (wn * TN + f % TN) * 16;
    if (vpart)
      store_v_tile(p, v, row, col, lane);
    else
      store_row_quad<MODE>(p, v, row + c16, col + 4 * g);
  }
}

template <int MODE>
void launch_gemm_big(const GemmArgs& a, hipStream_t stream) {
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(gemm_big_kernel<MODE>),
      hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBigLds);
  (void)attr;
  const int64_t tiles = (a.M + 16 * kBigRows - 1) / (16 * kBigRows) * ((a.N + 255) / 256);
  hipLaunchKernelGGL(gemm_big_kernel<MODE>, dim3((unsigned)tiles), dim3(kBigThreads), kBigLds,
                     stream, a);
}

template <int MODE, bool NORM, int TM, int TN, int WM, int WN, int RING>
void launch_gemm_split(const GemmArgs& a, hipStream_t stream) {
  constexpr int BM = 16 * TM * WM, BN = 16 * TN * WN;
  constexpr size_t part = (size_t)8 * TM * TN * 64 * 16, rows = NORM ? (size_t)BM * kNormMaxK * 2 : 0;
  constexpr size_t lds = part > rows ? part : rows;
  static const hipError_t attr = hipFuncSetAttribute(
      reinterpret_cast<const void*>(gemm_split_kernel<MODE, NORM, TM, TN, WM, WN, RING>),
      hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  (void)attr;
  const int64_t tiles = (a.M + BM - 1) / BM * (a.N / BN);
  hipLaunchKernelGGL((gemm_split_kernel<MODE, NORM, TM, TN, WM, WN, RING>), dim3((unsigned)tiles),
                     dim3(kGemmThreads), lds, stream, a);
}

// The smallest tile whose workgroups (one per compute unit: their waves hold most of its registers)
// run at once, else the big kernel, whose loop is the fastest (1.6 PFLOP/s) once there is a round
// of tiles for it. Measured (us, the tile taken against its neighbours in this list):
//   M = 120,  K = 1024, N = 3072: 32 x 64 5.1, 32 x 32 (two rounds) 6.6, 64 x 64 6.7, big 16.5
//   M = 480,  K = 1024, N = 3072: 64 x 128 9.1, 64 x 64 (two rounds) 12.5, 128 x 128 13.7, big 16.7
//   M = 1287, K = 768,  N = 768:  64 x 64 6.4, 32 x 64 (two rounds) 9.1, 64 x 128 8.2, big 18.4
//   M = 1920, K = 1024, N = 3072: big 19.3, 128 x 128 (two rounds) 27.0
//   M = 3840, K = 1024, N = 1024: 128 x 128 17.9, 64 x 128 (two rounds) 19.9, big 22.7
constexpr int64_t kOneRound = 256;

// Whether a product makes its own normalised rows: a launch of rmsnorm_bf16_kernel (3 us, little of
// it work) fewer, for each workgroup's read of its rows in fp32 and their norm ahead of its first
// product. That pays with 16 x 32 tiles (two-layer forwards, us: 12 rows at H = 1024 52.6 -> 48.8, 48
// at 768 51.4 -> 46.8); 32-row tiles read twice as much before they start (120 rows at 1024 67.2 without, 69.4
// with).
inline bool gemm_norms(int64_t M, int K, int N) {
  return K <= kNormMaxK && (M + 15) / 16 * (N / 32) <= kOneRound;
}

// norm: A is the RMSNorm of a.Xn (gemm_norms holds), else a.A.
template <int MODE>
void launch_gemm(const GemmArgs& a, hipStream_t stream, bool norm = false) {
  auto fits = [&](int bm, int bn) { return (a.M + bm - 1) / bm * (a.N / bn) <= kOneRound; };
  if constexpr (MODE != kModeResid)
    if (norm) return launch_gemm_split<MODE, true, 1, 2, 1, 1, 4>(a, stream);
  if (fits(16, 32))
    launch_gemm_split<MODE, false, 1, 2, 1, 1, 4>(a, stream);
  else if (fits(32, 32))
    launch_gemm_split<MODE, false, 2, 2, 1, 1, 4>(a, stream);
  else if (fits(32, 64))
    launch_gemm_split<MODE, false, 2, 4, 1, 1, 4>(a, stream);
  else if (fits(64, 64))
    launch_gemm_split<MODE, false, 4, 4, 1, 1, 3>(a, stream);
  else if (fits(64, 128))
    launch_gemm_split<MODE, false, 4, 4, 1, 2, 3>(a, stream);
  else if (fits(128, 128))
    launch_gemm_split<MODE, false, 4, 4, 2, 2, 3>(a, stream);
  else
    launch_gemm_big<MODE>(a, stream);
}

}  // namespace
}  // namespace lilicorr
