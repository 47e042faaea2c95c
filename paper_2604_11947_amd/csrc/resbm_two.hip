// HIP kernels of the two-linears-per-side bottleneck, of the encoder fused into the
// FFN output projection and of the decoder fused into the next block's norm and QKV
// projection, for gfx950, and their C ABI.
//
// Paper: ResBM, Sec. 3.2 (encoder and decoder each two linear layers with a
// non-linearity between them; encoder at the end of stage l, decoder at the
// start of stage l+1, only b crosses the boundary), Eq. 2 and Eq. 5 (the
// encoder's skip keeps columns [0, r) of the attention output).  With the
// intermediate width m:
//     encoder  u = z W1,  b = x_attn P^id + phi(u) W2
//     decoder  v = b W3,  z~ = phi(v) W4
// and the backward steps are the adjoints of these maps.
//
// Every product of those steps is C = A B over bf16 operands with float32
// accumulation, two template switches saying which of A and B is stored
// K-contiguous.  Epilogues: bf16 or float32 store, a store of phi(C) beside C,
// multiplication by phi'(X) of a saved pre-activation (with or without phi(X)
// beside it), addition of identity-path columns, a split-K partial sum, or the
// encoder's contraction of the output tile.  The n x m products (2 T n m flops
// each) are matrix-core bound; the r-wide ones stream a T x m tensor and are
// memory bound.
//
// Three kernels, chosen by rows_for, wide_for and narrow_for: k_gemm_big (256 x
// 256 tiles) and k_gemm_mid (128 x 128) are pipelined (operands straight into LDS,
// counted waits, two wave groups half a phase apart, persistent over tiles);
// k_gemm stages 64 x {32, 64, 128} or 128 x 128 tiles through registers, double
// buffered with one barrier per 64-deep stage, and can apply phi to A on the way.
// Products are v_mfma_f32_16x16x32_bf16 with the B operand in the first slot, so a
// lane's accumulator holds four consecutive columns of one output row.
// K-contiguous operands are staged as [rows][64] and read as 16-byte chunks;
// the others as [64][rows] and read transposed with ds_read_b64_tr_b16.
// Split-K partial sums are added in split order by a second kernel, so every
// result is reproducible bit for bit.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "resbm.h"
#include "resbm_buffer.hpp"
#include "resbm_host.hpp"
#include "resbm_mfma.hpp"

namespace resbm2 {

using resbm::bf16x4;
using resbm::bf16x8;
using resbm::bld16;
using resbm::bld8;
using resbm::bst16;
using resbm::bst8;
using resbm::f32x4;
using resbm::kMaxRange;
using resbm::kOOB;
using resbm::make_rsrc;
using resbm::rsrc_t;

constexpr int KT = 64;  // K depth of one stage

enum Epi : int {
  kEpiBf16 = 0,   // C = rne(acc)
  kEpiF32 = 1,    // C = acc (float32)
  kEpiDphi = 2,   // C = rne(acc * phi'(X))   (X: saved pre-activation, same shape as C)
  kEpiAdd = 3,    // C = rne(acc + X) on columns < x_cols, rne(acc) elsewhere
  kEpiPart = 4,   // partial[split] = acc (float32, M x N contiguous per split)
  kEpiBf16Phi = 5,  // C = rne(acc) and D = rne(phi(acc)) (a pre-activation and its activation)
  kEpiDphiPhi = 7,  // C = rne(acc * phi'(X)) and D = rne(phi(X)) (X as for kEpiDphi)
  kEpiEncode = 6,   // C = rne(acc) (the FFN output z) and D[tile column][row] = C_tile W_e[tile rows]
};

struct GemmArgs {
  int M, N, K;
  const void* A; int64_t lda; int64_t a_bytes;
  const void* B; int64_t ldb; int64_t b_bytes;
  void* C; int64_t ldc; int64_t c_bytes;
  const void* X; int64_t ldx; int64_t x_bytes; int x_cols;
  void* D; int64_t ldd; int64_t d_bytes;
  int kc;  // K per split (a multiple of KT); gridDim.z splits
};

// SiLU, a sigmoid(a) with sigmoid(a) = 1 / (1 + 2^(-a log2 e)) from the
// hardware exp2 and reciprocal (about 1 ulp each).
__device__ __forceinline__ float silu(float a) {
  return a * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-a * 1.44269504088896341f));
}

// SiLU on 8 bf16 values, each result rounded to bf16 (the operand the next
// product consumes).
__device__ __forceinline__ uint4 silu8(uint4 v) {
  bf16x8 h = __builtin_bit_cast(bf16x8, v);
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = (__bf16)silu((float)h[e]);
  return __builtin_bit_cast(uint4, h);
}

// Column permutation of a [KT][I] tile (I a multiple of 128) that is read with
// ds_read_b64_tr_b16: the low four bits of the 8-element chunk index are XORed
// with 2 (row % 4 + 4 ((row / 8) % 2)).  One transposed read of 32 lanes touches
// two adjacent chunks in each of 8 rows (r0 .. r0 + 3 and r0 + 8 .. r0 + 11);
// the XOR values are 8 distinct even numbers, so the 16 chunks land on 16
// distinct 16-byte bank slots.  Chunks stay in their row and 256-byte window,
// so whole-row copies stay conflict-free too.  (An XOR with the row's low four
// bits leaves two rows of each such read on the same banks.)
__device__ __forceinline__ int tr_col(int row, int col) {
  const int f = ((row & 3) | ((row >> 1) & 4)) << 1;
  return ((((col >> 3) ^ f) & 15) | ((col >> 3) & ~15)) << 3 | (col & 7);
}

// Column permutation of a K-contiguous [I][64] tile: the chunk index is XORed
// with (row / 2) % 8.
__device__ __forceinline__ int kc_col(int row, int col) {
  return ((((col >> 3) ^ (row >> 1)) & 7) << 3) | (col & 7);
}

// Position of element (row, col) in a staged tile.  K-contiguous operands are
// staged [I][64] (row = index along M or N, col = k); the others [64][I]
// (row = k, col = index), I = 32, 64 or a multiple of 128.
template <bool KC, int I>
__device__ __forceinline__ int tile_pos(int row, int col) {
  if constexpr (KC) {
    static_assert(KT == 64, "kc_col permutes the 8 chunks of a 64-element row");
    return row * KT + kc_col(row, col);
  } else if constexpr (I % 128 == 0) {
    return row * I + tr_col(row, col);
  } else {
    return row * I + resbm::tile_col<I>(row, col);
  }
}

// Operand fragment for 16 indices starting at i0 and the 32-deep K step kk of
// the staged tile: lane (row16, grp) receives Op[i0 + row16][32 kk + 8 grp + e].
template <bool KC, int I>
__device__ __forceinline__ bf16x8 frag(const __bf16* tile, int i0, int kk, int row16, int grp) {
  if constexpr (KC) {
    return __builtin_bit_cast(bf16x8,
                              *reinterpret_cast<const uint4*>(tile + tile_pos<true, I>(i0 + row16, 32 * kk + 8 * grp)));
  } else {
    // Two ds_read_b64_tr_b16: within a 16-lane group, lane j addresses row
    // 32 kk + 8 grp + 4 q + j / 4, columns i0 + 4 (j % 4) .. + 3, and lane i
    // collects four consecutive rows of column i0 + i.
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    s16x4 h[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int row = 32 * kk + 8 * grp + 4 * q + (row16 >> 2);
      const __bf16* p = tile + tile_pos<false, I>(row, i0 + 4 * (row16 & 3));
      h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)(p));
    }
    return __builtin_bit_cast(bf16x8, (short __attribute__((ext_vector_type(8)))){h[0][0], h[0][1], h[0][2], h[0][3],
                                                                                 h[1][0], h[1][1], h[1][2], h[1][3]});
  }
}

// One operand of a GEMM stage: which 16-byte chunks a thread moves from global
// memory into the staged tile.  NI = extent along M or N (for range checks).
template <bool KC, int I, int NTH>
struct Operand {
  static constexpr int CHUNKS = I * KT / 8;
  static constexpr int PER = CHUNKS / NTH;
  static_assert(CHUNKS % NTH == 0, "tile chunks must divide over the block");
  uint4 r[PER];

  // Chunk c covers 8 elements: K-contiguous (row = c / 8 along I, k = 8 (c % 8));
  // otherwise (row = c / (I / 8) along k, index = 8 (c % (I / 8))).
  __device__ __forceinline__ void load(rsrc_t src, int64_t ld, int i0, int NI, int k0, int kend, int tid) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = tid + NTH * p;
      int idx, k;
      if constexpr (KC) {
        idx = i0 + c / 8;
        k = k0 + 8 * (c % 8);
      } else {
        k = k0 + c / (I / 8);
        idx = i0 + 8 * (c % (I / 8));
      }
      const bool ok = idx < NI && k < kend;
      const int64_t off = KC ? ((int64_t)idx * ld + k) * 2 : ((int64_t)k * ld + idx) * 2;
      r[p] = bld16(src, ok ? (uint32_t)off : kOOB);
    }
  }
  template <bool PHI>
  __device__ __forceinline__ void put(__bf16* tile, int tid) const {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int c = tid + NTH * p;
      const int row = KC ? c / 8 : c / (I / 8);
      const int col = KC ? 8 * (c % 8) : 8 * (c % (I / 8));
      *reinterpret_cast<uint4*>(tile + tile_pos<KC, I>(row, col)) = PHI ? silu8(r[p]) : r[p];
    }
  }
};

// Direct-to-LDS staging of a k-major [64][I] operand tile (buffer loads with the
// LDS destination): wave w of NW moves the 1 KiB blocks p NW + w of the tile, lane l
// filling bytes [16 l, 16 l + 16) of its block, so each lane fetches the chunk
// whose swizzled position that is (tr_col's XOR, its own inverse).  Chunks outside
// [0, NI) x [0, kend) are fetched at kOOB and land as zeros.
template <int I, int NW>
__device__ __forceinline__ void dma_tile(rsrc_t src, int64_t ld, int i0, int NI, int k0, int kend, __bf16* tile,
                                         int wave, int lane) {
  static_assert(I % 128 == 0, "direct staging of a k-major tile needs rows of a multiple of 128");
  constexpr int BLOCKS = I * KT * 2 / 1024;
  static_assert(BLOCKS % NW == 0, "tile blocks must divide over the waves");
#pragma unroll
  for (int p = 0; p < BLOCKS / NW; ++p) {
    const int blk = p * NW + wave;
    const int o = blk * 1024 + lane * 16;
    const int row = o / (I * 2), pc = (o >> 4) % (I / 8);
    const int f = ((row & 3) | ((row >> 1) & 4)) << 1;  // tr_col's XOR
    const int k = k0 + row, idx = i0 + 8 * (((pc ^ f) & 15) | (pc & ~15));
    const bool ok = idx < NI && k < kend;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (__attribute__((address_space(3))) void*)(tile + blk * 512), 16,
                                             ok ? (uint32_t)(((int64_t)k * ld + idx) * 2) : kOOB, 0, 0, 0);
  }
}

// Block index -> tile index.  Consecutive blocks are dispatched to the eight
// XCDs in turn; each XCD is given a contiguous range of tiles, and tile indices
// run along N first, so the tiles resident on one XCD share the rows of A (the
// token stream in the T-row products) through its L2.
__device__ __forceinline__ int xcd_tile(int id, int nb) {
  const int x = id & 7, li = id >> 3;
  return x * (nb >> 3) + min(x, nb & 7) + li;
}

// Fragment-ordered hi/lo bf16 copy of a row-major float32 matrix W (rows x
// cols, row stride ld) for the B slot of a contraction over its rows: fragment
// f = ks * nc + cb, lane (row16, grp) holds W[32 ks + 8 grp + e][16 cb + row16]
// (zeros outside the matrix); per fragment 1 KiB of hi parts, then 1 KiB of lo
// parts.  One block of 64 lanes per fragment.
__global__ __launch_bounds__(64) void k_frag_prep(const float* __restrict__ W, int rows, int cols, int64_t ld, int nc,
                                                  __bf16* __restrict__ out) {
  const int l = threadIdx.x, row16 = l & 15, grp = l >> 4;
  const int f = blockIdx.x;
  const int ks = f / nc, cb = f % nc;
  const int c = 16 * cb + row16;
  bf16x8 hi, lo;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const int j = 32 * ks + 8 * grp + e;
    const float w = (j < rows && c < cols) ? W[(int64_t)j * ld + c] : 0.0f;
    __bf16 h, q;
    resbm::split_hi_lo(w, h, q);
    hi[e] = h;
    lo[e] = q;
  }
  reinterpret_cast<bf16x8*>(out)[(int64_t)(2 * f) * 64 + l] = hi;
  reinterpret_cast<bf16x8*>(out)[(int64_t)(2 * f + 1) * 64 + l] = lo;
}

// Encoder contraction in the epilogue of the FFN output projection (z = h W_down,
// Sec. 3.2 places the encoder right after the feed-forward layer): the block's
// rounded 256 x 256 tile of z goes to LDS (over the stage buffers), and wave w
// multiplies rows 32 w .. 32 w + 31 of it by the tile's 256 rows of W_e
// (float32, as hi + lo bf16 fragments prepared by k_frag_prep, in X), writing
// the float32 partial sum D[tile column][row][0 .. r).  The partials are added
// in tile order by k_enc_finish.  Columns of the tile at or beyond N hold products of
// other W_down elements (HalfSrc::issue) and are staged as zeros: W_e's rows are zero
// there, but an infinity among those products would make 0 x inf of every a.
__device__ __forceinline__ void encode_epilogue(const GemmArgs& g, const f32x4 (&acc)[8][4], __bf16* tile, int m0,
                                                int n0) {
  constexpr int BN = 256;
  const int lane = threadIdx.x & 63, row16 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  __syncthreads();  // every wave has finished reading the last stage
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int ml = (i >> 2) * 128 + wm * 64 + (i & 3) * 16 + row16;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int nl = (j >> 1) * 128 + wn * 32 + (j & 1) * 16 + 4 * grp;
      const bool on = n0 + nl < g.N;  // N % 8 == 0: all four or none
      bf16x4 h;
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = (__bf16)(on ? acc[i][j][e] : 0.0f);
      *reinterpret_cast<uint2*>(tile + ml * 256 + resbm::wide_col(ml, nl)) = __builtin_bit_cast(uint2, h);
    }
  }
  __syncthreads();
  const rsrc_t rw = make_rsrc(g.X, g.x_bytes);
  const int r = g.x_cols, nt = n0 / BN, nc = (r + 63) / 64 * 4;
  const rsrc_t rd = make_rsrc(g.D, g.d_bytes);
  for (int jg = 0; jg < r; jg += 64) {
    f32x4 a2[2][4];
#pragma unroll
    for (int ib = 0; ib < 2; ++ib)
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) a2[ib][jb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 2
    for (int ks = 0; ks < 8; ++ks) {
      bf16x8 zf[2], hi[4], lo[4];
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        const uint32_t off = (uint32_t)((((n0 >> 5) + ks) * nc + (jg >> 4) + jb) * 2048 + lane * 16);
        hi[jb] = __builtin_bit_cast(bf16x8, bld16(rw, off));
        lo[jb] = __builtin_bit_cast(bf16x8, bld16(rw, off + 1024));
      }
#pragma unroll
      for (int ib = 0; ib < 2; ++ib) {
        const int row = 32 * wave + 16 * ib + row16, col = 32 * ks + 8 * grp;
        zf[ib] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(tile + row * 256 + resbm::wide_col(row, col)));
      }
#pragma unroll
      for (int jb = 0; jb < 4; ++jb)
#pragma unroll
        for (int ib = 0; ib < 2; ++ib) {
          a2[ib][jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo[jb], zf[ib], a2[ib][jb], 0, 0, 0);
          a2[ib][jb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi[jb], zf[ib], a2[ib][jb], 0, 0, 0);
        }
    }
    // lane (row16, grp) of (ib, jb) holds D[row][jg + 16 jb + 4 grp .. + 3] of tile row 32 w + 16 ib + row16
#pragma unroll
    for (int ib = 0; ib < 2; ++ib) {
      const int t = m0 + 32 * wave + 16 * ib + row16;
#pragma unroll
      for (int jb = 0; jb < 4; ++jb) {
        const int jj = jg + 16 * jb + 4 * grp;
        const bool ok = t < g.M && jj < r;
        const int64_t off = (((int64_t)nt * g.M + t) * r + jj) * 4;
        bst16(rd, ok ? (uint32_t)off : kOOB, __builtin_bit_cast(uint4, a2[ib][jb]));
      }
    }
  }
}

// ---------------------------------------------------------------- the pipelined core
// The operand tiles of the pipelined kernels are staged in "halves": 128
// indices along M or N by 64 along K (16 KiB), moved straight into LDS by the
// block's 8 waves (two 1 KiB buffer loads per wave and half, LDS destination).
// A K-contiguous half is laid out [128][64] with kc_col's permutation, the
// other [64][128] with tr_col's; each lane fetches the 16-byte chunk whose
// position it fills (both permutations are XORs, their own inverse).
constexpr int kHalf = 128 * KT;  // elements

template <bool KC>
struct HalfSrc {
  uint32_t off[2];   // byte offset of this lane's chunk in the first half, per load
  int k[2];          // its first k within the stage
  uint32_t step;     // bytes from the first half to the second
  __device__ __forceinline__ void init(int64_t ld, int wave, int lane) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int o = (p * 8 + wave) * 1024 + lane * 16;
      if constexpr (KC) {
        const int row = o >> 7, pc = (o >> 4) & 7;
        k[p] = 8 * ((pc ^ (row >> 1)) & 7);  // kc_col's XOR
        off[p] = (uint32_t)((row * ld + k[p]) * 2);
      } else {
        const int row = o >> 8, pc = (o >> 4) & 15;
        const int f = ((row & 3) | ((row >> 1) & 4)) << 1;  // tr_col's XOR
        k[p] = row;
        off[p] = (uint32_t)((row * ld + 8 * (pc ^ f)) * 2);
      }
    }
    step = (uint32_t)(KC ? 256 * ld : 256);
  }
  // Half h of the stage whose descriptor is src, krem the K that is left from
  // the stage's start (chunks at or beyond it become zeros).  Indices past the
  // operand's extent need no test: a K-contiguous row past the last lies outside
  // the descriptor, and a column past the last holds some other element of the
  // operand, which only reaches elements of the tile that are not part of the
  // result: they are not stored, and encode_epilogue leaves them out.
  __device__ __forceinline__ void issue(rsrc_t src, int h, int krem, __bf16* half, int wave) const {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const uint32_t o = k[p] < krem ? off[p] + (h ? step : 0u) : kOOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          src, (__attribute__((address_space(3))) void*)(half + (p * 8 + wave) * 512), 16, o, 0, 0, 0);
    }
  }
};

// Byte offset of this lane's part of fragment (0, 0) in a staged half, for a
// wave whose indices start at w0 (a multiple of 32): see read_frags.
template <bool KC>
__device__ __forceinline__ uint32_t frag_base(int w0, int row16, int grp) {
  if constexpr (KC) {
    return 2u * ((w0 + row16) * KT + ((grp ^ (row16 >> 1)) & 7) * 8);
  } else {
    const int f = (((row16 >> 2) & 3) | ((grp & 1) << 2)) << 1;
    return 2u * ((8 * grp + (row16 >> 2)) * 128 + (((w0 >> 3) + ((row16 & 3) >> 1)) ^ f) * 8 + 4 * (row16 & 1));
  }
}

// Fragments f[i][kk] (indices w0 + 16 i .. + 15, 32-deep K step kk) of the half
// OFF bytes past the one that `a` (an LDS byte address, frag_base included)
// points into, with the wait for them.  The reads are one asm block because
// the compiler, seeing them beside the buffer loads that fill other halves,
// waits for those loads too (vmcnt(6) where 12 may stay in flight).
typedef long i64x2 __attribute__((ext_vector_type(2)));
template <bool KC, int OFF>
__device__ __forceinline__ void read_frags4(bf16x8 (&f)[4][2], uint32_t a) {
  if constexpr (KC) {
    const uint32_t b = a ^ 64;
    asm volatile(
        "ds_read_b128 %0, %8 offset:%10\n\tds_read_b128 %1, %9 offset:%10\n\t"
        "ds_read_b128 %2, %8 offset:%11\n\tds_read_b128 %3, %9 offset:%11\n\t"
        "ds_read_b128 %4, %8 offset:%12\n\tds_read_b128 %5, %9 offset:%12\n\t"
        "ds_read_b128 %6, %8 offset:%13\n\tds_read_b128 %7, %9 offset:%13\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[1][0]), "=&v"(f[1][1]), "=&v"(f[2][0]), "=&v"(f[2][1]),
          "=&v"(f[3][0]), "=&v"(f[3][1])
        : "v"(a), "v"(b), "n"(OFF), "n"(OFF + 2048), "n"(OFF + 4096), "n"(OFF + 6144)
        : "memory");
  } else {
    const uint32_t b = a ^ 32, c = a ^ 64, d = a ^ 96;
    long h[4][4];
    asm volatile(
        "ds_read_b64_tr_b16 %0, %16 offset:%20\n\tds_read_b64_tr_b16 %1, %16 offset:%21\n\t"
        "ds_read_b64_tr_b16 %2, %16 offset:%22\n\tds_read_b64_tr_b16 %3, %16 offset:%23\n\t"
        "ds_read_b64_tr_b16 %4, %17 offset:%20\n\tds_read_b64_tr_b16 %5, %17 offset:%21\n\t"
        "ds_read_b64_tr_b16 %6, %17 offset:%22\n\tds_read_b64_tr_b16 %7, %17 offset:%23\n\t"
        "ds_read_b64_tr_b16 %8, %18 offset:%20\n\tds_read_b64_tr_b16 %9, %18 offset:%21\n\t"
        "ds_read_b64_tr_b16 %10, %18 offset:%22\n\tds_read_b64_tr_b16 %11, %18 offset:%23\n\t"
        "ds_read_b64_tr_b16 %12, %19 offset:%20\n\tds_read_b64_tr_b16 %13, %19 offset:%21\n\t"
        "ds_read_b64_tr_b16 %14, %19 offset:%22\n\tds_read_b64_tr_b16 %15, %19 offset:%23\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(h[0][0]), "=&v"(h[0][1]), "=&v"(h[0][2]), "=&v"(h[0][3]), "=&v"(h[1][0]), "=&v"(h[1][1]),
          "=&v"(h[1][2]), "=&v"(h[1][3]), "=&v"(h[2][0]), "=&v"(h[2][1]), "=&v"(h[2][2]), "=&v"(h[2][3]),
          "=&v"(h[3][0]), "=&v"(h[3][1]), "=&v"(h[3][2]), "=&v"(h[3][3])
        : "v"(a), "v"(b), "v"(c), "v"(d), "n"(OFF), "n"(OFF + 1024), "n"(OFF + 8192), "n"(OFF + 9216)
        : "memory");
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) f[i][kk] = __builtin_bit_cast(bf16x8, (i64x2){h[i][2 * kk], h[i][2 * kk + 1]});
  }
}
template <bool KC, int OFF>
__device__ __forceinline__ void read_frags2(bf16x8 (&f)[2][2], uint32_t a) {
  if constexpr (KC) {
    const uint32_t b = a ^ 64;
    asm volatile(
        "ds_read_b128 %0, %4 offset:%6\n\tds_read_b128 %1, %5 offset:%6\n\t"
        "ds_read_b128 %2, %4 offset:%7\n\tds_read_b128 %3, %5 offset:%7\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(f[0][0]), "=&v"(f[0][1]), "=&v"(f[1][0]), "=&v"(f[1][1])
        : "v"(a), "v"(b), "n"(OFF), "n"(OFF + 2048)
        : "memory");
  } else {
    const uint32_t b = a ^ 32;
    long h[2][4];
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8 offset:%10\n\tds_read_b64_tr_b16 %1, %8 offset:%11\n\t"
        "ds_read_b64_tr_b16 %2, %8 offset:%12\n\tds_read_b64_tr_b16 %3, %8 offset:%13\n\t"
        "ds_read_b64_tr_b16 %4, %9 offset:%10\n\tds_read_b64_tr_b16 %5, %9 offset:%11\n\t"
        "ds_read_b64_tr_b16 %6, %9 offset:%12\n\tds_read_b64_tr_b16 %7, %9 offset:%13\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(h[0][0]), "=&v"(h[0][1]), "=&v"(h[0][2]), "=&v"(h[0][3]), "=&v"(h[1][0]), "=&v"(h[1][1]),
          "=&v"(h[1][2]), "=&v"(h[1][3])
        : "v"(a), "v"(b), "n"(OFF), "n"(OFF + 1024), "n"(OFF + 8192), "n"(OFF + 9216)
        : "memory");
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) f[i][kk] = __builtin_bit_cast(bf16x8, (i64x2){h[i][2 * kk], h[i][2 * kk + 1]});
  }
}

// A block barrier that nothing is scheduled across.
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Work items of a pipelined kernel: (K split, tile) pairs, tiles along N first.
// XCD x (blocks x, x + 8, ...) is given a contiguous range of items, so that
// the items in flight on one XCD share the rows of A through its L2, and its
// blocks walk that range in turn.
struct WorkList {
  int next, end, stride;
  __device__ __forceinline__ void init(int total) {
    const int x = blockIdx.x & 7, li = blockIdx.x >> 3, G = gridDim.x;
    const int begin = x * (total >> 3) + min(x, total & 7);
    end = begin + (total >> 3) + (x < (total & 7) ? 1 : 0);
    stride = (G >> 3) + (x < (G & 7) ? 1 : 0);
    next = begin + li;
  }
};
struct Item {
  int m0, n0, split, kbeg, klen;
};

// Reads the operands of the items in order, one 64-deep stage after another,
// running ahead of the products across item boundaries.
template <bool AK, bool BKC, int BM, int BN>
struct StageCursor {
  HalfSrc<AK> ha;
  HalfSrc<BKC> hb;
  uint32_t oa, ob, sa, sb;  // byte offsets of the next stage, and per stage
  int krem;                 // K left in the item (<= 0: stages of zeros)
  __device__ __forceinline__ void start(const GemmArgs& g, const Item& it) {
    oa = (uint32_t)((AK ? (int64_t)it.m0 * g.lda + it.kbeg : (int64_t)it.kbeg * g.lda + it.m0) * 2);
    ob = (uint32_t)((BKC ? (int64_t)it.n0 * g.ldb + it.kbeg : (int64_t)it.kbeg * g.ldb + it.n0) * 2);
    krem = it.klen;
  }
  __device__ __forceinline__ void init(const GemmArgs& g, int wave, int lane) {
    ha.init(g.lda, wave, lane);
    hb.init(g.ldb, wave, lane);
    sa = (uint32_t)((AK ? KT : KT * g.lda) * 2);
    sb = (uint32_t)((BKC ? KT : KT * g.ldb) * 2);
  }
  __device__ __forceinline__ rsrc_t desc(const void* p, int64_t bytes, uint32_t o) const {
    return __builtin_amdgcn_make_buffer_rsrc((char*)const_cast<void*>(p) + (krem > 0 ? o : 0u), (short)0,
                                             krem > 0 ? (uint32_t)bytes - o : 0u, 0x00020000);
  }
  __device__ __forceinline__ rsrc_t a(const GemmArgs& g) const { return desc(g.A, g.a_bytes, oa); }
  __device__ __forceinline__ rsrc_t b(const GemmArgs& g) const { return desc(g.B, g.b_bytes, ob); }
  __device__ __forceinline__ void advance() {
    oa += sa;
    ob += sb;
    krem -= KT;
  }
};

// The i-th work item's tile and K range.
template <int BM, int BN>
__device__ __forceinline__ Item item_of(const GemmArgs& g, int i) {
  const int tn = (g.N + BN - 1) / BN, tm = (g.M + BM - 1) / BM;
  Item it;
  it.split = i / (tm * tn);
  const int t = i - it.split * (tm * tn);
  it.m0 = t / tn * BM;
  it.n0 = t % tn * BN;
  it.kbeg = it.split * g.kc;
  it.klen = min(g.K, it.kbeg + g.kc) - it.kbeg;
  return it;
}

// The descriptor of the result for a tile that starts at row m0.  A float32 weight
// gradient may take 8 GiB (its bf16 weight up to 4), so its descriptor starts at that
// row; the others cover the whole result: T-row ones and intermediates are below
// 4 GiB by the shape rules, partial sums below 512 x 256 KiB by split_for.
template <int EPI>
__device__ __forceinline__ rsrc_t out_desc(const GemmArgs& g, int m0) {
  const int64_t skip = EPI == kEpiF32 ? (int64_t)m0 * g.ldc * 4 : 0;
  return make_rsrc((const char*)g.C + skip, g.c_bytes - skip);
}

// Stores four consecutive columns n .. n + 3 of row m of the result with the
// epilogue EPI (out of range: dropped).  Offsets of elements in range are below
// 4 GiB, so 32-bit arithmetic is exact for them (kEpiF32: from row m0 on).
template <int EPI>
__device__ __forceinline__ void store_c4(const GemmArgs& g, rsrc_t rc, rsrc_t rx, rsrc_t rd, int split, int m0, int m,
                                         int n, f32x4 v) {
  const bool ok = m < g.M && n < g.N;
  if constexpr (EPI == kEpiF32 || EPI == kEpiPart) {
    const uint32_t off =
        EPI == kEpiPart ? ((uint32_t)split * g.M + m) * g.N + n : (uint32_t)(m - m0) * (uint32_t)g.ldc + n;
    bst16(rc, ok ? off * 4 : kOOB, __builtin_bit_cast(uint4, v));
  } else {
    if constexpr (EPI == kEpiDphi || EPI == kEpiDphiPhi || EPI == kEpiAdd) {
      const bool xok = ok && (EPI != kEpiAdd || n < g.x_cols);
      const uint2 xr = bld8(rx, xok ? ((uint32_t)m * (uint32_t)g.ldx + n) * 2 : kOOB);
      const bf16x4 x = __builtin_bit_cast(bf16x4, xr);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (EPI == kEpiAdd) v[e] += (float)x[e];
        else v[e] *= resbm::silu_grad((float)x[e]);
      }
      if constexpr (EPI == kEpiDphiPhi) {
        bf16x4 p;
#pragma unroll
        for (int e = 0; e < 4; ++e) p[e] = (__bf16)silu((float)x[e]);
        bst8(rd, ok ? ((uint32_t)m * (uint32_t)g.ldd + n) * 2 : kOOB, __builtin_bit_cast(uint2, p));
      }
    }
    bf16x4 h;
#pragma unroll
    for (int e = 0; e < 4; ++e) h[e] = (__bf16)v[e];
    bst8(rc, ok ? ((uint32_t)m * (uint32_t)g.ldc + n) * 2 : kOOB, __builtin_bit_cast(uint2, h));
    if constexpr (EPI == kEpiBf16Phi) {
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = (__bf16)silu(v[e]);  // from the float32 accumulator
      bst8(rd, ok ? ((uint32_t)m * (uint32_t)g.ldd + n) * 2 : kOOB, __builtin_bit_cast(uint2, h));
    }
  }
}

// Stores per lane of one store_pair<EPI>.
constexpr int pair_stores(int epi) { return epi == kEpiF32 || epi == kEpiPart || epi == kEpiBf16Phi || epi == kEpiDphiPhi ? 2 : 1; }

constexpr bool reads_x(int epi) { return epi == kEpiDphi || epi == kEpiDphiPhi || epi == kEpiAdd; }
// X at the eight columns that this lane stores of a pair (see store_pair).
template <int EPI>
__device__ __forceinline__ uint4 load_pair(const GemmArgs& g, rsrc_t rx, int m, int n, int grp) {
  const int c8 = n - 4 * (grp & 1) + 16 * (grp & 1);  // n = ... + 4 grp
  const bool ok = m < g.M && c8 < (EPI == kEpiAdd ? g.x_cols : g.N);
  return bld16(rx, ok ? ((uint32_t)m * (uint32_t)g.ldx + c8) * 2 : kOOB);
}

// Stores two adjacent 16 x 16 tiles: this lane's four columns n .. n + 3 of the
// first and n + 16 .. n + 19 of the second, row m.  bf16 results: lanes of even
// and odd groups exchange halves first, so that each stores eight consecutive
// columns (even groups of the first tile, odd groups of the second): half the
// store instructions, 64 bytes of a row each instead of 32 (the two-linear step at
// 16384 x 4096 x 1024: 872 -> 836 us).  u: what load_pair gave.
template <int EPI>
__device__ __forceinline__ void store_pair(const GemmArgs& g, rsrc_t rc, rsrc_t rd, int split, int m0, int m, int n,
                                           int grp, f32x4 v0, f32x4 v1, uint4 u) {
  if constexpr (EPI == kEpiF32 || EPI == kEpiPart) {
    store_c4<EPI>(g, rc, rc, rd, split, m0, m, n, v0);
    store_c4<EPI>(g, rc, rc, rd, split, m0, m, n + 16, v1);
  } else {
    f32x4 v[2] = {v0, v1};
    const int c8 = n - 4 * (grp & 1) + 16 * (grp & 1);  // n = ... + 4 grp
    const bool ok = m < g.M && c8 < g.N;                // N % 8 == 0: all eight or none
    // (a's odd rows of 16 lanes, b's even rows) change places; its own inverse
    auto swap = [](uint32_t& a, uint32_t& b) {
      const auto x = __builtin_amdgcn_permlane16_swap(a, b, false, false);
      a = x[0];
      b = x[1];
    };
    if constexpr (reads_x(EPI)) {
      if constexpr (EPI == kEpiDphiPhi)
        bst16(rd, ok ? ((uint32_t)m * (uint32_t)g.ldd + c8) * 2 : kOOB, silu8(u));
      swap(u.x, u.z);
      swap(u.y, u.w);
      const bf16x4 x[2] = {__builtin_bit_cast(bf16x4, make_uint2(u.x, u.y)),
                           __builtin_bit_cast(bf16x4, make_uint2(u.z, u.w))};
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (EPI == kEpiAdd) v[p][e] += (float)x[p][e];
          else v[p][e] *= resbm::silu_grad((float)x[p][e]);
        }
    }
    auto put = [&](rsrc_t r, int64_t ld, bf16x4 h0, bf16x4 h1) {
      uint2 a = __builtin_bit_cast(uint2, h0), b = __builtin_bit_cast(uint2, h1);
      swap(a.x, b.x);
      swap(a.y, b.y);
      bst16(r, ok ? ((uint32_t)m * (uint32_t)ld + c8) * 2 : kOOB, make_uint4(a.x, a.y, b.x, b.y));
    };
    bf16x4 h[2];
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int e = 0; e < 4; ++e) h[p][e] = (__bf16)v[p][e];
    put(rc, g.ldc, h[0], h[1]);
    if constexpr (EPI == kEpiBf16Phi) {
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e) h[p][e] = (__bf16)silu(v[p][e]);  // from the float32 accumulator
      put(rd, g.ldd, h[0], h[1]);
    }
  }
}

// Stores a wave's rows mr + row(i), i < FI, and columns nr + 128 q, q < FQ, of a tile at
// (m0, n0).  X is read for G pairs at a time, ahead of their stores: one load in front
// of each store left a chain of round trips, each waiting for the stores before it
// and the stages in flight.  kEpiAdd: only the tiles that hold some of X's columns read it.
// encode2_bwd with the fused skip gradient, m = 16: 4096 x 4096 50.1 -> 41.1 us, 16384 x
// 4096 126 -> 99.7 (a block walks tiles of one column there, and one in 32 had the chain);
// the two-linear step at 16384 x 4096 x 1024: 855 -> 833, timed in turn.
template <int EPI, int FI, int FQ, int NJ>
__device__ __forceinline__ void store_rows(const GemmArgs& g, rsrc_t rc, rsrc_t rx, rsrc_t rd, int split, int m0,
                                           int mr, int nr, int grp, const f32x4 (&acc)[FI][NJ]) {
  constexpr int G = 4;  // pairs
  static_assert(FI * FQ % G == 0 && NJ == 2 * FQ, "groups of pairs cover the tile");
#pragma unroll
  for (int p0 = 0; p0 < FI * FQ; p0 += G) {
    uint4 x[G];
#pragma unroll
    for (int p = 0; p < G; ++p) {
      const int i = (p0 + p) / FQ, q = (p0 + p) % FQ;
      x[p] = make_uint4(0, 0, 0, 0);
      if constexpr (reads_x(EPI)) x[p] = load_pair<EPI>(g, rx, mr + (i >> 2) * 128 + (i & 3) * 16, nr + q * 128, grp);
    }
#pragma unroll
    for (int p = 0; p < G; ++p) {
      const int i = (p0 + p) / FQ, q = (p0 + p) % FQ;
      store_pair<EPI>(g, rc, rd, split, m0, mr + (i >> 2) * 128 + (i & 3) * 16, nr + q * 128, grp, acc[i][2 * q],
                      acc[i][2 * q + 1], x[p]);
    }
  }
}
template <int EPI, int FI, int FQ, int NJ>
__device__ __forceinline__ void store_tile(const GemmArgs& g, rsrc_t rc, rsrc_t rx, rsrc_t rd, const Item& it, int mr,
                                           int nr, int grp, const f32x4 (&acc)[FI][NJ]) {
  if (EPI == kEpiAdd && it.n0 >= g.x_cols)
    store_rows<EPI == kEpiAdd ? kEpiBf16 : EPI, FI, FQ>(g, rc, rx, rd, it.split, it.m0, mr, nr, grp, acc);
  else
    store_rows<EPI, FI, FQ>(g, rc, rx, rd, it.split, it.m0, mr, nr, grp, acc);
}

// The value v, opaque to the optimizer: what an epilogue derives from it is
// formed there, not hoisted out of the loop over work items (the addresses of
// 32 stores would take the registers that the stages need).
__device__ __forceinline__ int here(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// C = A B in 256 x 256 tiles, 8 waves; wave (wm, wn) owns rows 128 h + 64 wm ..
// + 63 and columns 128 q + 32 wn .. + 31 for h, q = 0, 1.  A 64-deep stage is
// four phases, one quadrant (h, q) of 16 products each.  A phase is a load
// section (issue one half of the stage after next into the half that every
// wave finished reading in the phase before, read the 8 or 4 fragments that the
// quadrant lacks, wait for them and for the half that the next phase reads)
// and a product section, each ended by a barrier; waves 4-7 run one section
// behind waves 0-3, so each SIMD has one wave multiplying while the other
// loads.  The stage before a half is read, 6 others are in flight behind it
// (vmcnt(12)); nothing drains.  Stages of even and odd parity take B's halves
// in opposite order, so that a stage's first B half is read in the last phase
// of the stage before and the phases read 8, 4, 8, 4 fragments.
// The stream of stages runs on across work items (K extents padded to an even
// number of stages): the next tile's operands load while this one's results
// are stored.  kEpiEncode reuses the stage buffers and runs one item per block.
// What bounds it: matrix cores at the clock this load allows (a registers-only
// probe of the same products reaches 2.0 PFLOP/s), then the operand stream.
// 16384 x 4096 x 14336 with the encoder: 1.35-1.42 PFLOP/s by box and clocks
// (1400 us; the library's product without the encoder, timed in turn, 1399), against
// 1.17 for the double-buffered kernel it replaced (one barrier and a full drain per
// stage; 1639 us); without the half-phase offset of the waves 0.87 of its rate.
template <bool AK, bool BKC, int EPI>
__global__ __launch_bounds__(512) void k_gemm_big(GemmArgs g, int total) {
  constexpr int BM = 256, BN = 256;
  __shared__ __attribute__((aligned(1024))) __bf16 smem[8 * kHalf];  // [parity][A0 A1 B0 B1]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row16 = lane & 15, grp = lane >> 4;
  const int wm = wave >> 2, wn = wave & 3;

  WorkList wl;
  wl.init(total);
  Item cur = item_of<BM, BN>(g, wl.next);
  StageCursor<AK, BKC, BM, BN> cs;
  cs.init(g, wave, lane);
  cs.start(g, cur);

  f32x4 acc[8][4];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();
  bf16x8 fa[4][2], fb0[2][2], fb1[2][2];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const uint32_t la = lds0 + frag_base<AK>(wm * 64, row16, grp), lb = lds0 + frag_base<BKC>(wn * 32, row16, grp);
  constexpr uint32_t ODD = 8 * kHalf;  // bytes from the even to the odd stage's halves
  constexpr int A0 = 0, A1 = 2 * kHalf, B0 = 4 * kHalf, B1 = 6 * kHalf;
  auto mul = [&](int h, int q, const bf16x8 (&fb)[2][2]) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[4 * h + i][2 * q + j] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][kk], fa[i][kk], acc[4 * h + i][2 * q + j], 0, 0, 0);
  };
  // end of a load section; `st`: the previous item's stores (16 pairs per lane)
  // were issued after the half waited for
  auto loaded = [&](bool st) {
    if (st) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(12 + 16 * pair_stores(EPI)) : "memory");
    else asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    phase_barrier();
  };
  __bf16* const even = smem;
  __bf16* const odd = smem + 4 * kHalf;

  // two stages; the halves of the two stages after them are issued
  auto pair = [&](bool st) {
    {
      const rsrc_t ra = cs.a(g), rb = cs.b(g);
      cs.hb.issue(rb, 0, cs.krem, even + 2 * kHalf, wave);
      read_frags4<AK, A0>(fa, la);
      loaded(st);
      mul(0, 0, fb0);
      phase_barrier();
      cs.ha.issue(ra, 0, cs.krem, even, wave);
      read_frags2<BKC, B1>(fb1, lb);
      loaded(st);
      mul(0, 1, fb1);
      phase_barrier();
      cs.hb.issue(rb, 1, cs.krem, even + 3 * kHalf, wave);
      read_frags4<AK, A1>(fa, la);
      loaded(st);
      mul(1, 1, fb1);
      phase_barrier();
      cs.ha.issue(ra, 1, cs.krem, even + kHalf, wave);
      read_frags2<BKC, B1>(fb1, lb + ODD);
      loaded(st);
      mul(1, 0, fb0);
      phase_barrier();
      cs.advance();
    }
    {
      const rsrc_t ra = cs.a(g), rb = cs.b(g);
      cs.hb.issue(rb, 1, cs.krem, odd + 3 * kHalf, wave);
      read_frags4<AK, A0>(fa, la + ODD);
      loaded(st);
      mul(0, 1, fb1);
      phase_barrier();
      cs.ha.issue(ra, 0, cs.krem, odd, wave);
      read_frags2<BKC, B0>(fb0, lb + ODD);
      loaded(st);
      mul(0, 0, fb0);
      phase_barrier();
      cs.hb.issue(rb, 0, cs.krem, odd + 2 * kHalf, wave);
      read_frags4<AK, A1>(fa, la + ODD);
      loaded(false);
      mul(1, 0, fb0);
      phase_barrier();
      cs.ha.issue(ra, 1, cs.krem, odd + kHalf, wave);
      read_frags2<BKC, B0>(fb0, lb);
      loaded(false);
      mul(1, 1, fb1);
      phase_barrier();
      cs.advance();
    }
  };

  // stages 0 and 1, in the order in which their halves are read
  {
    const rsrc_t ra = cs.a(g), rb = cs.b(g);
    cs.hb.issue(rb, 0, cs.krem, even + 2 * kHalf, wave);
    cs.ha.issue(ra, 0, cs.krem, even, wave);
    cs.hb.issue(rb, 1, cs.krem, even + 3 * kHalf, wave);
    cs.ha.issue(ra, 1, cs.krem, even + kHalf, wave);
    cs.advance();
  }
  {
    const rsrc_t ra = cs.a(g), rb = cs.b(g);
    cs.hb.issue(rb, 1, cs.krem, odd + 3 * kHalf, wave);
    cs.ha.issue(ra, 0, cs.krem, odd, wave);
    cs.hb.issue(rb, 0, cs.krem, odd + 2 * kHalf, wave);
    cs.ha.issue(ra, 1, cs.krem, odd + kHalf, wave);
    cs.advance();
  }
  asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
  phase_barrier();
  read_frags2<BKC, B0>(fb0, lb);
  phase_barrier();
  if (wm == 1) phase_barrier();  // waves 4-7 run one section behind

  const rsrc_t rx = make_rsrc(g.X, g.x_bytes), rd = make_rsrc(g.D, g.d_bytes);
  bool stored = false;
  for (;;) {
    const int npair = (cur.klen + 2 * KT - 1) / (2 * KT);
    wl.next += wl.stride;
    const bool more = wl.next < wl.end;
    Item nxt = cur;
    if (more) nxt = item_of<BM, BN>(g, wl.next);
    // before the last pair the cursor goes on to the next item (or to stages of zeros)
    auto go_on = [&]() {
      if (more) cs.start(g, nxt);
      else cs.krem = 0;
    };
    for (int p = 0; p < npair; ++p) {
      if (p == npair - 1) go_on();
      pair(stored && p == 0);
    }
    if constexpr (EPI != kEpiEncode) {
      const rsrc_t rc = out_desc<EPI>(g, cur.m0);
      const int mr = here(cur.m0 + wm * 64 + row16), nr = here(cur.n0 + wn * 32 + 4 * grp);
      store_tile<EPI, 8, 2>(g, rc, rx, rd, cur, mr, nr, grp, acc);
    }
    if (EPI == kEpiEncode || !more) break;
    stored = true;
    cur = nxt;
    clear();
  }
  if (wm == 0) phase_barrier();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  if constexpr (EPI == kEpiEncode) {
    const rsrc_t rc = out_desc<EPI>(g, cur.m0);
    store_rows<kEpiBf16, 8, 2>(g, rc, rx, rd, 0, 0, cur.m0 + wm * 64 + row16, cur.n0 + wn * 32 + 4 * grp, grp, acc);
    encode_epilogue(g, acc, smem, cur.m0, cur.n0);
  }
}

// C = A B in 128 x 128 tiles, for results with too few 256 x 256 tiles to fill
// the chip: 8 waves of 64 x 32, one phase of 16 products per 64-deep stage, the
// stages in a ring of four (128 KiB), three in flight; sections, wave offset
// and the stream across items as in k_gemm_big.
template <bool AK, bool BKC, int EPI>
__global__ __launch_bounds__(512) void k_gemm_mid(GemmArgs g, int total) {
  constexpr int BM = 128, BN = 128;
  __shared__ __attribute__((aligned(1024))) __bf16 smem[8 * kHalf];  // [ring][A B]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row16 = lane & 15, grp = lane >> 4;
  const int wm = wave >> 2, wn = wave & 3;

  WorkList wl;
  wl.init(total);
  Item cur = item_of<BM, BN>(g, wl.next);
  StageCursor<AK, BKC, BM, BN> cs;
  cs.init(g, wave, lane);
  cs.start(g, cur);
  // the item that the cursor is on: stages left to issue, and the item after it
  int left = (cur.klen + KT - 1) / KT;
  int ahead = wl.next;

  f32x4 acc[4][2];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();
  bf16x8 fa[4][2], fb[2][2];
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
  const uint32_t la = lds0 + frag_base<AK>(wm * 64, row16, grp), lb = lds0 + frag_base<BKC>(wn * 32, row16, grp);
  auto issue = [&](int slot) {
    __bf16* const p = smem + slot * 2 * kHalf;
    const rsrc_t ra = cs.a(g), rb = cs.b(g);
    cs.ha.issue(ra, 0, cs.krem, p, wave);
    cs.hb.issue(rb, 0, cs.krem, p + kHalf, wave);
    cs.advance();
    if (--left == 0) {  // on to the next item, or to stages of zeros
      ahead += wl.stride;
      if (ahead < wl.end) {
        const Item it = item_of<BM, BN>(g, ahead);
        cs.start(g, it);
        left = (it.klen + KT - 1) / KT;
      } else {
        cs.krem = 0;
        left = 1;  // stays dead: krem only falls, `ahead` stays past the end
      }
    }
  };
  issue(0);
  issue(1);
  issue(2);
  asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  phase_barrier();
  if (wm == 1) phase_barrier();  // waves 4-7 run one section behind

  const rsrc_t rx = make_rsrc(g.X, g.x_bytes), rd = make_rsrc(g.D, g.d_bytes);
  int slot = 0;
  bool stored = false;
  for (;;) {
    const int nst = (cur.klen + KT - 1) / KT;
    for (int s = 0; s < nst; ++s) {
      issue((slot + 3) & 3);
      const uint32_t o = slot * 4 * kHalf;
      read_frags4<AK, 0>(fa, la + o);
      read_frags2<BKC, 2 * kHalf>(fb, lb + o);
      // the next stage has landed; 4 pairs' stores follow it after an item's end
      if (stored && s < 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 + 4 * pair_stores(EPI)) : "memory");
      else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
      phase_barrier();
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j][kk], fa[i][kk], acc[i][j], 0, 0, 0);
      phase_barrier();
      slot = (slot + 1) & 3;
    }
    const rsrc_t rc = out_desc<EPI>(g, cur.m0);
    const int mr = here(cur.m0 + wm * 64 + row16), nr = here(cur.n0 + wn * 32 + 4 * grp);
    store_tile<EPI, 4, 1>(g, rc, rx, rd, cur, mr, nr, grp, acc);
    wl.next += wl.stride;
    if (wl.next >= wl.end) break;
    stored = true;
    cur = item_of<BM, BN>(g, wl.next);
    clear();
  }
  if (wm == 0) phase_barrier();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// C = A B in tiles of 64 x {32, 64, 128} (the r-wide results, and T-row products
// whose 128 x 128 tiles would leave most of the chip idle) or 128 x 128 by four waves,
// staged through registers, double buffered, one barrier per 64-deep stage; PHI_A
// applies SiLU to A's elements as they are staged.
template <bool AK, bool BKC, int BM, int BN, int WM, int WN, int EPI, bool PHI_A>
__global__ __launch_bounds__(64 * WM * WN) void k_gemm(GemmArgs g) {
  constexpr int NTH = 64 * WM * WN;
  constexpr int FM = BM / (16 * WM), FN = BN / (16 * WN);
  static_assert(FM * 16 * WM == BM && FN * 16 * WN == BN, "wave tiling must cover the block tile");
  __shared__ __attribute__((aligned(16))) __bf16 s_a0[BM * KT], s_a1[BM * KT];
  __shared__ __attribute__((aligned(16))) __bf16 s_b0[BN * KT], s_b1[BN * KT];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row16 = lane & 15, grp = lane >> 4;
  const int wm = wave % WM, wn = wave / WM;
  const int tiles_n = (g.N + BN - 1) / BN;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int m0 = (t / tiles_n) * BM, n0 = (t % tiles_n) * BN;
  const int kbeg = blockIdx.z * g.kc, kend = min(g.K, kbeg + g.kc);
  const int nst = (kend - kbeg + KT - 1) / KT;

  const rsrc_t ra = make_rsrc(g.A, g.a_bytes), rb = make_rsrc(g.B, g.b_bytes);

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  auto products_kk = [&](const __bf16* ta, const __bf16* tb, int kk) {
    {
      bf16x8 fa[FM], fb[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) fa[i] = frag<AK, BM>(ta, (wm * FM + i) * 16, kk, row16, grp);
#pragma unroll
      for (int j = 0; j < FN; ++j) fb[j] = frag<BKC, BN>(tb, (wn * FN + j) * 16, kk, row16, grp);
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
  };
  static_assert(KT == 64, "a stage is two 32-deep halves");
  auto products = [&](const __bf16* ta, const __bf16* tb) {
    products_kk(ta, tb, 0);
    products_kk(ta, tb, 1);
  };

  Operand<AK, BM, NTH> opa;
  Operand<BKC, BN, NTH> opb;
  if (nst > 0) {
    opa.load(ra, g.lda, m0, g.M, kbeg, kend, tid);
    opb.load(rb, g.ldb, n0, g.N, kbeg, kend, tid);
    opa.template put<PHI_A>(s_a0, tid);
    opb.template put<false>(s_b0, tid);
  }
  __syncthreads();
  for (int s = 0; s < nst; ++s) {
    const bool more = s + 1 < nst;
    if (more) {
      opa.load(ra, g.lda, m0, g.M, kbeg + (s + 1) * KT, kend, tid);
      opb.load(rb, g.ldb, n0, g.N, kbeg + (s + 1) * KT, kend, tid);
    }
    products(s & 1 ? s_a1 : s_a0, s & 1 ? s_b1 : s_b0);
    if (more) {
      opa.template put<PHI_A>(s & 1 ? s_a0 : s_a1, tid);
      opb.template put<false>(s & 1 ? s_b0 : s_b1, tid);
    }
    __syncthreads();
  }

  // lane (row16, grp) of tile (i, j) holds C[m][n .. n + 3]
  const rsrc_t rc = out_desc<EPI>(g, m0);
  const rsrc_t rx = make_rsrc(g.X, g.x_bytes);
  const rsrc_t rd = make_rsrc(g.D, g.d_bytes);
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
      store_c4<EPI>(g, rc, rx, rd, blockIdx.z, m0, m0 + (wm * FM + i) * 16 + row16, n0 + (wn * FN + j) * 16 + 4 * grp,
                    acc[i][j]);
}

// ---------------------------------------------------------------- decoder into RMSNorm + QKV
// out = RMSNorm(b W_d) W_qkv.  RMSNorm scales rows of b W_d and its columns (by
// gamma), so with s_t the row scale
//     out[t] = s_t (b[t] W_d diag(gamma)) W_qkv = s_t b[t] M,   M = W_d diag(gamma) W_qkv  (r x N):
// contracting the weights first takes 2 r (n N + T N) operations instead of
// 2 T n N, and the T x n rows of z~ gamma are never rounded to bf16.  What is
// left is one read of W_qkv and one write of out (1024 x 4096 x 6144, r = 32:
// 63 MB).  M is formed again in every call, strip by strip, in the blocks that
// use it; the row scales come from z~ itself, in float32.
struct DqArgs {
  int T, n, N, r;
  const __bf16* b;       // T x r
  const float* W_d;      // r x n
  const float* gamma;    // n
  const __bf16* W;       // n x N, row-major
  int64_t w_bytes;
  float* ssq;            // [ncg][T] sums of squares of z~ over groups of `cols` columns
  int ncg, cols;         // cols a multiple of 512
  __bf16* wf;            // W_d diag(gamma), hi and lo fragments of the first npre 64-row units
  int npre;
  __bf16* out;           // T x N, row stride ld_out
  int64_t ld_out, out_bytes;
  float eps;
  int rows;              // rows of out per block (a multiple of 16)
};
constexpr int kScRows = 1024;  // row scales held in LDS at a time (a multiple of 256)

// W_d[j][k .. k + 7] gamma[k .. k + 7] (zeros at rows >= r) as hi + lo parts: the
// operand of M, lane (row16, grp) with j = 16 jt + row16, k = k0 + 8 grp.
__device__ __forceinline__ resbm::SFragB wd_gamma(const DqArgs& g, int j, int k) {
  float w[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  if (j < g.r) {
    const float4* p = reinterpret_cast<const float4*>(g.W_d + (int64_t)j * g.n + k);
    const float4* q = reinterpret_cast<const float4*>(g.gamma + k);
    const float4 a = p[0], b = p[1], x = q[0], y = q[1];
    w[0] = a.x * x.x; w[1] = a.y * x.y; w[2] = a.z * x.z; w[3] = a.w * x.w;
    w[4] = b.x * y.x; w[5] = b.y * y.y; w[6] = b.z * y.z; w[7] = b.w * y.w;
  }
  resbm::SFragB f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    __bf16 h, l;
    resbm::split_hi_lo(w[e], h, l);
    f.hi[e] = h;
    f.lo[e] = l;
  }
  return f;
}

// What k_qkv_strip needs of W_d.  blockIdx.y < ncg: sums of squares of z~ over
// one column group for 64 tokens (a wave takes 64 columns at a time, W_d as hi
// and lo: two products).  blockIdx.y == ncg: the fragments, a wave each
// (fragment f = (2 unit + ks) 2 KS + jt: 1 KiB of hi parts, 1 KiB of lo parts).
template <int KS>
__global__ __launch_bounds__(512) void k_qkv_prep(DqArgs g) {
  constexpr int JT = 2 * KS;
  __shared__ float s_q[8][64];
  const int lane = threadIdx.x & 63, row16 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if ((int)blockIdx.y == g.ncg) {
    for (int f = blockIdx.x * 8 + wave; f < g.npre * 2 * JT; f += gridDim.x * 8) {
      const resbm::SFragB w = wd_gamma(g, 16 * (f % JT) + row16, 32 * (f / JT) + 8 * grp);
      reinterpret_cast<bf16x8*>(g.wf)[(int64_t)(2 * f) * 64 + lane] = w.hi;
      reinterpret_cast<bf16x8*>(g.wf)[(int64_t)(2 * f + 1) * 64 + lane] = w.lo;
    }
    return;
  }
  const int t0 = blockIdx.x * 64;
  const rsrc_t rb = make_rsrc(g.b + (int64_t)t0 * g.r, (int64_t)min(64, g.T - t0) * g.r * 2);
  bf16x8 bf[4][KS];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int j = 32 * ks + 8 * grp;
      bf[mt][ks] = __builtin_bit_cast(
          bf16x8, bld16(rb, j < g.r ? (uint32_t)(((16 * mt + row16) * g.r + j) * 2) : kOOB));
    }
  float q[4] = {0.f, 0.f, 0.f, 0.f};
  const int cend = min(g.n, ((int)blockIdx.y + 1) * g.cols);
  for (int c0 = blockIdx.y * g.cols + 64 * wave; c0 < cend; c0 += 512) {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      resbm::SFragB w[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int j = 32 * ks + 8 * grp + e, c = c0 + 16 * ct + row16;  // n % 64 == 0: c < n
          __bf16 h, l;
          resbm::split_hi_lo(j < g.r ? g.W_d[(int64_t)j * g.n + c] : 0.0f, h, l);
          w[ks].hi[e] = h;
          w[ks].lo[e] = l;
        }
#pragma unroll
      for (int mt = 0; mt < 4; ++mt) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks].lo, bf[mt][ks], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks].hi, bf[mt][ks], acc, 0, 0, 0);
        }
        // lane (row16, grp): z~[t0 + 16 mt + row16][c0 + 16 ct + 4 grp + v]
#pragma unroll
        for (int v = 0; v < 4; ++v) q[mt] = fmaf(acc[v], acc[v], q[mt]);
      }
    }
  }
#pragma unroll
  for (int mt = 0; mt < 4; ++mt) {
    float v = q[mt];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (grp == 0) s_q[wave][16 * mt + row16] = v;
  }
  __syncthreads();
  if (threadIdx.x < 64 && t0 + (int)threadIdx.x < g.T) {
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < 8; ++w) v += s_q[w][threadIdx.x];
    g.ssq[(int64_t)blockIdx.y * g.T + t0 + threadIdx.x] = v;
  }
}

// The columns [c0, c0 + 16 CT) of out for the rows [tb, te) as sums over n of
// z~ gamma (rounded to bf16) times W_qkv: the strips whose part of M is not finite.
// There the order matters.  M[j][c] is an infinity or NaN for every j where one
// weight of the column is infinite, and its sum over j NaN, where the sum over n has
// one infinite term with a sign of its own.  No tiles and no LDS: weights like these
// are an error to be seen in the output, not a load to be fast for.
template <int KS, int CT, int NW>
__device__ __forceinline__ void qkv_direct(const DqArgs& g, int c0, int tb, int te) {
  const int lane = threadIdx.x & 63, row16 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const rsrc_t rb = make_rsrc(g.b, (int64_t)g.T * g.r * 2), ro = make_rsrc(g.out, g.out_bytes);
  const float inv_n = 1.0f / (float)g.n;
  for (int t0 = tb + 16 * wave; t0 < te; t0 += 16 * NW) {
    const int t = t0 + row16;
    bf16x8 bv[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int j = 32 * ks + 8 * grp;
      bv[ks] = __builtin_bit_cast(bf16x8, bld16(rb, t < te && j < g.r ? (uint32_t)(((int64_t)t * g.r + j) * 2) : kOOB));
    }
    f32x4 o[CT];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) o[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int c = 0; c < g.n; c += 32) {
      bf16x8 zg;  // z~[t] gamma at columns c + 16 (e / 4) + 4 grp + e % 4
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          resbm::SFragB w;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const int j = 32 * ks + 8 * grp + e;
            __bf16 hi, lo;
            resbm::split_hi_lo(j < g.r ? g.W_d[(int64_t)j * g.n + c + 16 * h + row16] : 0.0f, hi, lo);
            w.hi[e] = hi;
            w.lo[e] = lo;
          }
          z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.lo, bv[ks], z, 0, 0, 0);
          z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.hi, bv[ks], z, 0, 0, 0);
        }
        const float4 gm = *reinterpret_cast<const float4*>(g.gamma + c + 16 * h + 4 * grp);
        zg[4 * h] = (__bf16)(z[0] * gm.x);
        zg[4 * h + 1] = (__bf16)(z[1] * gm.y);
        zg[4 * h + 2] = (__bf16)(z[2] * gm.z);
        zg[4 * h + 3] = (__bf16)(z[3] * gm.w);
      }
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const int col = c0 + 16 * ct + row16;
        bf16x8 w;
#pragma unroll
        for (int e = 0; e < 8; ++e)
          w[e] = col < g.N ? g.W[(int64_t)(c + 16 * (e >> 2) + 4 * grp + (e & 3)) * g.N + col] : (__bf16)0.0f;
        o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, zg, o[ct], 0, 0, 0);
      }
    }
    float q = 0.0f;
    for (int k = 0; k < g.ncg; ++k) q += t < te ? g.ssq[(int64_t)k * g.T + t] : 0.0f;
    const float sc = 1.0f / sqrtf(q * inv_n + g.eps);
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {  // lane (row16, grp): out[t][c0 + 16 ct + 4 grp + v]
      const int col = c0 + 16 * ct + 4 * grp;
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = (__bf16)(o[ct][e] * sc);
      bst8(ro, t < te && col < g.N ? (uint32_t)(((int64_t)t * g.ld_out + col) * 2) : kOOB, __builtin_bit_cast(uint2, v));
    }
  }
}

// Columns [16 CT blockIdx.x, ...) of out for g.rows tokens.  The NW waves take
// the 64-row units of W_qkv in turn: a unit goes through the wave's own LDS
// tile and is read back transposed, W_d gamma (hi and lo: two products) comes
// from the cache in fragment order (or, behind the units that the workspace
// holds, is split here); the next units' loads are in flight meanwhile (two with
// eight waves; one with sixteen, and in 64-column strips at r > 32, whose registers
// hold no more: two spilled 93 there, one 16, 192 -> 163 us at 16384 x 4096 x 6144,
// r = 64).  The waves' parts
// of M meet in LDS in wave order and are kept there as three bf16 planes, which
// hold all 24 bits of the float32 sums: the sum over r that follows may cancel
// (rows of W_d that share a component, a payload orthogonal to it), and with two
// planes the error was then up to 1.4 times that of z~ formed first in float32
// (1.9e-2 against 1.4e-2 of the result where the component is 1000 times the
// differences; three planes 1.4e-2).  Then the waves take 32-row tiles of out in turn.
// Against the 256 x 256 tiles that rebuilt z~ gamma per stage: 158 -> 36.4 us at
// 1024 x 4096 x 6144, r = 32 (37.3 with eight waves instead of sixteen), and
// 973 -> 94 at 16384 rows.  What bounds it: the latency of W_qkv's 64-row units
// at few rows, the writes of out at many.
// (Splitting W_d gamma in every block instead of reading fragments: 43.8 us.)
template <int KS, int CT, int NW>
__global__ __launch_bounds__(64 * NW) void k_qkv_strip(DqArgs g) {
  constexpr int KP = 32 * KS, JT = 2 * KS, WC = 16 * CT, LPR = WC / 8, RPI = 64 / LPR, NQ = 64 / RPI;
  constexpr int STAGE = NW * 64 * WC * 2, PP = KP + 4, PART = NW * WC * PP * 4;
  // units of W_qkv in flight per wave
  constexpr int AHEAD = NW == 8 && KS * CT < 8 ? 2 : 1;
  __shared__ __attribute__((aligned(16))) char smem[STAGE > PART ? STAGE : PART];
  static_assert(3 * WC * KP * 2 <= PART, "the planes of M take the parts' place");
  __shared__ float s_sc[kScRows];
  const int lane = threadIdx.x & 63, row16 = lane & 15, grp = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c0 = xcd_tile(blockIdx.x, gridDim.x) * WC, nu = g.n / 64;
  __bf16* const tile = reinterpret_cast<__bf16*>(smem) + wave * 64 * WC;
  const rsrc_t rw = make_rsrc(g.W, g.w_bytes), rf = make_rsrc(g.wf, (int64_t)g.npre * 4 * JT * 1024);
  const int wrow = lane / LPR, wcol = 8 * (lane % LPR);
  const bool con = c0 + wcol < g.N;

  // scales of the rows [ts, ts + kScRows) of the block's range
  const int tb = blockIdx.y * g.rows, te = min(g.T, tb + g.rows);
  const float inv_n = 1.0f / (float)g.n;
  auto row_scales = [&](int ts) {
    for (int i = threadIdx.x; i < kScRows && ts + i < te; i += 64 * NW) {
      float q = 0.0f;
      for (int k = 0; k < g.ncg; ++k) q += g.ssq[(int64_t)k * g.T + ts + i];
      s_sc[i] = 1.0f / sqrtf(q * inv_n + g.eps);
    }
  };

  uint4 wa[NQ], wb[NQ], dq[2][JT][2];
  auto load_w = [&](uint4 (&wq)[NQ], int u) {
    const bool on = u < nu;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      wq[q] = bld16<2>(rw, on && con ? (uint32_t)(((int64_t)(64 * u + q * RPI + wrow) * g.N + c0 + wcol) * 2) : kOOB);
  };
  auto load_d = [&](int u) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt)
#pragma unroll
        for (int p = 0; p < 2; ++p)
          dq[ks][jt][p] = bld16(rf, u < g.npre ? (uint32_t)(((((2 * u + ks) * JT + jt) * 2 + p) * 64 + lane) * 16) : kOOB);
  };
  f32x4 acc[JT][CT];
#pragma unroll
  for (int jt = 0; jt < JT; ++jt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) acc[jt][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
  // unit u, its rows of W_qkv in wq (reloaded with those of the unit after next;
  // issued behind the next unit's W_d, so that the wait for those leaves them in flight)
  auto unit = [&](uint4 (&wq)[NQ], int u) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int row = q * RPI + wrow;
      *reinterpret_cast<uint4*>(tile + row * WC + resbm::lds_col<WC>(row, wcol)) = wq[q];
    }
    resbm::SFragB d[2][JT];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int jt = 0; jt < JT; ++jt) {
        if (u < g.npre) {
          d[ks][jt].hi = __builtin_bit_cast(bf16x8, dq[ks][jt][0]);
          d[ks][jt].lo = __builtin_bit_cast(bf16x8, dq[ks][jt][1]);
        } else {
          d[ks][jt] = wd_gamma(g, 16 * jt + row16, 64 * u + 32 * ks + 8 * grp);
        }
      }
    load_d(u + NW);
    load_w(wq, u + AHEAD * NW);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the wave's own tile is complete
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int ct = 0; ct < CT; ++ct) {
        const bf16x8 w = resbm::tr_plane<WC>(tile, 32 * ks, 16 * ct, row16, grp);
#pragma unroll
        for (int jt = 0; jt < JT; ++jt) {
          acc[jt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[ks][jt].lo, w, acc[jt][ct], 0, 0, 0);
          acc[jt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(d[ks][jt].hi, w, acc[jt][ct], 0, 0, 0);
        }
      }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read before the next unit overwrites it
  };
  load_w(wa, wave);
  load_d(wave);
  if constexpr (AHEAD == 2) load_w(wb, wave + NW);
  row_scales(tb);  // (read behind the barriers below)
  for (int u = wave; u < nu; u += AHEAD * NW) {
    unit(wa, u);
    if constexpr (AHEAD == 2) {
      if (u + NW < nu) unit(wb, u + NW);
    }
  }
  __syncthreads();  // the parts overlap the tiles
  // lane (row16, grp): part of M[16 jt + 4 grp + v][c0 + 16 ct + row16]
  float* const part = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int jt = 0; jt < JT; ++jt)
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
      *reinterpret_cast<float4*>(part + (wave * WC + 16 * ct + row16) * PP + 16 * jt + 4 * grp) =
          make_float4(acc[jt][ct][0], acc[jt][ct][1], acc[jt][ct][2], acc[jt][ct][3]);
  __syncthreads();
  constexpr int NI = (WC * KP / 4 + 64 * NW - 1) / (64 * NW);
  float m4[NI][4];
  int odd = 0;  // an infinity or NaN among this thread's sums (or one that bf16 rounds to infinity)
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int idx = threadIdx.x + i * 64 * NW, c = idx / (KP / 4), j = 4 * (idx % (KP / 4));
    m4[i][0] = m4[i][1] = m4[i][2] = m4[i][3] = 0.0f;
    if (idx < WC * KP / 4) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float4 p = *reinterpret_cast<const float4*>(part + (w * WC + c) * PP + j);
        m4[i][0] += p.x; m4[i][1] += p.y; m4[i][2] += p.z; m4[i][3] += p.w;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) odd |= !(fabsf(m4[i][e]) < 3.38e38f);
  }
  if (__syncthreads_or(odd)) {  // (a barrier: the planes overlap the parts)
    qkv_direct<KS, CT, NW>(g, c0, tb, te);
    return;
  }
  __bf16* const planes = reinterpret_cast<__bf16*>(smem);
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int idx = threadIdx.x + i * 64 * NW, c = idx / (KP / 4), j = 4 * (idx % (KP / 4));
    if (idx < WC * KP / 4) {
      bf16x4 p[3];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const __bf16 h = (__bf16)m4[i][e];
        const float rest = m4[i][e] - (float)h;  // exact
        const __bf16 q = (__bf16)rest;
        p[0][e] = h;
        p[1][e] = q;
        p[2][e] = (__bf16)(rest - (float)q);
      }
      const int pos = c * KP + resbm::tile_col<KP>(c, j);
#pragma unroll
      for (int k = 0; k < 3; ++k) *reinterpret_cast<uint2*>(planes + k * WC * KP + pos) = __builtin_bit_cast(uint2, p[k]);
    }
  }
  __syncthreads();

  // M as the first operand: row i of tile ct is column expand_col(ct, i), so that
  // a lane ends up with runs of 8 consecutive columns
  bf16x8 m[CT][KS][3];
#pragma unroll
  for (int ct = 0; ct < CT; ++ct)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int c = resbm::expand_col<CT>(0, ct, row16), pos = c * KP + resbm::tile_col<KP>(c, 32 * ks + 8 * grp);
#pragma unroll
      for (int k = 0; k < 3; ++k)
        m[ct][ks][k] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(planes + k * WC * KP + pos));
    }
  const rsrc_t rb = make_rsrc(g.b, (int64_t)g.T * g.r * 2), ro = make_rsrc(g.out, g.out_bytes);
  bf16x8 bn[2][KS];
  auto load_b = [&](int t) {
#pragma unroll
    for (int p = 0; p < 2; ++p)
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int j = 32 * ks + 8 * grp, tp = t + 16 * p;
        bn[p][ks] =
            __builtin_bit_cast(bf16x8, bld16(rb, tp < te && j < g.r ? (uint32_t)(((int64_t)tp * g.r + j) * 2) : kOOB));
      }
  };
  for (int ts = tb; ts < te; ts += kScRows) {
    if (ts > tb) {
      __syncthreads();  // the scales of the rows before are used up
      row_scales(ts);
      __syncthreads();
    }
    const int tl = min(te, ts + kScRows);
    load_b(ts + 32 * wave + row16);
    for (int t0 = ts + 32 * wave; t0 < tl; t0 += 32 * NW) {
      bf16x8 bv[2][KS];
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) bv[p][ks] = bn[p][ks];
      load_b(t0 + 32 * NW + row16);
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        const int t = t0 + 16 * p + row16;
        const float sc = s_sc[t - ts];
        f32x4 o[CT];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
          o[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 2; k >= 0; --k)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
              o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m[ct][ks][k], bv[p][ks], o[ct], 0, 0, 0);
        }
#pragma unroll
        for (int h = 0; h < CT / 2; ++h) {
          const int c = c0 + 32 * h + 8 * grp;
          bf16x8 v;
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = (__bf16)(o[2 * h + (e >> 2)][e & 3] * sc);
          bst16(ro, t < te && c < g.N ? (uint32_t)(((int64_t)t * g.ld_out + c) * 2) : kOOB,
                __builtin_bit_cast(uint4, v));
        }
      }
    }
  }
}

// The other order, for many tokens and a narrow n (see qkv_by_tiles): out on 256 x 256
// tiles (8 waves of 128 x 64, 64-deep stages, double buffered).  The A operand of every stage -- 64 columns
// of z~ for the tile's 256 rows -- is rebuilt in the block instead of read:
// wave w forms rows [32 w, 32 w + 32) of it as b W_d (W_d hi and lo: two
// products per 16 x 16 piece and 32-deep k-step of r), multiplies by gamma and
// rounds to bf16 into the LDS tile; W_qkv streams straight into LDS.  Each wave
// also sums the squares of its rows' float32 z~ over the whole K loop; the row
// scale 1 / sqrt(mean z~^2 + eps) is applied in the epilogue (RMSNorm is a
// per-row scale of z~ gamma).  The rebuild costs 2 KS / 4 of the tile's
// products (W_d as hi + lo, KS = r / 32 rounded up).
template <int KS>
__global__ __launch_bounds__(512) void k_dec_qkv(DqArgs g) {
  constexpr int BM = 256, BN = 256, WM = 2, WN = 4, NW = 8;
  constexpr int FM = BM / (16 * WM), FN = BN / (16 * WN);
  __shared__ __attribute__((aligned(16))) __bf16 s_a0[BM * KT], s_a1[BM * KT];
  __shared__ __attribute__((aligned(16))) __bf16 s_b0[BN * KT], s_b1[BN * KT];
  __shared__ float s_ssq[BM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row16 = lane & 15, grp = lane >> 4;
  const int wm = wave % WM, wn = wave / WM;
  const int tiles_n = (g.N + BN - 1) / BN;
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const int m0 = (t / tiles_n) * BM, n0 = (t % tiles_n) * BN;
  const int nst = g.n / KT;
  const int nc = g.n / 16;

  const rsrc_t rw = make_rsrc(g.W, g.w_bytes);
  const rsrc_t rbr = make_rsrc(g.b + (int64_t)m0 * g.r, (int64_t)max(0, min(BM, g.T - m0)) * g.r * 2);
  const rsrc_t rwd = make_rsrc(g.wf, (int64_t)KS * nc * 2048);
  const rsrc_t rg = make_rsrc(g.gamma, (int64_t)g.n * 4);

  // b rows of this wave's rebuild (the A slot: lane holds b[row][32 ks + 8 grp + e])
  bf16x8 bfr[2][KS];
#pragma unroll
  for (int rb = 0; rb < 2; ++rb)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int row = 32 * wave + 16 * rb + row16, j = 32 * ks + 8 * grp;
      bfr[rb][ks] = __builtin_bit_cast(bf16x8, bld16(rbr, j < g.r ? (uint32_t)((row * g.r + j) * 2) : kOOB));
    }
  // W_d fragments and gamma of a stage, loaded one stage ahead
  struct Wd {
    bf16x8 hi[4][KS], lo[4][KS];
    float4 gm[4];
  };
  auto load_wd = [&](Wd& w, int s) {
    const bool ok = s < nst;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) {
      const int c16 = (s * KT) / 16 + cb;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const int64_t f = (int64_t)ks * nc + c16;
        w.hi[cb][ks] = __builtin_bit_cast(bf16x8, bld16(rwd, ok ? (uint32_t)(((2 * f) * 64 + lane) * 16) : kOOB));
        w.lo[cb][ks] = __builtin_bit_cast(bf16x8, bld16(rwd, ok ? (uint32_t)(((2 * f + 1) * 64 + lane) * 16) : kOOB));
      }
      const uint4 gv = bld16(rg, ok ? (uint32_t)((s * KT + 16 * cb + 4 * grp) * 4) : kOOB);
      w.gm[cb] = make_float4(__builtin_bit_cast(float, gv.x), __builtin_bit_cast(float, gv.y),
                             __builtin_bit_cast(float, gv.z), __builtin_bit_cast(float, gv.w));
    }
  };
  float ssq[2] = {0.f, 0.f};
  // z~ gamma for the stage's 64 columns and the wave's 32 rows, into the A tile
  auto rebuild = [&](const Wd& w, __bf16* a) {
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.hi[cb][ks], bfr[rb][ks], acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w.lo[cb][ks], bfr[rb][ks], acc, 0, 0, 0);
        }
        // lane (row16, grp): z~[row][16 cb + 4 grp + v]
        const float gv[4] = {w.gm[cb].x, w.gm[cb].y, w.gm[cb].z, w.gm[cb].w};
        bf16x4 h;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          ssq[rb] = fmaf(acc[v], acc[v], ssq[rb]);
          h[v] = (__bf16)(acc[v] * gv[v]);
        }
        const int row = 32 * wave + 16 * rb + row16;
        *reinterpret_cast<uint2*>(a + tile_pos<true, BM>(row, 16 * cb + 4 * grp)) = __builtin_bit_cast(uint2, h);
      }
  };

  f32x4 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto products_kk = [&](const __bf16* ta, const __bf16* tb, int kk) {
    bf16x8 fa[FM], fb[FN];
#pragma unroll
    for (int i = 0; i < FM; ++i) fa[i] = frag<true, BM>(ta, (wm * FM + i) * 16, kk, row16, grp);
#pragma unroll
    for (int j = 0; j < FN; ++j) fb[j] = frag<false, BN>(tb, (wn * FN + j) * 16, kk, row16, grp);
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
  };

  Wd wd;
  load_wd(wd, 0);
  // stage 0: its A tile and the B tile
  rebuild(wd, s_a0);
  load_wd(wd, 1);
  dma_tile<BN, NW>(rw, g.N, n0, g.N, 0, g.n, s_b0, wave, lane);
  auto step = [&](int s, const __bf16* a, const __bf16* b, __bf16* na, __bf16* nb) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (s + 1 < nst) {
      dma_tile<BN, NW>(rw, g.N, n0, g.N, (s + 1) * KT, g.n, nb, wave, lane);
      rebuild(wd, na);
      load_wd(wd, s + 2);
    }
    products_kk(a, b, 0);
    products_kk(a, b, 1);
  };
  for (int s = 0; s < nst; s += 2) {
    step(s, s_a0, s_b0, s_a1, s_b1);
    if (s + 1 < nst) step(s + 1, s_a1, s_b1, s_a0, s_b0);
  }

  // row sums of squares: the four lane groups of a row, then one writer per row
#pragma unroll
  for (int rb = 0; rb < 2; ++rb) {
    float v = ssq[rb];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (grp == 0) s_ssq[32 * wave + 16 * rb + row16] = v;
  }
  __syncthreads();

  const rsrc_t ro = make_rsrc(g.out, g.out_bytes);
  const float inv_n = 1.0f / (float)g.n;
#pragma unroll
  for (int i = 0; i < FM; ++i) {
    const int ml = (wm * FM + i) * 16 + row16;
    const int m = m0 + ml;
    const float sc = 1.0f / sqrtf(s_ssq[ml] * inv_n + g.eps);
#pragma unroll
    for (int j = 0; j < FN; ++j) {
      const int n = n0 + (wn * FN + j) * 16 + 4 * grp;
      const bool ok = m < g.T && n < g.N;
      bf16x4 h;
#pragma unroll
      for (int e = 0; e < 4; ++e) h[e] = (__bf16)(acc[i][j][e] * sc);
      bst8(ro, ok ? (uint32_t)(((int64_t)m * g.ld_out + n) * 2) : kOOB, __builtin_bit_cast(uint2, h));
    }
  }
}

// out[i] = sum over s in order of part[s][i], i < count (count % 4 == 0).
__global__ __launch_bounds__(256) void k_splitk_sum(const float* __restrict__ part, int S, int64_t count,
                                                    float* __restrict__ out) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (q * 4 >= count) return;
  const float4* p = reinterpret_cast<const float4*>(part) + q;
  float4 a = p[0];
  for (int s = 1; s < S; ++s) {
    const float4 b = p[(int64_t)s * (count / 4)];
    a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
  }
  reinterpret_cast<float4*>(out)[q] = a;
}

// a = sum over the NT column tiles, in order, of the encoder partials;
// b = rne(x_attn[:, :r] + phi(a)); a_save = a.  4 columns per thread.
__global__ __launch_bounds__(256) void k_enc_finish(int64_t T, int r, int NT, int act, const float* __restrict__ part,
                                                    const __bf16* __restrict__ x, int64_t ld_x, __bf16* __restrict__ b,
                                                    float* __restrict__ a_save) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int per = r / 4;
  if (q >= T * per) return;
  const int64_t t = q / per;
  const int c = (int)(q % per) * 4;
  float4 a = *reinterpret_cast<const float4*>(part + t * r + c);
  for (int k = 1; k < NT; ++k) {
    const float4 p = *reinterpret_cast<const float4*>(part + ((int64_t)k * T + t) * r + c);
    a.x += p.x; a.y += p.y; a.z += p.z; a.w += p.w;
  }
  if (a_save) *reinterpret_cast<float4*>(a_save + t * r + c) = a;
  const bf16x4 xv = __builtin_bit_cast(bf16x4, *reinterpret_cast<const uint2*>(x + t * ld_x + c));
  const float av[4] = {a.x, a.y, a.z, a.w};
  bf16x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = (__bf16)((float)xv[e] + resbm::act_phi(av[e], act));
  *reinterpret_cast<uint2*>(b + t * r + c) = __builtin_bit_cast(uint2, o);
}

// g_x[t][0 .. r) <- rne(g_x + g_b), 4 columns per thread (r % 8 == 0).
__global__ __launch_bounds__(256) void k_skip_grad(int64_t T, int r, const __bf16* __restrict__ g_b,
                                                   __bf16* __restrict__ g_x, int64_t ld_gx) {
  const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int per = r / 4;
  if (q >= T * per) return;
  const int64_t t = q / per;
  const int c = (int)(q % per) * 4;
  const bf16x4 b = __builtin_bit_cast(bf16x4, *reinterpret_cast<const uint2*>(g_b + t * r + c));
  uint2* px = reinterpret_cast<uint2*>(g_x + t * ld_gx + c);
  bf16x4 x = __builtin_bit_cast(bf16x4, *px);
#pragma unroll
  for (int e = 0; e < 4; ++e) x[e] = (__bf16)((float)x[e] + (float)b[e]);
  *px = __builtin_bit_cast(uint2, x);
}

}  // namespace resbm2

// ============================================================ host side
using namespace resbm2;

namespace {

constexpr size_t kWsAlign2 = 256;
constexpr int kNumBlocks = 256;      // compute units: persistent grids, and what split-K aims at

using resbm_host::aligned;
using resbm_host::extent;
using resbm_host::ld_ok;
using resbm_host::overlap;
size_t round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
bool shape_ok2(int64_t T, int n, int m, int r) {
  return T >= 0 && T <= (1ll << 31) && n >= 8 && n <= 65536 && n % 8 == 0 && m >= 8 && m <= 65536 && m % 8 == 0 &&
         r >= 8 && r <= n && r % 8 == 0;
}
bool fits(size_t bytes) { return bytes <= (size_t)kMaxRange; }

// Block tile shapes: 256 x 256 and 128 x 128 (the pipelined kernels), 128 x 128 by
// four waves (64 KiB of LDS: two blocks per unit) and narrow ones.  Products with
// M = r use 128 x 128; the rows beyond r only reach discarded outputs.
enum Shape { kBig = 0, kWide = 1, kNarrow32 = 2, kNarrow64 = 3, kNarrow128 = 4, kFour = 5 };

// Weight gradients: 256 x 256 unless M or N is below it (their token splits
// fill the chip either way).
Shape wide_for(int M, int N) { return M >= 256 && N >= 256 ? kBig : kWide; }
Shape narrow_for(int N) { return N <= 32 ? kNarrow32 : (N <= 64 ? kNarrow64 : kNarrow128); }
// T-row products (no split).  Times below: encode2_fwd with r = 8 and the identity,
// whose second product takes about 3 us; every line compares all the shapes on 800
// random (M, N, K).
//  - N <= 64, or at most 128 tiles of 128 x 128: 64 x 32 and 64 x 64 tiles.  More
//    blocks, and no pipeline to fill: 1 x 8 x 8 5.4 us against 6.6 (128 x 128) and 9.3
//    (256 x 256), 8029 x 256 x 2040 28.5 against 31.0 and 47.7, 22 x 504 x 3984 34.5
//    against 47.5; beyond, their operand traffic costs (57388 x 440 x 472: 73 against 48).
//  - N < 256: tiles as wide as N need the pipelined 128 x 128 kernel up to one round
//    of blocks (23033 x 120 x 2072: 30.4 against 38.2 in narrow tiles), the four-wave
//    one beyond, whose two blocks per unit hold two rounds' tiles at once (53966 x 120 x
//    752: 28.9 against 29.7 and 31.1 in 256 x 256; 19040 x 176 x 152: 12.8, 13.8 and
//    15.1), and 256 x 256 from three rounds on if N > 128 (34600 x 160 x 416: 23.5
//    against 28.0 and 27.0).
//  - else a 64-deep stage of a full round of 256 blocks takes 1.4 us in 256 x 256
//    tiles and 0.7 in 128 x 128 ones (a quarter of the work, twice the operand bytes per
//    product), so the small tiles win where they need fewer than twice the rounds, i.e.
//    where at most 64 large tiles would leave most of the chip idle (1024 x 4096 x
//    14336: 161 against 258 us; 4096 x 4096 x 14336, 256 large tiles: 582 against 343);
//    where half a large tile would be padding; and where there is one stage (a pair of
//    stages is the large tiles' step; 35631 x 464 x 32: 22.2 against 25.1, but from some
//    three rounds of large tiles on those are level or better: 28855 x 3384 x 8 51.0
//    and 51.8, 16384 x 4096 x 32 37.6 and 35.3).
Shape rows_for(int M, int N, int K) {
  const int64_t big = ((int64_t)(M + 255) / 256) * ((N + 255) / 256), mid = ((int64_t)(M + 127) / 128) * ((N + 127) / 128);
  const int64_t rb = (big + kNumBlocks - 1) / kNumBlocks, rm = (mid + kNumBlocks - 1) / kNumBlocks;
  if (N <= 32) return kNarrow32;
  if (N <= 64 || mid <= kNumBlocks / 2) return kNarrow64;
  if (N < 256) return rm <= 1 ? kWide : (N <= 128 || rm <= 2 ? kFour : kBig);
  return K <= KT || M <= 128 || rm < 2 * rb ? kWide : kBig;
}
int shape_bm(Shape s) { return s == kBig ? 256 : (s == kWide || s == kFour ? 128 : 64); }
int shape_bn(Shape s) {
  return s == kBig ? 256 : (s == kWide || s == kFour || s == kNarrow128 ? 128 : (s == kNarrow32 ? 32 : 64));
}

struct Split {
  int S;
  int kc;
};
// Splits of a token-deep (K = T) product: enough blocks to fill the chip, each
// split at least 4 stages deep.
Split split_for(int M, int N, int K, Shape s) {
  const int64_t tiles = (int64_t)((M + shape_bm(s) - 1) / shape_bm(s)) * ((N + shape_bn(s) - 1) / shape_bn(s));
  int64_t S = (kNumBlocks + tiles - 1) / tiles;
  const int64_t maxS = std::max<int64_t>(1, K / (4 * KT));
  S = std::min(S, maxS);
  const int64_t per = (K + S - 1) / S;
  const int kc = (int)round_up((size_t)per, KT);
  return {(int)((K + kc - 1) / kc), kc};
}
size_t part_bytes(int M, int N, const Split& sp) {
  return sp.S > 1 ? round_up((size_t)sp.S * M * N * 4, kWsAlign2) : 0;
}

struct Plan2 {
  Split dW4, dW3, dW2, dW1;
  size_t inter;      // one T x m bf16 intermediate (phi(v), g_v or g_u)
  size_t enc_fwd, dec_fwd, dec_bwd, enc_bwd;
};
Plan2 make_plan2(int64_t T, int n, int m, int r) {
  Plan2 p;
  p.dW4 = split_for(m, n, (int)T, wide_for(m, n));
  p.dW3 = split_for(r, m, (int)T, kWide);
  p.dW2 = split_for(m, r, (int)T, narrow_for(r));
  p.dW1 = split_for(n, m, (int)T, wide_for(n, m));
  p.inter = round_up((size_t)T * m * 2, kWsAlign2);
  p.enc_fwd = p.inter;
  p.dec_fwd = p.inter;
  p.dec_bwd = 2 * p.inter + std::max(part_bytes(m, n, p.dW4), part_bytes(r, m, p.dW3));
  p.enc_bwd = p.inter + std::max(part_bytes(m, r, p.dW2), part_bytes(n, m, p.dW1));
  return p;
}

template <bool AK, bool BKC, int BM, int BN, int WM, int WN, int EPI, bool PHI>
void launch(const GemmArgs& g, int S, hipStream_t st) {
  const int tiles = ((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
  hipLaunchKernelGGL((k_gemm<AK, BKC, BM, BN, WM, WN, EPI, PHI>), dim3(tiles, 1, S), dim3(64 * WM * WN), 0, st, g);
}

// One block per compute unit walks the S * tiles work items of a pipelined
// kernel (kEpiEncode, which has the stage buffers to itself: a block per item).
template <bool AK, bool BKC, int EPI>
void launch_big(const GemmArgs& g, int S, hipStream_t st) {
  const int total = S * ((g.M + 255) / 256) * ((g.N + 255) / 256);
  const int grid = EPI == kEpiEncode ? total : std::min(total, kNumBlocks);
  hipLaunchKernelGGL((k_gemm_big<AK, BKC, EPI>), dim3(grid), dim3(512), 0, st, g, total);
}
template <bool AK, bool BKC, int EPI>
void launch_mid(const GemmArgs& g, int S, hipStream_t st) {
  const int total = S * ((g.M + 127) / 128) * ((g.N + 127) / 128);
  hipLaunchKernelGGL((k_gemm_mid<AK, BKC, EPI>), dim3(std::min(total, kNumBlocks)), dim3(512), 0, st, g, total);
}

// Runs C = op(A) op(B) with the epilogue EPI and tile shape s.  PHI is the dW2
// product's, whose tiles are narrow; 64 x 128 ones are r-wide results only.
template <bool AK, bool BKC, int EPI, bool PHI>
void gemm(Shape s, const GemmArgs& g, int S, hipStream_t st) {
  if constexpr (!PHI) {
    if (s == kBig) return launch_big<AK, BKC, EPI>(g, S, st);
    if (s == kWide) return launch_mid<AK, BKC, EPI>(g, S, st);
    if (s == kFour) return launch<AK, BKC, 128, 128, 2, 2, EPI, false>(g, S, st);
  }
  if constexpr (EPI == kEpiBf16 || EPI == kEpiAdd || EPI == kEpiF32 || EPI == kEpiPart) {
    if (s == kNarrow128) return launch<AK, BKC, 64, 128, 4, 1, EPI, PHI>(g, S, st);
  }
  if (s == kNarrow32) return launch<AK, BKC, 64, 32, 4, 1, EPI, PHI>(g, S, st);
  launch<AK, BKC, 64, 64, 4, 1, EPI, PHI>(g, S, st);
}

GemmArgs args(int M, int N, int K, const void* A, int64_t lda, size_t ab, const void* B, int64_t ldb, size_t bb,
              void* C, int64_t ldc, size_t cb) {
  GemmArgs g{};
  g.M = M; g.N = N; g.K = K;
  g.A = A; g.lda = lda; g.a_bytes = (int64_t)ab;
  g.B = B; g.ldb = ldb; g.b_bytes = (int64_t)bb;
  g.C = C; g.ldc = ldc; g.c_bytes = (int64_t)cb;
  g.kc = (int)round_up((size_t)K, KT);
  return g;
}

// A token-deep weight-gradient product (K = T): float32 result W (M x N,
// contiguous), split over tokens with the partial sums in `part` when that
// fills the chip better.  128 x 128 tiles take the four-wave kernel where its two
// blocks per unit save a second round (decode2_bwd 34580 x 2880 x 40 x 16, 23 tiles
// in 12 splits: 121.7 against 138.8 us; 49261 x 488 x 144 x 8, 256 items: 121.7 against
// 103.9) and where there are at most three stages, too few to fill the pipeline (T =
// 8: 11.5 against 12.5 us; T = 157: 14.7 and 15.5; T = 411: 21.5 and 20.8).
template <bool PHI>
void weight_grad(Shape s, GemmArgs g, const Split& sp, float* W, void* part, hipStream_t st) {
  if (s == kWide && ((int64_t)sp.S * ((g.M + 127) / 128) * ((g.N + 127) / 128) > kNumBlocks || sp.kc <= 3 * KT))
    s = kFour;
  if (sp.S == 1) {
    g.C = W; g.ldc = g.N; g.c_bytes = (int64_t)g.M * g.N * 4;
    gemm<false, false, kEpiF32, PHI>(s, g, 1, st);
    return;
  }
  g.C = part; g.c_bytes = (int64_t)sp.S * g.M * g.N * 4; g.kc = sp.kc;
  gemm<false, false, kEpiPart, PHI>(s, g, sp.S, st);
  const int64_t count = (int64_t)g.M * g.N;
  hipLaunchKernelGGL(k_splitk_sum, dim3((unsigned)((count / 4 + 255) / 256)), dim3(256), 0, st, (const float*)part,
                     sp.S, count, W);
}

// 16-column tiles per strip of decode_qkv_fwd.  32-column strips while out is short
// (more blocks: 37.5 us either way at 1024 x 4096 x 6144, r = 32; 27.6 against 52.4 at
// 300 x 2112 x 4000, r = 64); beyond, 64-column ones write whole 128-byte lines
// (16384 x 4096 x 6144: 94 against 113 us).  Above r = 32 they win later, the narrower
// out is the later (r = 64: 85 and 83 us at 4096 x 4096 x 6144, 137 against 118 at 8192
// rows; r = 48: 50 against 55 at 6000 x 2048 x 4000).
int qkv_ct(int64_t T, int KS) { return T <= (KS == 1 ? 2048 : 8192) ? 2 : 4; }

// Whether decode_qkv_fwd forms z~ gamma first, in 256 x 256 tiles, instead of the
// weights' product in strips of columns.  The workspace holds the row sums of n KS x 8
// tokens (`chunk`); more tokens go in chunks of two launches each, which a narrow n
// makes many, and a strip costs the same few microseconds however narrow n is:
// strips against tiles 1278 and 17 us at 65536 x 64 x 192, r = 32, 357 and 66 at
// 65536 x 256 x 768, 226 and 182 at 120000 x 1024 x 24, r = 64, 14.4 and 10.8 at
// 5 x 64 x 9528, but 36 and 159 at 1024 x 4096 x 6144 and 61 and 158 at 16384 x 1024 x
// 3072.  Both sides in microseconds, fitted to 445 shapes (n = 64 to 2048, T to 130000,
// N = 8 to 48000; 7 and 9 % off at one sigma): the wrong side was at most 11 % slower.
bool qkv_by_tiles(int64_t T, int n, int N, int KS, int64_t chunk) {
  auto rounds = [](int64_t blocks) { return (double)((blocks + kNumBlocks - 1) / kNumBlocks); };
  const double tiles = rounds(((T + 255) / 256) * ((N + 255) / 256)), chunks = (double)((T + chunk - 1) / chunk);
  const int wc = 16 * qkv_ct(std::min(T, chunk), KS);
  const double by_tiles = 8.0 + tiles * (1.1 + n / 64 * (KS == 1 ? 2.2 : 5.4)) + (double)T * N * 6.1e-7;
  const double by_strips = chunks * (9.3 + (KS == 1 ? 0.0 : 4.1) + n * 0.0041 +
                                     (rounds((N + wc - 1) / wc) - 1.0) * (4.7 + n * 0.0061)) +
                           (double)T * (n * (KS == 1 ? 1.6e-7 : 7.1e-7) + N * 7.2e-7);
  return by_tiles < by_strips;
}

template <int KS>
void launch_qkv(const DqArgs& g, int ct, int ranges, hipStream_t st) {
  hipLaunchKernelGGL(k_qkv_prep<KS>, dim3((g.T + 63) / 64, g.ncg + 1), dim3(512), 0, st, g);
  const dim3 grid((g.N + 16 * ct - 1) / (16 * ct), ranges);
  constexpr int NW = KS == 1 ? 16 : 8;
  if (ct == 2) hipLaunchKernelGGL((k_qkv_strip<KS, 2, NW>), grid, dim3(64 * NW), 0, st, g);
  else hipLaunchKernelGGL((k_qkv_strip<KS, 4, 8>), grid, dim3(512), 0, st, g);
}

int32_t check_ws(size_t need, const void* ws, size_t ws_bytes) {
  if (need == 0) return RESBM_OK;
  if (!ws) return RESBM_E_NULL;
  if (!aligned(ws, kWsAlign2)) return RESBM_E_ALIGN;
  return ws_bytes < need ? RESBM_E_WORKSPACE : RESBM_OK;
}

}  // namespace

extern "C" {

size_t resbm2_workspace_bytes(int64_t T, int32_t n, int32_t m, int32_t r) {
  if (!shape_ok2(T, n, m, r) || T == 0) return 0;
  const Plan2 p = make_plan2(T, n, m, r);
  return std::max(std::max(p.enc_fwd, p.dec_fwd), std::max(p.dec_bwd, p.enc_bwd));
}

int32_t resbm2_encode_fwd(int64_t T, int32_t n, int32_t m, int32_t r, int32_t act, const void* x_attn, int64_t ld_x,
                          const void* z, int64_t ld_z, const void* W1, const void* W2, void* b, void* u, void* ws,
                          size_t ws_bytes, void* stream) {
  if (act != RESBM_ACT_IDENTITY && act != RESBM_ACT_SILU) return RESBM_E_ACT;
  if (!shape_ok2(T, n, m, r)) return RESBM_E_SHAPE;
  if (T == 0) return RESBM_OK;
  const bool silu = act == RESBM_ACT_SILU;
  const Plan2 p = make_plan2(T, n, m, r);
  const size_t need = silu ? p.enc_fwd : 0;
  int32_t e = check_ws(need, ws, ws_bytes);
  if (e) return e;
  if (!x_attn || !z || !W1 || !W2 || !b || !u) return RESBM_E_NULL;
  if (!ld_ok(ld_x, n) || !ld_ok(ld_z, n)) return RESBM_E_SHAPE;
  if (!aligned(x_attn, 16) || !aligned(z, 16) || !aligned(W1, 16) || !aligned(W2, 16) || !aligned(b, 16) ||
      !aligned(u, 16))
    return RESBM_E_ALIGN;
  const size_t bx = extent(T, n, ld_x, 2), bz = extent(T, n, ld_z, 2), bw1 = (size_t)n * m * 2,
               bw2 = (size_t)m * r * 2, bb = (size_t)T * r * 2, bu = (size_t)T * m * 2;
  if (!fits(bx) || !fits(bz) || !fits(bu) || !fits(bw1)) return RESBM_E_SHAPE;
  if (overlap(b, bb, x_attn, bx) || overlap(b, bb, z, bz) || overlap(b, bb, W1, bw1) || overlap(b, bb, W2, bw2) ||
      overlap(u, bu, x_attn, bx) || overlap(u, bu, z, bz) || overlap(u, bu, W1, bw1) || overlap(u, bu, W2, bw2) ||
      overlap(u, bu, b, bb) || overlap(ws, need, x_attn, bx) || overlap(ws, need, z, bz) ||
      overlap(ws, need, W1, bw1) || overlap(ws, need, W2, bw2) || overlap(ws, need, b, bb) ||
      overlap(ws, need, u, bu))
    return RESBM_E_ALIAS;
  hipStream_t st = (hipStream_t)stream;
  const int Ti = (int)T;
  // u = z W1  (A = z, K-contiguous; B = W1 [n][m], m-contiguous), and with SiLU
  // also phi(u) (workspace), formed from the float32 accumulator
  GemmArgs g = args(Ti, m, n, z, ld_z, bz, W1, m, bw1, u, m, bu);
  if (silu) {
    g.D = ws; g.ldd = m; g.d_bytes = (int64_t)bu;
    gemm<true, false, kEpiBf16Phi, false>(rows_for(Ti, m, n), g, 1, st);
  } else {
    gemm<true, false, kEpiBf16, false>(rows_for(Ti, m, n), g, 1, st);
  }
  // b = x_attn[:, :r] + phi(u) W2
  g = args(Ti, r, m, silu ? ws : u, m, bu, W2, r, bw2, b, r, bb);
  g.X = x_attn; g.ldx = ld_x; g.x_bytes = (int64_t)bx; g.x_cols = r;
  gemm<true, false, kEpiAdd, false>(narrow_for(r), g, 1, st);
  return resbm_host::launch_status();
}

int32_t resbm2_decode_fwd(int64_t T, int32_t n, int32_t m, int32_t r, int32_t act, const void* b, const void* W3,
                          const void* W4, void* z_tilde, int64_t ld_zt, void* v, void* ws, size_t ws_bytes,
                          void* stream) {
  if (act != RESBM_ACT_IDENTITY && act != RESBM_ACT_SILU) return RESBM_E_ACT;
  if (!shape_ok2(T, n, m, r)) return RESBM_E_SHAPE;
  if (T == 0) return RESBM_OK;
  const bool silu = act == RESBM_ACT_SILU;
  const Plan2 p = make_plan2(T, n, m, r);
  const size_t need = silu ? p.dec_fwd : 0;
  int32_t e = check_ws(need, ws, ws_bytes);
  if (e) return e;
  if (!b || !W3 || !W4 || !z_tilde || !v) return RESBM_E_NULL;
  if (!ld_ok(ld_zt, n)) return RESBM_E_SHAPE;
  if (!aligned(b, 16) || !aligned(W3, 16) || !aligned(W4, 16) || !aligned(z_tilde, 16) || !aligned(v, 16))
    return RESBM_E_ALIGN;
  const size_t bb = (size_t)T * r * 2, bw3 = (size_t)r * m * 2, bw4 = (size_t)m * n * 2,
               bzt = extent(T, n, ld_zt, 2), bv = (size_t)T * m * 2;
  if (!fits(bzt) || !fits(bv) || !fits(bw4)) return RESBM_E_SHAPE;
  if (overlap(z_tilde, bzt, b, bb) || overlap(z_tilde, bzt, W3, bw3) || overlap(z_tilde, bzt, W4, bw4) ||
      overlap(v, bv, b, bb) || overlap(v, bv, W3, bw3) || overlap(v, bv, W4, bw4) || overlap(v, bv, z_tilde, bzt) ||
      overlap(ws, need, b, bb) || overlap(ws, need, W3, bw3) || overlap(ws, need, W4, bw4) ||
      overlap(ws, need, z_tilde, bzt) || overlap(ws, need, v, bv))
    return RESBM_E_ALIAS;
  hipStream_t st = (hipStream_t)stream;
  const int Ti = (int)T;
  // v = b W3, and with SiLU also phi(v) (workspace), formed from the float32 accumulator
  GemmArgs g = args(Ti, m, r, b, r, bb, W3, m, bw3, v, m, bv);
  if (silu) {
    g.D = ws; g.ldd = m; g.d_bytes = (int64_t)bv;
    gemm<true, false, kEpiBf16Phi, false>(rows_for(Ti, m, r), g, 1, st);
  } else {
    gemm<true, false, kEpiBf16, false>(rows_for(Ti, m, r), g, 1, st);
  }
  // z~ = phi(v) W4
  g = args(Ti, n, m, silu ? ws : v, m, bv, W4, n, bw4, z_tilde, ld_zt, bzt);
  gemm<true, false, kEpiBf16, false>(rows_for(Ti, n, m), g, 1, st);
  return resbm_host::launch_status();
}

int32_t resbm2_decode_bwd(int64_t T, int32_t n, int32_t m, int32_t r, int32_t act, const void* b, const void* v,
                          const void* g_zt, int64_t ld_gzt, const void* g_id, int64_t ld_gid, const void* W3,
                          const void* W4, void* g_b, float* dW3, float* dW4, void* ws, size_t ws_bytes,
                          void* stream) {
  if (act != RESBM_ACT_IDENTITY && act != RESBM_ACT_SILU) return RESBM_E_ACT;
  if (!shape_ok2(T, n, m, r)) return RESBM_E_SHAPE;
  if (T == 0) return RESBM_OK;
  const Plan2 p = make_plan2(T, n, m, r);
  int32_t e = check_ws(p.dec_bwd, ws, ws_bytes);
  if (e) return e;
  if (!b || !v || !g_zt || !W3 || !W4 || !g_b || !dW3 || !dW4) return RESBM_E_NULL;
  if (!ld_ok(ld_gzt, n) || (g_id && !ld_ok(ld_gid, n))) return RESBM_E_SHAPE;
  if (!aligned(b, 16) || !aligned(v, 16) || !aligned(g_zt, 16) || (g_id && !aligned(g_id, 16)) ||
      !aligned(W3, 16) || !aligned(W4, 16) || !aligned(g_b, 16) || !aligned(dW3, 16) || !aligned(dW4, 16))
    return RESBM_E_ALIGN;
  const size_t bb = (size_t)T * r * 2, bv = (size_t)T * m * 2, bg = extent(T, n, ld_gzt, 2),
               bid = g_id ? extent(T, n, ld_gid, 2) : 0, bw3 = (size_t)r * m * 2, bw4 = (size_t)m * n * 2,
               bd3 = (size_t)r * m * 4, bd4 = (size_t)m * n * 4;
  if (!fits(bg) || !fits(bid) || !fits(bv) || !fits(bw4) || !fits(p.dec_bwd)) return RESBM_E_SHAPE;
  const void* ins[] = {b, v, g_zt, g_id, W3, W4};
  const size_t inb[] = {bb, bv, bg, bid, bw3, bw4};
  void* outs[] = {g_b, dW3, dW4, ws};
  const size_t outb[] = {bb, bd3, bd4, p.dec_bwd};
  for (int o = 0; o < 4; ++o) {
    for (int i = 0; i < 6; ++i)
      if (overlap(outs[o], outb[o], ins[i], inb[i])) return RESBM_E_ALIAS;
    for (int o2 = o + 1; o2 < 4; ++o2)
      if (overlap(outs[o], outb[o], outs[o2], outb[o2])) return RESBM_E_ALIAS;
  }
  hipStream_t st = (hipStream_t)stream;
  const int Ti = (int)T;
  char* w = (char*)ws;
  void* g_v = w;
  void* pv = w + p.inter;
  void* part = w + 2 * p.inter;
  const bool silu = act == RESBM_ACT_SILU;
  // g_v = (g_zt W4^T) * phi'(v)   (B(k, j) = W4[j][k]: K-contiguous)
  GemmArgs g = args(Ti, m, n, g_zt, ld_gzt, bg, W4, n, bw4, g_v, m, bv);
  if (silu) {
    // and phi(v), from the v that the epilogue reads (16384 x 1024: a launch of 10.8 us)
    g.X = v; g.ldx = m; g.x_bytes = (int64_t)bv;
    g.D = pv; g.ldd = m; g.d_bytes = (int64_t)bv;
    gemm<true, true, kEpiDphiPhi, false>(rows_for(Ti, m, n), g, 1, st);
  } else {
    gemm<true, true, kEpiBf16, false>(rows_for(Ti, m, n), g, 1, st);
  }
  // dW4 = phi(v)^T g_zt   (A(i, k) = phi(v)[k][i], B(k, j) = g_zt[k][j])
  g = args(m, n, Ti, silu ? pv : v, m, bv, g_zt, ld_gzt, bg, nullptr, 0, 0);
  weight_grad<false>(wide_for(m, n), g, p.dW4, dW4, part, st);
  // dW3 = b^T g_v
  g = args(r, m, Ti, b, r, bb, g_v, m, bv, nullptr, 0, 0);
  weight_grad<false>(kWide, g, p.dW3, dW3, part, st);
  // g_b = g_v W3^T + g_id[:, :r]
  g = args(Ti, r, m, g_v, m, bv, W3, m, bw3, g_b, r, bb);
  if (g_id) {
    g.X = g_id; g.ldx = ld_gid; g.x_bytes = (int64_t)bid; g.x_cols = r;
    gemm<true, true, kEpiAdd, false>(narrow_for(r), g, 1, st);
  } else {
    gemm<true, true, kEpiBf16, false>(narrow_for(r), g, 1, st);
  }
  return resbm_host::launch_status();
}

int32_t resbm2_encode_bwd(int64_t T, int32_t n, int32_t m, int32_t r, int32_t act, const void* z, int64_t ld_z,
                          const void* u, const void* g_b, const void* W1, const void* W2, void* g_z, int64_t ld_gz,
                          void* g_x, int64_t ld_gx, float* dW1, float* dW2, void* ws, size_t ws_bytes,
                          void* stream) {
  if (act != RESBM_ACT_IDENTITY && act != RESBM_ACT_SILU) return RESBM_E_ACT;
  if (!shape_ok2(T, n, m, r)) return RESBM_E_SHAPE;
  if (T == 0) return RESBM_OK;
  const Plan2 p = make_plan2(T, n, m, r);
  int32_t e = check_ws(p.enc_bwd, ws, ws_bytes);
  if (e) return e;
  if (!z || !u || !g_b || !W1 || !W2 || !g_z || !dW1 || !dW2) return RESBM_E_NULL;
  if (!ld_ok(ld_z, n) || !ld_ok(ld_gz, n) || (g_x && !ld_ok(ld_gx, n))) return RESBM_E_SHAPE;
  if (!aligned(z, 16) || !aligned(u, 16) || !aligned(g_b, 16) || !aligned(W1, 16) || !aligned(W2, 16) ||
      !aligned(g_z, 16) || (g_x && !aligned(g_x, 16)) || !aligned(dW1, 16) || !aligned(dW2, 16))
    return RESBM_E_ALIGN;
  const bool fused = g_x == g_z;
  if (fused && ld_gx != ld_gz) return RESBM_E_ALIAS;
  const size_t bz = extent(T, n, ld_z, 2), bu = (size_t)T * m * 2, bgb = (size_t)T * r * 2,
               bw1 = (size_t)n * m * 2, bw2 = (size_t)m * r * 2, bgz = extent(T, n, ld_gz, 2),
               bgx = (g_x && !fused) ? extent(T, n, ld_gx, 2) : 0, bd1 = (size_t)n * m * 4,
               bd2 = (size_t)m * r * 4;
  if (!fits(bz) || !fits(bu) || !fits(bgz) || !fits(bgx) || !fits(bw1) || !fits(p.enc_bwd)) return RESBM_E_SHAPE;
  const void* ins[] = {z, u, g_b, W1, W2};
  const size_t inb[] = {bz, bu, bgb, bw1, bw2};
  void* outs[] = {g_z, fused ? nullptr : g_x, dW1, dW2, ws};
  const size_t outb[] = {bgz, bgx, bd1, bd2, p.enc_bwd};
  for (int o = 0; o < 5; ++o) {
    for (int i = 0; i < 5; ++i)
      if (overlap(outs[o], outb[o], ins[i], inb[i])) return RESBM_E_ALIAS;
    for (int o2 = o + 1; o2 < 5; ++o2)
      if (overlap(outs[o], outb[o], outs[o2], outb[o2])) return RESBM_E_ALIAS;
  }
  hipStream_t st = (hipStream_t)stream;
  const int Ti = (int)T;
  char* w = (char*)ws;
  void* g_u = w;
  void* part = w + p.inter;
  const bool silu = act == RESBM_ACT_SILU;
  // g_u = (g_b W2^T) * phi'(u)   (B(k, j) = W2[j][k]: K-contiguous)
  GemmArgs g = args(Ti, m, r, g_b, r, bgb, W2, r, bw2, g_u, m, bu);
  if (silu) {
    g.X = u; g.ldx = m; g.x_bytes = (int64_t)bu;
    gemm<true, true, kEpiDphi, false>(rows_for(Ti, m, r), g, 1, st);
  } else {
    gemm<true, true, kEpiBf16, false>(rows_for(Ti, m, r), g, 1, st);
  }
  // dW2 = phi(u)^T g_b
  g = args(m, r, Ti, u, m, bu, g_b, r, bgb, nullptr, 0, 0);
  if (silu) weight_grad<true>(narrow_for(r), g, p.dW2, dW2, part, st);
  else weight_grad<false>(narrow_for(r), g, p.dW2, dW2, part, st);
  // dW1 = z^T g_u
  g = args(n, m, Ti, z, ld_z, bz, g_u, m, bu, nullptr, 0, 0);
  weight_grad<false>(wide_for(n, m), g, p.dW1, dW1, part, st);
  // g_z = g_u W1^T (+ g_b on columns [0, r) when g_x is g_z)   (B(k, j) = W1[j][k])
  g = args(Ti, n, m, g_u, m, bu, W1, m, bw1, g_z, ld_gz, bgz);
  if (fused) {
    g.X = g_b; g.ldx = r; g.x_bytes = (int64_t)bgb; g.x_cols = r;
    gemm<true, true, kEpiAdd, false>(rows_for(Ti, n, m), g, 1, st);
  } else {
    gemm<true, true, kEpiBf16, false>(rows_for(Ti, n, m), g, 1, st);
    if (g_x) {
      const int64_t cnt = T * (r / 4);
      hipLaunchKernelGGL(k_skip_grad, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, T, r,
                         (const __bf16*)g_b, (__bf16*)g_x, ld_gx);
    }
  }
  return resbm_host::launch_status();
}

// Workspace of the fused encoder: the float32 partial sums (one T x r slice per
// 256 columns of z), then the W_e fragments (k_frag_prep: 256-row tiles, r
// rounded up to 64 columns).
static size_t ffn_part_bytes(int64_t T, int n, int r) {
  return round_up((size_t)((n + 255) / 256) * (size_t)T * r * 4, kWsAlign2);
}
static size_t ffn_frag_count(int n, int r) { return (size_t)((n + 255) / 256 * 8) * (size_t)((r + 63) / 64 * 4); }

size_t resbm_ffn_encode_workspace_bytes(int64_t T, int32_t n, int32_t r) {
  if (T <= 0 || n < 8 || n > 65536 || n % 8 || r < 8 || r > n || r % 8) return 0;
  return ffn_part_bytes(T, n, r) + round_up(ffn_frag_count(n, r) * 2048, kWsAlign2);
}

int32_t resbm_ffn_encode_fwd(int64_t T, int32_t d_ff, int32_t n, int32_t r, int32_t act, const void* h, int64_t ld_h,
                             const void* W_down, const void* x_attn, int64_t ld_x, const float* W_e, void* z,
                             int64_t ld_z, void* b, float* a_save, void* ws, size_t ws_bytes, void* stream) {
  if (act != RESBM_ACT_IDENTITY && act != RESBM_ACT_SILU) return RESBM_E_ACT;
  if (T < 0 || T > (1ll << 31) || d_ff < 8 || d_ff > 262144 || d_ff % 8 || n < 8 || n > 65536 || n % 8 || r < 8 ||
      r > n || r % 8)
    return RESBM_E_SHAPE;
  if (T == 0) return RESBM_OK;
  const size_t need = resbm_ffn_encode_workspace_bytes(T, n, r);
  int32_t e = check_ws(need, ws, ws_bytes);
  if (e) return e;
  if (!h || !W_down || !x_attn || !W_e || !z || !b) return RESBM_E_NULL;
  if (!ld_ok(ld_h, d_ff) || !ld_ok(ld_x, n) || !ld_ok(ld_z, n)) return RESBM_E_SHAPE;
  if (!aligned(h, 16) || !aligned(W_down, 16) || !aligned(x_attn, 16) || !aligned(W_e, 16) || !aligned(z, 16) ||
      !aligned(b, 16) || (a_save && !aligned(a_save, 16)))
    return RESBM_E_ALIGN;
  const size_t bh = extent(T, d_ff, ld_h, 2), bwd = (size_t)d_ff * n * 2, bx = extent(T, n, ld_x, 2),
               bwe = (size_t)n * r * 4, bz = extent(T, n, ld_z, 2), bb = (size_t)T * r * 2,
               ba = a_save ? (size_t)T * r * 4 : 0;
  if (!fits(bh) || !fits(bwd) || !fits(bz) || !fits(need)) return RESBM_E_SHAPE;
  const void* ins[] = {h, W_down, x_attn, W_e};
  const size_t inb[] = {bh, bwd, bx, bwe};
  void* outs[] = {z, b, a_save, ws};
  const size_t outb[] = {bz, bb, ba, need};
  for (int o = 0; o < 4; ++o) {
    for (int i = 0; i < 4; ++i)
      if (overlap(outs[o], outb[o], ins[i], inb[i])) return RESBM_E_ALIAS;
    for (int o2 = o + 1; o2 < 4; ++o2)
      if (overlap(outs[o], outb[o], outs[o2], outb[o2])) return RESBM_E_ALIAS;
  }
  hipStream_t st = (hipStream_t)stream;
  // W_e fragments, then z = h W_down with the encoder partials in the epilogue
  const size_t pb = ffn_part_bytes(T, n, r), nf = ffn_frag_count(n, r);
  char* wf = (char*)ws + pb;
  hipLaunchKernelGGL(k_frag_prep, dim3((unsigned)nf), dim3(64), 0, st, W_e, n, r, (int64_t)r, (r + 63) / 64 * 4,
                     (__bf16*)wf);
  GemmArgs g = args((int)T, n, d_ff, h, ld_h, bh, W_down, n, bwd, z, ld_z, bz);
  g.X = wf; g.x_cols = r; g.x_bytes = (int64_t)(nf * 2048);
  g.D = ws; g.d_bytes = (int64_t)pb;
  launch_big<true, false, kEpiEncode>(g, 1, st);
  const int64_t cnt = T * (r / 4);
  hipLaunchKernelGGL(k_enc_finish, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, T, r, (n + 255) / 256, act,
                     (const float*)ws, (const __bf16*)x_attn, ld_x, (__bf16*)b, a_save);
  return resbm_host::launch_status();
}

size_t resbm_decode_qkv_workspace_bytes(int32_t n, int32_t r) {
  if (n < 64 || n > 65536 || n % 64 || r < 8 || r > 64 || r % 8) return 0;
  return round_up((size_t)((r + 31) / 32) * (n / 16) * 2048, kWsAlign2);
}

int32_t resbm_decode_qkv_fwd(int64_t T, int32_t n, int32_t r, int32_t N, const void* b, const float* W_d,
                             const float* gamma, const void* W_qkv, float eps, void* out, int64_t ld_out, void* ws,
                             size_t ws_bytes, void* stream) {
  if (T < 0 || T > (1ll << 31) - 256 || n < 64 || n > 65536 || n % 64 || r < 8 || r > 64 || r % 8 || N < 8 ||
      N > 262144 || N % 8 || !(eps >= 0.0f))
    return RESBM_E_SHAPE;
  if (T == 0) return RESBM_OK;
  const size_t need = resbm_decode_qkv_workspace_bytes(n, r);
  int32_t e = check_ws(need, ws, ws_bytes);
  if (e) return e;
  if (!b || !W_d || !gamma || !W_qkv || !out) return RESBM_E_NULL;
  if (!ld_ok(ld_out, N)) return RESBM_E_SHAPE;
  if (!aligned(b, 16) || !aligned(W_d, 16) || !aligned(gamma, 16) || !aligned(W_qkv, 16) || !aligned(out, 16))
    return RESBM_E_ALIGN;
  const size_t bb = (size_t)T * r * 2, bwd = (size_t)r * n * 4, bg = (size_t)n * 4, bw = (size_t)n * N * 2,
               bo = extent(T, N, ld_out, 2);
  if (!fits(bw) || !fits(bo) || !fits(bb)) return RESBM_E_SHAPE;
  const void* ins[] = {b, W_d, gamma, W_qkv};
  const size_t inb[] = {bb, bwd, bg, bw};
  for (int i = 0; i < 4; ++i)
    if (overlap(out, bo, ins[i], inb[i]) || overlap(ws, need, ins[i], inb[i])) return RESBM_E_ALIAS;
  if (overlap(out, bo, ws, need)) return RESBM_E_ALIAS;
  hipStream_t st = (hipStream_t)stream;
  // The workspace holds the sums of squares of a chunk of tokens (at most a
  // quarter of it: 8 n tokens, 16 n above r = 32) and, behind them, as many units
  // of W_d's fragments as fit.
  const int KS = (r + 31) / 32;
  const int64_t most = (int64_t)(need / 16) / 64 * 64;
  DqArgs g{};
  g.n = n; g.N = N; g.r = r;
  g.W_d = W_d; g.gamma = gamma;
  g.W = (const __bf16*)W_qkv; g.w_bytes = (int64_t)bw;
  g.ssq = (float*)ws;
  g.ld_out = ld_out;
  g.eps = eps;
  if (qkv_by_tiles(T, n, N, KS, most)) {
    hipLaunchKernelGGL(k_frag_prep, dim3((unsigned)(KS * (n / 16))), dim3(64), 0, st, W_d, r, n, (int64_t)n, n / 16,
                       (__bf16*)ws);
    g.T = (int)T;
    g.b = (const __bf16*)b;
    g.wf = (__bf16*)ws;
    g.out = (__bf16*)out;
    g.out_bytes = (int64_t)bo;
    const unsigned tiles = (unsigned)(((T + 255) / 256) * ((N + 255) / 256));
    if (KS == 1) hipLaunchKernelGGL(k_dec_qkv<1>, dim3(tiles), dim3(512), 0, st, g);
    else hipLaunchKernelGGL(k_dec_qkv<2>, dim3(tiles), dim3(512), 0, st, g);
    return resbm_host::launch_status();
  }
  for (int64_t t0 = 0; t0 < T; t0 += most) {
    g.T = (int)std::min(most, T - t0);
    g.b = (const __bf16*)b + t0 * r;
    g.out = (__bf16*)out + t0 * ld_out;
    g.out_bytes = (int64_t)extent(g.T, N, ld_out, 2);
    for (g.cols = 512;; g.cols *= 2) {
      g.ncg = (n + g.cols - 1) / g.cols;
      if (g.ncg == 1 || (size_t)g.ncg * g.T * 16 <= need) break;
    }
    const size_t sq = round_up((size_t)g.ncg * g.T * 4, kWsAlign2);
    g.wf = (__bf16*)((char*)ws + sq);
    g.npre = (int)std::min<size_t>(n / 64, (need - sq) / (KS * 8192));
    const int ct = qkv_ct(g.T, KS), strips = (N + 16 * ct - 1) / (16 * ct);
    // token ranges: blocks for the whole chip, one per compute unit (two: 74 against 44 us at 1024 rows)
    int ranges = std::max(1, std::min(kNumBlocks / strips, (g.T + 255) / 256));
    g.rows = (int)round_up((size_t)(g.T + ranges - 1) / ranges, 256);
    ranges = (g.T + g.rows - 1) / g.rows;
    if (KS == 1) launch_qkv<1>(g, ct, ranges, st);
    else launch_qkv<2>(g, ct, ranges, st);
  }
  return resbm_host::launch_status();
}

}  // extern "C"
