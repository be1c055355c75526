// Read-only skinny-product passes of a level on the matrix cores (App. A,
// with the OLD power P_j):  X = P_j U_j,  Y^T = V_j^T P_j.
//
// BF16-shadow form (storage FP32): every stored power below the top keeps a
// bfloat16 copy S_j, rewritten by the update pass that adds U_j V_j^T to
// P_j.  k_skinny_bf16 reads the shadow (2 bytes per element) and multiplies
// bfloat16 x bfloat16 with float accumulation (v_mfma_f32_32x32x16_bf16).
// k_skinny_f32 reads the float power itself and multiplies in float
// (v_mfma_f32_32x32x2f32): the FP32 method's products at level ranks where
// the vector units, not HBM, would bound a fused pass; k_skinny16_f32 is
// its 16-column form (v_mfma_f32_16x16x4f32), and k_xprod_f32 forms X alone
// with P loaded straight into the operand registers (no LDS staging).
// All write the partial X / Y layouts of the fused pass, so the common tail
// assembles the next factors; the Gram V_j^T U_j is formed in FP64 apart.
//
// Lane layouts (64 lanes, l = lane, h = l / 32):
//   bf16 32x32x16  A: lane l holds A[l % 32][8 h + e], e = 0..7
//                  B: lane l holds B[8 h + e][l % 32]
//   f32 32x32x2    A: lane l holds A[l % 32][h];  B: B[h][l % 32]
//   both           C: element v of lane l is C[8 (v / 4) + 4 h + v % 4][l % 32]
#include "lv_device.h"

#include <type_traits>

namespace lv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int TCB = 256;   // tile columns
constexpr int CRB = 64;    // rows per LDS chunk
constexpr int SPAD = 8;    // LDS row padding (bf16 elements, keeps 16-byte alignment)

// Compile-time loop: f(std::integral_constant<int, I>) for I = 0 .. N-1, so
// that arrays indexed by I stay in registers.
template <int I, int N, typename F> __device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

__device__ __forceinline__ bf16x8 lds8(const uint16_t* p) {
  return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(p));
}

// Factor entries past column R are the zero padding of the factor blocks.
// Their loads still take place, at column min(c, R - 1), which the row holds:
// a load under a condition becomes a branch of its own, after which the
// compiler waits for it alone, so a run of guarded loads would be served one
// round trip at a time.  fac_clamped is the raw load (prefetches zero the
// padding when they are staged, so that no wait follows the load), and
// fac_or_zero the padded entry.
__device__ __forceinline__ float fac_clamped(const float* __restrict__ row, const int c, const int R) {
  return row[c < R ? c : R - 1];
}
__device__ __forceinline__ float fac_or_zero(const float* __restrict__ row, const int c, const int R) {
  const float v = fac_clamped(row, c, R);
  return c < R ? v : 0.f;
}

// Piece (16 bytes) g of a staged shadow row r sits at g ^ tr_swizzle(r): 4
// pieces further per row, one per group of 4 rows.
__device__ __forceinline__ int tr_swizzle(const int r) { return 4 * (r & 3) | ((r >> 2) & 3); }

// B operand (32x32x16) of rows r0 .. r0 + 15 and columns c0 .. c0 + 31 of a
// staged block with rows of LD values: lanes 16 g .. 16 g + 15 take rows 8 (g /
// 2) .. + 7 of columns 16 (g % 2) .. + 15; lane i of a group addresses row i /
// 4, columns 4 (i % 4) .. + 3 of each 4-row half.
template <int LD> __device__ __forceinline__ bf16x8 tr_operand(uint16_t* s, const int r0, const int c0, const int lane) {
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef short v8s __attribute__((ext_vector_type(8)));
  const int li = lane & 15;
  const int c = c0 + (lane >> 4 & 1) * 16 + li % 4 * 4;
  v4s h[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int r = r0 + 8 * (lane >> 5) + 4 * e + li / 4;
    uint16_t* at = s + r * LD + ((c / 8) ^ tr_swizzle(r)) * 8 + c % 8;
    h[e] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)at);
  }
  return __builtin_bit_cast(bf16x8, (v8s)__builtin_shufflevector(h[0], h[1], 0, 1, 2, 3, 4, 5, 6, 7));
}

// Tile: about tile_rows x 256 columns of S (the slices of a column tile
// interleave by 64-row chunks), walked in chunks through LDS; the next
// chunk or two of S and of V_j are held in registers while the current one
// is used.
// Factor columns are padded with zeros to 32 NB.
//   X: per chunk, wave w forms rows [32 (w % 2), + 32) of the half w / 2 of the
//      tile's columns as two chains, one per quarter; the halves are added a
//      chunk later, (a + b) + (c + d): one partial per (row, column tile).
//   Y: wave w keeps the accumulators of tile columns [64 w, 64 w + 64) for
//      every factor block over all chunks of the tile (K = rows); one
//      partial per (column, row tile).
// The B operand of Y needs 8 consecutive rows of one column: transposed reads.
// n = 7168, R = 32 (103 MB of shadow): 39 us with eight 2-byte reads per Y
// operand and X on two waves, 32 us so.
template <int NB>
__device__ __forceinline__ void skinny_body(const uint16_t* __restrict__ S, const int64_t ldp, const int n_pad,
                                            const int tile_rows, const float* __restrict__ Uj,
                                            const float* __restrict__ Vj, const int W, const int R,
                                            float* __restrict__ partX, float* __restrict__ partY, const int pR,
                                            const int ct, const int rt) {
  constexpr int RP = 32 * NB;
  __shared__ __align__(16) uint16_t sS[CRB * TCB];
  __shared__ __align__(16) uint16_t sUt[RP][TCB + SPAD];
  __shared__ __align__(16) uint16_t sVt[RP][CRB + SPAD];
  __shared__ __align__(16) float sX[2][NB][CRB * 32];   // halves of X

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col0 = ct * TCB;
  // interleaved chunks: slice rt of ns takes chunks rt, rt + ns, ... (CS
  // rows apart), so the grid streams one band of rows at a time
  const int ns = (n_pad + tile_rows - 1) / tile_rows;
  const int CS = ns * CRB;
  const int row0 = rt * CRB;
  const int rend = n_pad;
  const int l32 = lane % 32, lh = lane / 32;
  const int mb = wave & 1, half = wave >> 1;   // X: 32 rows of a chunk, half of the columns
  // chunk staging: thread -> rows tid / 32 + 8 i, 16-byte column group tid % 32
  const int srow = tid / 32, sgrp = tid % 32;

  constexpr int VPT = RP * CRB / 256;   // V_j values staged per thread and chunk
  // NB = 1: two chunks in flight, buffers A and B alternating (a tile may
  // have an odd number of chunks: tile_rows is any multiple of 64 and the
  // last tile may be ragged, so the second chunk of a pair and its fetch are
  // guarded); larger NB: one chunk (the accumulators need the registers)
  constexpr int DEPTH = NB == 1 ? 2 : 1;
  u16x8 preA[CRB / 8], preB[CRB / 8];
  float pvA[VPT], pvB[VPT];
  auto fetch = [&](u16x8 (&pre)[CRB / 8], float (&pv)[VPT], const int r0) {
#pragma unroll
    for (int i = 0; i < CRB / 8; ++i)
      pre[i] = __builtin_nontemporal_load(reinterpret_cast<const u16x8*>(S + (int64_t)(r0 + srow + 8 * i) * ldp + col0 +
                                                                     sgrp * 8));
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int idx = tid + 256 * i;
      const int rr = idx / RP, c = idx % RP;
      pv[i] = fac_clamped(Vj + (int64_t)(r0 + rr) * W, c, R);
    }
  };
  fetch(preA, pvA, row0);
  if constexpr (DEPTH == 2) {
    if (row0 + CS < rend) fetch(preB, pvB, row0 + CS);
  }

  // U_j rows of the tile's columns, transposed: sUt[c][k] = U_j[col0 + k][c]
  batched_stage<RP * TCB / 256, 256, float>(
      tid, RP * TCB, [&](int idx) { const int c = idx % RP; return fac_or_zero(Uj + (int64_t)(col0 + idx / RP) * W, c, R); },
      [&](int idx, float v) { sUt[idx % RP][idx / RP] = bf16_rne(v); });

  v16f yacc[NB][2];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) yacc[a][b][v] = 0.f;

  // piece (4 factor columns) j of a row of the halves
  auto xat = [](const int row, const int j) { return row * 32 + (j ^ ((row >> 1) & 7)) * 4; };
  // X rows of the chunk at r0: both halves
  auto store_x = [&](const int r0) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = (tid + 256 * i) / 8, j = tid % 8, c = nb * 32 + 4 * j;
        if (c >= R) continue;
        const f32x4 x = *reinterpret_cast<const f32x4*>(&sX[0][nb][xat(row, j)]) +
                        *reinterpret_cast<const f32x4*>(&sX[1][nb][xat(row, j)]);
        float* px = partX + ((int64_t)ct * n_pad + r0 + row) * pR + c;
        if (c + 4 <= R) *reinterpret_cast<f32x4*>(px) = x;
        else
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (c + e < R) px[e] = x[e];
      }
  };

  auto chunk = [&](u16x8 (&pre)[CRB / 8], float (&pv)[VPT], const int cr0) {
    __syncthreads();   // the previous chunk is no longer read, its halves of X are there
#pragma unroll
    for (int i = 0; i < CRB / 8; ++i) {
      const int r = srow + 8 * i;
      *reinterpret_cast<u16x8*>(&sS[r * TCB + (sgrp ^ tr_swizzle(r)) * 8]) = pre[i];
    }
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int idx = tid + 256 * i;
      sVt[idx % RP][idx / RP] = bf16_rne(idx % RP < R ? pv[i] : 0.f);
    }
    if (cr0 != row0) store_x(cr0 - CS);
    __syncthreads();
    if (cr0 + DEPTH * CS < rend) fetch(pre, pv, cr0 + DEPTH * CS);

    {
      const int r = mb * 32 + l32;
      const int rat = r * TCB + (lh ^ tr_swizzle(r)) * 8;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        v16f xq[2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int v = 0; v < 16; ++v) xq[q][v] = 0.f;
#pragma unroll 2
        for (int ks = 0; ks < TCB / 64; ++ks)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int c = 16 * ((2 * half + q) * (TCB / 64) + ks);
            xq[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds8(&sUt[nb * 32 + l32][c + 8 * lh]), lds8(sS + (rat ^ c)),
                                                            xq[q], 0, 0, 0);
          }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4 x;
#pragma unroll
          for (int e = 0; e < 4; ++e) x[e] = xq[0][4 * q + e] + xq[1][4 * q + e];
          *reinterpret_cast<f32x4*>(&sX[half][nb][xat(r, 2 * q + lh)]) = x;
        }
      }
    }

    // Y^T += V_chunk^T S_chunk
#pragma unroll
    for (int ks = 0; ks < CRB / 16; ++ks) {
#pragma unroll
      for (int cbi = 0; cbi < 2; ++cbi) {
        const bf16x8 b = tr_operand<TCB>(sS, ks * 16, (2 * wave + cbi) * 32, lane);
#pragma unroll
        for (int nbr = 0; nbr < NB; ++nbr)
          yacc[nbr][cbi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds8(&sVt[nbr * 32 + l32][ks * 16 + 8 * lh]), b,
                                                                   yacc[nbr][cbi], 0, 0, 0);
      }
    }
  };

  int last = row0;
  if constexpr (DEPTH == 2) {
    for (int cr0 = row0; cr0 < rend; cr0 += 2 * CS) {
      chunk(preA, pvA, cr0);
      last = cr0;
      if (cr0 + CS < rend) {
        chunk(preB, pvB, cr0 + CS);
        last = cr0 + CS;
      }
    }
  } else {
    for (int cr0 = row0; cr0 < rend; cr0 += CS) {
      chunk(preA, pvA, cr0);
      last = cr0;
    }
  }
  __syncthreads();
  store_x(last);

#pragma unroll
  for (int nbr = 0; nbr < NB; ++nbr)
#pragma unroll
    for (int cbi = 0; cbi < 2; ++cbi) {
      // values 4 q .. 4 q + 3 of a lane are four consecutive factor columns
      float* py = partY + ((int64_t)rt * n_pad + col0 + (2 * wave + cbi) * 32 + l32) * pR + nbr * 32 + 4 * lh;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = nbr * 32 + 4 * lh + 8 * q;
        if (c + 4 <= R)
          *reinterpret_cast<f32x4*>(py + 8 * q) = f32x4{yacc[nbr][cbi][4 * q], yacc[nbr][cbi][4 * q + 1],
                                                        yacc[nbr][cbi][4 * q + 2], yacc[nbr][cbi][4 * q + 3]};
        else
#pragma unroll
          for (int e = 0; e < 3; ++e)
            if (c + e < R) py[8 * q + e] = yacc[nbr][cbi][4 * q + e];
      }
    }
}

// Two waves per SIMD (two work-groups per CU, which the LDS allows): the
// one-block form would otherwise take 258 registers and run one wave per SIMD.
template <int NB>
__global__ void __launch_bounds__(256, 2) k_skinny_bf16(const SkinnyDesc d) {
  skinny_body<NB>(static_cast<const uint16_t*>(d.src), d.ldp, d.n_pad, d.tile_rows, d.Uj, d.Vj, d.W, d.R, d.partX, d.partY, d.pR, blockIdx.x,
                  blockIdx.y);
}

// Index of the descriptor whose block range holds block b (sorted by
// block_begin, the first at 0).
__device__ __forceinline__ int find_skinny(const SkinnyDesc* __restrict__ ds, int nd, int b) {
  int lo = 0, hi = nd - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (ds[mid].block_begin <= b) lo = mid; else hi = mid - 1;
  }
  return lo;
}

template <int NB>
__global__ void __launch_bounds__(256, 2) k_skinny_bf16_multi(const SkinnyDesc* __restrict__ ds, int nd) {
  const SkinnyDesc d = load_desc(ds, find_skinny(ds, nd, (int)blockIdx.x));
  const int local = (int)blockIdx.x - d.block_begin;
  skinny_body<NB>(static_cast<const uint16_t*>(d.src), d.ldp, d.n_pad, d.tile_rows, d.Uj, d.Vj, d.W, d.R, d.partX, d.partY, d.pR,
                  local % d.nct, local / d.nct);
}


// ---------------------------------------------------------------- ranks from 64
//
// The factors of these ranks are kept in bfloat16 as well, transposed (column
// c of U_j is row c of Ut: n_pad values), so that every matrix-core operand but
// one is 16 consecutive bytes and goes through LDS without conversion.  Y's B
// operand needs 8 consecutive rows of one column: ds_read_b64_tr_b16, which
// hands lane i of 16 the column i of the 4 x 16 block whose 16 pieces of 8
// bytes the lanes address.

// One block: rows [64 (blk % tiles), + 64) of 32 columns of U or V, transposed
// and rounded into Ut / Vt.
__device__ __forceinline__ void fac16_body(const Fac16Desc& d, int blk) {
  __shared__ float t[64][33];
  const int tid = threadIdx.x;
  const int tiles = d.n_pad / 64, cols = d.cols / 32;
  const int row0 = blk % tiles * 64;
  blk /= tiles;
  const bool isv = blk >= cols;
  const int c0 = (isv ? blk - cols : blk) * 32;
  const float* __restrict__ src = d.U + (isv ? (int64_t)d.n_pad * d.W + d.dv : 0) + (int64_t)row0 * d.W + c0;
  uint16_t* __restrict__ dst = d.Ut + (int64_t)((isv ? d.W + d.dv : 0) + c0) * d.n_pad + row0;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int e = tid + 256 * i;
    t[e / 32][e % 32] = src[(int64_t)(e / 32) * d.W + e % 32];
  }
  __syncthreads();
  const int c = tid / 8, r8 = tid % 8 * 8;
  u16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = bf16_rne(t[r8 + e][c]);
  *reinterpret_cast<u16x8*>(dst + (int64_t)c * d.n_pad + r8) = o;
}

__global__ void __launch_bounds__(256) k_fac16(const Fac16Desc d) { fac16_body(d, blockIdx.x); }

__global__ void __launch_bounds__(256) k_fac16_multi(const Fac16Desc* __restrict__ ds, int nd) {
  const Fac16Desc d = load_desc(ds, find_desc(ds, nd, (int)blockIdx.x));
  fac16_body(d, (int)blockIdx.x - d.block_begin);
}

// X = S U and Y = S^T V as two products of their own in one launch, the
// summation range split over wide_splits() work-groups.  What bounds it: the
// partial sums.  One pass over 2-D tiles (skinny_body) leaves about 2
// sqrt(work-groups) partials of each entry (42 at n = 7168: 308 MB at R = 256,
// written and read again); a product on its own leaves as many as its range is
// split (5 and 5 there), and reading the shadow twice costs less from R = 64
// on.  Work-group: 128 rows (X) or columns (Y) of S by BN factor columns, 4
// waves in 2 x 2, 64-deep steps through LDS, the next step in registers
// meanwhile.
//   X: A = S rows, B = Ut rows; Y: A = Vt rows, B = S columns (transposed reads).
// 16-byte pieces of the staged rows are permuted so that the operand reads
// touch all banks evenly.  At n = 7168 (the 2-D pass, which converts float
// factors as it stages them -> this): R = 64 56.5 -> 48.0 us, R = 128 113 ->
// 59 us, R = 256 226 -> 118 us, and the tail that adds the partials 51 -> 32 us
// and 228 -> 153 us at R = 128 and 256.  At R = 32 the 2-D pass stays (39 us;
// from bfloat16 factors 46 us).
// A split's sum is kept in two stages, so that a longer range costs no
// accuracy: chains of kGemmRun steps (192 terms, 12 matrix instructions), added
// up in float (at most 11 of them, kWideTerms terms).  The variance of a
// chain's rounding error grows with its length: in units of one instruction's,
// half the 12 instructions plus half the 11 additions, 11.5 for X and for Y,
// where one float chain per 256 columns (X) and per 512 rows (Y), the partials
// of a pass over 2-D tiles, has 8 and 16.  A rank-32 update at n = 7157, k = 16
// (three such levels): 982 to 1005 us with one chain per split, 1004 to 1022 us
// so; the products by themselves then R = 64 48 -> 54 us, R = 128 59 -> 56 to 69
// us, R = 256 118 -> 137 us.
constexpr int kGemmTile = 128, kGemmStep = 64, kGemmRun = 3;
template <int BN, bool YP>
__device__ __forceinline__ void skinny_gemm_body(const SkinnyDesc& d, uint16_t* sS, uint16_t* sF, const int tile,
                                                 const int split, const int splits) {
  constexpr int TM = kGemmTile, KS = kGemmStep;
  constexpr int SP = TM * KS / 8 / 256, FP = BN * KS / 8 / 256;   // pieces per thread
  constexpr int WB = BN / 64;                                      // 32-wide factor blocks per wave
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = wave_id();
  const int wm = wave >> 1, wn = wave & 1;
  const int l32 = lane & 31, lh = lane >> 5;
  const int n_pad = d.n_pad, pR = d.pR;
  const int m0 = tile * TM;
  const int nsteps = n_pad / KS;
  const int s0 = (int)((int64_t)nsteps * split / splits), s1 = (int)((int64_t)nsteps * (split + 1) / splits);
  const uint16_t* __restrict__ S = static_cast<const uint16_t*>(d.src);
  const uint16_t* __restrict__ F = reinterpret_cast<const uint16_t*>(YP ? d.Vj : d.Uj);

  u16x8 ps[SP], pf[FP];
  auto fetch = [&](const int st) {
    const int64_t k0 = (int64_t)st * KS;
    static_for<0, SP>([&](auto i) {
      const int q = tid + 256 * i;
      if constexpr (YP) ps[i] = *reinterpret_cast<const u16x8*>(S + (k0 + q / (TM / 8)) * d.ldp + m0 + q % (TM / 8) * 8);
      else ps[i] = *reinterpret_cast<const u16x8*>(S + (int64_t)(m0 + q / 8) * d.ldp + k0 + q % 8 * 8);
    });
    static_for<0, FP>([&](auto i) {
      const int q = tid + 256 * i;
      pf[i] = *reinterpret_cast<const u16x8*>(F + (int64_t)(q / 8) * n_pad + k0 + q % 8 * 8);
    });
  };
  // rows of 8 pieces (128 bytes): two rows apart by one piece
  auto piece = [](const int r, const int g) { return r * KS + (g ^ ((r >> 1) & 7)) * 8; };
  fetch(s0);
  v16f sum[2][WB];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) sum[a][b][v] = 0.f;

  for (int st = s0; st < s1;) {
    const int run = min(st + kGemmRun, s1);
    v16f acc[2][WB];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;
    for (; st < run; ++st) {
      __syncthreads();
      static_for<0, SP>([&](auto i) {
        const int q = tid + 256 * i;
        if constexpr (YP) {
          const int r = q / (TM / 8);
          *reinterpret_cast<u16x8*>(&sS[r * TM + ((q % (TM / 8)) ^ tr_swizzle(r)) * 8]) = ps[i];
        } else {
          *reinterpret_cast<u16x8*>(&sS[piece(q / 8, q % 8)]) = ps[i];
        }
      });
      static_for<0, FP>([&](auto i) {
        const int q = tid + 256 * i;
        *reinterpret_cast<u16x8*>(&sF[piece(q / 8, q % 8)]) = pf[i];
      });
      __syncthreads();
      if (st + 1 < s1) fetch(st + 1);
#pragma unroll
      for (int ks = 0; ks < KS / 16; ++ks) {
        bf16x8 so[2], fo[WB];
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          if constexpr (YP) so[a] = tr_operand<TM>(sS, ks * 16, wm * 64 + a * 32, lane);
          else so[a] = lds8(&sS[piece(wm * 64 + a * 32 + l32, 2 * ks + lh)]);
        }
#pragma unroll
        for (int b = 0; b < WB; ++b) fo[b] = lds8(&sF[piece(wn * 32 * WB + b * 32 + l32, 2 * ks + lh)]);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
          for (int b = 0; b < WB; ++b)
            acc[a][b] = YP ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(fo[b], so[a], acc[a][b], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f32_32x32x16_bf16(so[a], fo[b], acc[a][b], 0, 0, 0);
      }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < WB; ++b)
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[a][b][v] += acc[a][b][v];
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < WB; ++b) {
      const int m = m0 + wm * 64 + a * 32, c = wn * 32 * WB + b * 32;
      if constexpr (YP) {
        // values 4 q .. 4 q + 3 of a lane are four consecutive factor columns
        float* py = d.partY + ((int64_t)split * n_pad + m + l32) * pR + c + 4 * lh;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4*>(py + 8 * q) =
              f32x4{sum[a][b][4 * q], sum[a][b][4 * q + 1], sum[a][b][4 * q + 2], sum[a][b][4 * q + 3]};
      } else {
        float* px = d.partX + ((int64_t)split * n_pad + m + 4 * lh) * pR + c + l32;
#pragma unroll
        for (int v = 0; v < 16; ++v) px[(8 * (v / 4) + v % 4) * pR] = sum[a][b][v];
      }
    }
}

// Work-groups of one launch: the X products, then the Y products; tiles of one
// split are neighbours (they share the factor rows of its range).
template <int BN>
__device__ __forceinline__ void skinny_gemm(const SkinnyDesc& d, int blk) {
  __shared__ __align__(16) uint16_t sS[kGemmTile * kGemmStep];
  __shared__ __align__(16) uint16_t sF[BN * kGemmStep];
  const int tiles = d.n_pad / kGemmTile, splits = wide_splits(d.n_pad);
  const bool yp = blk >= tiles * splits;
  if (yp) blk -= tiles * splits;
  if (yp) skinny_gemm_body<BN, true>(d, sS, sF, blk % tiles, blk / tiles, splits);
  else skinny_gemm_body<BN, false>(d, sS, sF, blk % tiles, blk / tiles, splits);
}

template <int BN>
__global__ void __launch_bounds__(256, 2) k_skinny_gemm(const SkinnyDesc d) { skinny_gemm<BN>(d, blockIdx.x); }

template <int BN>
__global__ void __launch_bounds__(256, 2) k_skinny_gemm_multi(const SkinnyDesc* __restrict__ ds, int nd) {
  const SkinnyDesc d = load_desc(ds, find_skinny(ds, nd, (int)blockIdx.x));
  skinny_gemm<BN>(d, (int)blockIdx.x - d.block_begin);
}

// ---------------------------------------------------------------- shared passes
//
// A shadowed level of rank R <= kChain16Rank for T successive updates of a
// batch: X = S U, Y = S^T V from the bfloat16 values of P as the update finds
// it, then P += U V^T, T times over, at one read and write of P and one write
// of the shadow: 10 n^2 / T bytes an update, where k_skinny_bf16 and
// k_level_update read the shadow, read and write P and write the shadow for
// each, 12 n^2.  The shadow is not read: it is P rounded.
//
// Every sum has the order of those two kernels, so the results are the same
// bit for bit: an X partial is the sum of the chains over the quarters of a
// tile's columns, (a + b) + (c + d), a Y partial the chain over the slice's
// interleaved 64-row chunks, both of v_mfma_f32_32x32x16_bf16 (operands
// exchanged: a lane then holds consecutive factor columns of one row or
// column); the delta is the fused multiply-add chain over the factor columns
// from zero (v_mfma_f32_16x16x4f32 adds its four products in index order with
// one rounding each; ranks 1 and 2 end in zero products) or, at rank 32, the
// three split products of update_split_body.
//
// Work-group: one 256-column tile's slice, 8 waves, one group per compute unit
// (LDS); a wave keeps the 64 x 32 block of its columns of a chunk in registers
// over the T updates and passes its rounded values through LDS to the others.
// All a chunk needs is requested a chunk ahead and V stays in registers: loads
// return in order, so an operand asked for behind the next chunk's P would
// arrive behind it (rank 32: 794 us so against 990 us with operands loaded as
// they are used).  What bounds it: up to rank 8 the traffic, then the steps
// between barriers (barrier, LDS reads, matrix instructions in sequence: a
// group's 8 waves are all there are to overlap).
//
// n = 16384 (1.07 GB of P, 0.54 GB of shadow; the traffic alone 430 us), passes
// by themselves, in us: rank 4 four updates 640, rank 8 706, rank 16 952, rank
// 32 two updates 604; an update alone 520 to 610 for its two passes.  A batch
// of 8 rank-4 updates, k = 16: 23.5 -> 9.4 ms.
//
// Operands are prepared by k_chain_factors: per update Ut and Vt (bfloat16, R
// rows of n_pad) and the factors of the delta (U then V: floats, max(R, 4) rows
// of n_pad; at rank 32 the high and the low bfloat16 parts, n_pad rows of 32).
constexpr int chain_rows(int R) { return R < 4 ? 4 : R; }

template <int R>
__device__ __forceinline__ void chain_factors_body(const ChainDesc& d, const float* __restrict__ slab, const int side,
                                                   const int ver, const int tile) {
  __shared__ float t[64][R + 1];
  const int tid = threadIdx.x;
  const float* src = slab + (int64_t)tile * 64 * d.W;
  for (int e = tid; e < 64 * R; e += 256) t[e / R][e % R] = src[(int64_t)(e / R) * d.W + e % R];
  __syncthreads();
  const int64_t n = d.n_pad, r0 = (int64_t)tile * 64;
  uint16_t* f16 = d.f16 + ((int64_t)ver * 2 + side) * R * n;
  for (int e = tid; e < 64 * R; e += 256) f16[(int64_t)(e / 64) * n + r0 + e % 64] = bf16_rne(t[e % 64][e / 64]);
  if constexpr (R < 32) {
    constexpr int RK = chain_rows(R);
    float* f = static_cast<float*>(d.f32) + ((int64_t)ver * 2 + side) * RK * n;
    for (int e = tid; e < 64 * RK; e += 256) f[(int64_t)(e / 64) * n + r0 + e % 64] = e / 64 < R ? t[e % 64][e / 64] : 0.f;
  } else {
    uint16_t* h = static_cast<uint16_t*>(d.f32) + ((int64_t)ver * 2 + side) * 2 * R * n;
    for (int e = tid; e < 64 * R; e += 256) {
      const float x = t[e / R][e % R];
      const uint16_t hi = bf16_rne(x);
      h[r0 * R + e] = hi;
      h[n * R + r0 * R + e] = bf16_rne(x - __builtin_bit_cast(float, (uint32_t)hi << 16));
    }
  }
}

template <int R>
__global__ void __launch_bounds__(256) k_chain_factors(const ChainDesc d) {
  const int ver = blockIdx.y, side = blockIdx.z;
  chain_factors_body<R>(d, (side ? d.V : d.U) + ver * d.vs.s, side, ver, blockIdx.x);
}

constexpr int kChainWaves = 8;
template <int R, int T>
__global__ void __launch_bounds__(64 * kChainWaves, 2) k_shadow_chain(const ChainDesc d) {
  constexpr int NT = 64 * kChainWaves;
  constexpr int RK = chain_rows(R);
  constexpr int CH = 64;                      // rows per chunk
  constexpr int CW = TCB / kChainWaves;       // columns per wave
  static_assert(CW == 32 && T % 2 == 0, "one 32-column block per wave; the shadow buffers alternate over T + 1 writes");
  // staged rows, padded so that operand reads touch all banks evenly: Ut of
  // the tile's columns; per update of a chunk U (floats: RK rows of 64; rank
  // 32: 64 rows of 32 high and of 32 low parts) and Vt (R rows of 64)
  constexpr int US = TCB + 8;
  constexpr int FS = R < 32 ? 80 * 2 : 40, VS = CH + 8;            // row strides in 16-bit units
  constexpr int FROWS = R < 32 ? RK : 2 * CH;
  constexpr int OPS = FROWS * FS + R * VS;                         // one update's
  constexpr int FPR = R < 32 ? 16 : 4;                             // 16-byte pieces of a U row
  constexpr int PIECES = FROWS * FPR + R * 8;                      // and of one update
  constexpr int NP = (T * PIECES + NT - 1) / NT;
  __shared__ __align__(16) uint16_t sS[2 * CH * TCB];
  __shared__ __align__(16) uint16_t sU[T * R * US];
  __shared__ __align__(16) uint16_t sO[T * OPS];
  // X: each wave forms 32 rows over a quarter (R <= 16) or, every other update,
  // over a half of the tile's columns; the parts are added in LDS after the
  // next barrier
  constexpr int PARTS = R <= 16 ? 4 : 2, RX = R < 4 ? 4 : R;
  __shared__ __align__(16) float sX[2 * PARTS * CH * RX];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = wave_id();
  const int l32 = lane & 31, lh = lane >> 5, l16 = lane & 15, lq = lane >> 4;
  const int ct = blockIdx.x, rt = blockIdx.y;
  const int n_pad = d.n_pad;
  const int64_t n = n_pad, ldp = d.ldp;
  const int ns = (n_pad + d.tile_rows - 1) / d.tile_rows;
  const int nchunks = n_pad / CH;
  const int col0 = ct * TCB, wc = wave * CW;
  const int cr = l32 < R ? l32 : R - 1;       // operand rows past R feed results that are not kept
  if (rt >= nchunks) return;                  // (a slice has a chunk: tile_rows >= 64)

  // the wave's 64 x 32 block: 8 groups of four consecutive columns per lane
  auto grow = [](auto g) { return g / 2 * 16; };   // group's first row and column
  auto gcol = [](auto g) { return g % 2 * 16; };
  const int lrow = l16, lcol = wc + 4 * lq;
  const unsigned poff = (unsigned)(lrow * ldp + lcol) * 4;
  // The next chunk's operands, and its values where T R <= 32, are requested a
  // chunk ahead; beyond, the values once the chunk's are stored: the registers
  // would spill, and a reload waits for every load before it (rank 16, four
  // updates: 1288 us spilled, 952 us so; four updates at ranks 1, 2 and 4 still
  // keep 5, 3 and 9 registers in scratch).
  constexpr bool AHEAD = T * R <= 32;
  f32x4 p[8], pn[AHEAD ? 8 : 1];
  u16x8 on[NP];
  auto load = [&](const int ch) {
    const int64_t r0 = (int64_t)ch * CH;
    static_for<0, NP>([&](auto i) {
      const int q = tid + NT * i, t = q / PIECES, e = q % PIECES;
      if (T * PIECES % NT != 0 && q >= T * PIECES) return;
      const uint16_t* src;
      if (e >= FROWS * FPR) {
        const int f = e - FROWS * FPR;
        src = d.f16 + ((int64_t)(2 * t + 1) * R + f / 8) * n + r0 + f % 8 * 8;
      } else if (R < 32) {
        src = reinterpret_cast<const uint16_t*>(static_cast<const float*>(d.f32) + ((int64_t)(2 * t) * RK + e / FPR) * n + r0 + e % FPR * 4);
      } else {
        src = static_cast<const uint16_t*>(d.f32) + ((int64_t)(4 * t) + e / (FPR * CH)) * R * n + r0 * R + e % (FPR * CH) * 8;
      }
      on[i] = *reinterpret_cast<const u16x8*>(src);
    });
  };
  auto load_p = [&](auto& dst, const int ch) {
    const float* src = d.P + (int64_t)ch * CH * ldp + col0;
    static_for<0, 8>([&](auto g) {
      dst[g] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(at_byte(src + grow(g) * ldp + gcol(g), poff)));
    });
  };
  auto stage = [&](uint16_t* ops) {
    static_for<0, NP>([&](auto i) {
      const int q = tid + NT * i, t = q / PIECES, e = q % PIECES;
      if (T * PIECES % NT != 0 && q >= T * PIECES) return;
      const int f = e - FROWS * FPR;
      const int at = f >= 0 ? FROWS * FS + f / 8 * VS + f % 8 * 8 : e / FPR * FS + e % FPR * 8;
      *reinterpret_cast<u16x8*>(&ops[t * OPS + at]) = on[i];
    });
  };
  // (the permutation repeats every 16 rows and acts on the column's bits, of
  // which a group's are zero in the lane's)
  const int pat = lrow * TCB + (((lcol / 8) ^ tr_swizzle(lrow)) * 8 + lcol % 8);
  auto put = [&](uint16_t* buf) {
    static_for<0, 8>([&](auto g) {
      ushort4 h;
      h.x = bf16_rne(p[g][0]); h.y = bf16_rne(p[g][1]); h.z = bf16_rne(p[g][2]); h.w = bf16_rne(p[g][3]);
      *reinterpret_cast<ushort4*>(&buf[grow(g) * TCB + (pat ^ gcol(g))]) = h;
    });
  };
  // piece (4 factor columns) j of a row of X parts
  auto xat = [](const int row, const int j) { return row * RX + (j ^ ((row * RX / 64) & (RX / 4 - 1))) * 4; };
  auto sum_x = [&](const float* parts, const int t, const int64_t r0) {
    constexpr int G = RX / 4;
    if (CH * G < NT && tid >= CH * G) return;
    const int row = tid / G, j = tid % G;
    auto part = [&](const int i) { return *reinterpret_cast<const f32x4*>(&parts[i * CH * RX + xat(row, j)]); };
    f32x4 x = part(0) + part(1);
    if constexpr (PARTS == 4) x = x + (part(2) + part(3));
    float* px = d.partX + t * d.vs.x + ((int64_t)ct * n + r0 + row) * R + 4 * j;
    if constexpr (R < 4) {
#pragma unroll
      for (int c = 0; c < R; ++c) px[c] = x[c];
    } else {
      *reinterpret_cast<f32x4*>(px) = x;
    }
  };
  load(rt);
  if constexpr (AHEAD) load_p(pn, rt);
  else load_p(p, rt);

  for (int q = tid; q < T * R * (TCB / 8); q += NT) {
    const int row = q / (TCB / 8), g = q % (TCB / 8);
    *reinterpret_cast<u16x8*>(&sU[row * US + g * 8]) =
        *reinterpret_cast<const u16x8*>(d.f16 + ((int64_t)(row / R) * 2 * R + row % R) * n + col0 + g * 8);
  }
  // V of the wave's columns (rank 32: operand row m is column m with bits 2 and
  // 3 exchanged, see the update)
  constexpr int VN = R < 32 ? RK / 4 : 2;
  float vv[T][2][R < 32 ? VN : 1];
  bf16x8 vh[T][2], vl[T][2];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    if constexpr (R < 32) {
      const float* fv = static_cast<const float*>(d.f32) + ((int64_t)(2 * t + 1) * RK + lq) * n + col0 + wc + l16;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int e = 0; e < VN; ++e) vv[t][b][e] = fv[(int64_t)(4 * e) * n + 16 * b];
    } else {
      const uint16_t* hv = static_cast<const uint16_t*>(d.f32) + (int64_t)(4 * t + 2) * R * n +
                           (int64_t)(col0 + wc + (l32 & 19) + (l32 & 4) * 2 + (l32 & 8) / 2) * R + 8 * lh;
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        vh[t][k] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(hv + 16 * k));
        vl[t][k] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u16x8*>(hv + n * R + 16 * k));
      }
    }
  }

  v16f yacc[T];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) yacc[t][v] = 0.f;
  stage(sO);

  // A shadow buffer and one of X parts are written again two writes on: the
  // last readers are then past a barrier in between.
  int sb = 0;
  for (int ch = rt; ch < nchunks; ch += ns) {
    const int64_t r0 = (int64_t)ch * CH;
    if constexpr (AHEAD) static_for<0, 8>([&](auto g) { p[g] = pn[g]; });
    if (ch + ns < nchunks) {
      load(ch + ns);
      if constexpr (AHEAD) load_p(pn, ch + ns);
    }
    static_for<0, T>([&](auto t) {
      asm volatile("" ::: "memory");   // keeps a later update's operands out of the registers
      uint16_t* buf = sS + sb * (CH * TCB);
      const uint16_t* ops = sO + t * OPS;
      put(buf);
      __syncthreads();
      sb ^= 1;
      if constexpr (t > 0) sum_x(sX + ((t - 1) & 1) * PARTS * CH * RX, t - 1, r0);

      if (PARTS == 4 || (wave >> 2) == (t & 1)) {
        constexpr int KS = 4;                 // steps of a quarter
        const int part = (wave >> 1) & (PARTS - 1);
        const int r = (wave & 1) * 32 + l32;
        const int rat = r * TCB + (lh ^ tr_swizzle(r)) * 8;
        const uint16_t* u = sU + (t * R + cr) * US + 8 * lh;
        v16f x[4 / PARTS];
#pragma unroll
        for (int i = 0; i < 4 / PARTS; ++i) {
#pragma unroll
          for (int v = 0; v < 16; ++v) x[i][v] = 0.f;
        }
#pragma unroll
        for (int i = 0; i < 4 / PARTS; ++i) {
          if (i > 0) asm volatile("" ::: "memory");
#pragma unroll
          for (int k = 0; k < KS; ++k) {
            const int c = (part * (4 / PARTS) + i) * KS + k;
            x[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds8(u + 16 * c), lds8(buf + (rat ^ (16 * c))), x[i], 0, 0, 0);
          }
        }
        if constexpr (PARTS == 2)
#pragma unroll
          for (int v = 0; v < 16; ++v) x[0][v] += x[1][v];
        float* px = sX + ((t & 1) * PARTS + part) * CH * RX;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (8 * q + 4 * lh < R)
            *reinterpret_cast<f32x4*>(&px[xat(r, 2 * q + lh)]) = f32x4{x[0][4 * q], x[0][4 * q + 1], x[0][4 * q + 2], x[0][4 * q + 3]};
      }
      asm volatile("" ::: "memory");
      const uint16_t* ov = ops + FROWS * FS + cr * VS + 8 * lh;
#pragma unroll
      for (int ks = 0; ks < CH / 16; ++ks)
        yacc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds8(ov + 16 * ks), tr_operand<TCB>(buf, ks * 16, wc, lane),
                                                          yacc[t], 0, 0, 0);
      // P += U V^T
      if constexpr (R < 32) {
        const float* ou = reinterpret_cast<const float*>(ops) + lq * (FS / 2) + l16;
        asm volatile("" ::: "memory");
#pragma unroll
        for (int a = 0; a < 4; ++a) {
          float uu[VN];
#pragma unroll
          for (int e = 0; e < VN; ++e) uu[e] = ou[4 * e * (FS / 2) + 16 * a];
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < VN; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[t][b][e], uu[e], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) p[2 * a + b][v] += acc[v];
          }
        }
      } else {
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          const uint16_t* ou = ops + (32 * a + l32) * FS + 8 * lh;
          v16f acc;
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            const bf16x8 uh = lds8(ou + 16 * k), ul = lds8(ou + CH * FS + 16 * k);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh[t][k], ul, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vl[t][k], uh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vh[t][k], uh, acc, 0, 0, 0);
          }
          // A quad of columns of a row per lane, 32 rows wide; exchanging lanes
          // 16-31 (48-63) of one quad with lanes 0-15 (32-47) of the next leaves
          // the 16-row groups above, whose lanes cover 64 bytes of a row (32
          // bytes a row: 794 us, see above; 64: 604 us).
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const auto w = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, (float)acc[8 * h + e]),
                                                              __builtin_bit_cast(unsigned, (float)acc[8 * h + 4 + e]), false,
                                                              false);
              p[4 * a + h][e] += __builtin_bit_cast(float, (unsigned)w[0]);
              p[4 * a + 2 + h][e] += __builtin_bit_cast(float, (unsigned)w[1]);
            }
        }
      }
    });
    {
      float* dst = d.P + r0 * ldp + col0;
      static_for<0, 8>([&](auto g) {
        __builtin_nontemporal_store(p[g], reinterpret_cast<f32x4*>(
            reinterpret_cast<char*>(dst + grow(g) * ldp + gcol(g)) + poff));
      });
    }
    uint16_t* buf = sS + sb * (CH * TCB);
    put(buf);
    if constexpr (!AHEAD)
      if (ch + ns < nchunks) load_p(p, ch + ns);
    __syncthreads();
    sb ^= 1;
    sum_x(sX + ((T - 1) & 1) * PARTS * CH * RX, T - 1, r0);
    if (ch + ns < nchunks) stage(sO);   // (this chunk's are no longer read)
    static_for<0, CH * TCB / 8 / NT>([&](auto i) {
      const int q = tid + NT * i, r = q / (TCB / 8), g = q % (TCB / 8);
      *reinterpret_cast<u16x8*>(d.S + (r0 + r) * ldp + col0 + g * 8) =
          *reinterpret_cast<const u16x8*>(&buf[r * TCB + (g ^ tr_swizzle(r)) * 8]);
    });
  }

  static_for<0, T>([&](auto t) {
    float* py = d.partY + t * d.vs.y + ((int64_t)rt * n + col0 + wc + l32) * R;
    if constexpr (R < 4) {
      if (lh == 0)
#pragma unroll
        for (int c = 0; c < R; ++c) py[c] = yacc[t][c];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (8 * q + 4 * lh < R)
          *reinterpret_cast<f32x4*>(py + 8 * q + 4 * lh) =
              f32x4{yacc[t][4 * q], yacc[t][4 * q + 1], yacc[t][4 * q + 2], yacc[t][4 * q + 3]};
    }
  });
}

template <int R>
hipError_t shadow_chain_r(const ChainDesc& d, int nver, hipStream_t s) {
  hipLaunchKernelGGL((k_chain_factors<R>), dim3((unsigned)(d.n_pad / 64), (unsigned)nver, 2), dim3(256), 0, s, d);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid((unsigned)(d.n_pad / TCB), (unsigned)((d.n_pad + d.tile_rows - 1) / d.tile_rows));
  if (nver == 2) hipLaunchKernelGGL((k_shadow_chain<R, 2>), grid, dim3(64 * kChainWaves), 0, s, d);
  else if (nver == chain16_updates(R)) hipLaunchKernelGGL((k_shadow_chain<R, chain16_updates(R)>), grid, dim3(64 * kChainWaves), 0, s, d);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// Update fused into the float skinny pass (R = 16 or 32 factor columns, one
// launch): blocks of 512 threads, waves 0-3 form X and Y on the matrix cores
// as the read-only pass does and waves 4-7 apply P += U_j V_j^T to the same
// chunk on the vector units: update wave wu takes rows wu + 4 i of the chunk
// and lane g the columns 4 g .. 4 g + 3; the old values come from the chunk
// in LDS, U_j rows of the chunk from sUr, V_j rows of the tile's columns
// from sVc (sVc[c][k] = V_j[col0 + k][c]); the delta is summed over c in
// order from zero and added once; the new rows go straight to HBM.  The
// matrix-core and vector work of a chunk share the SIMDs.
template <int CR, int SW, int UW>
__device__ __forceinline__ void chunk_update(float* __restrict__ P, const int64_t ldp, const int col0, const int cr0,
                                             const int R, const float (*sP)[SW], const float (*sUr)[UW],
                                             const float (*sVc)[SW], const int wu, const int lane) {
  float d[CR / 4][4];
#pragma unroll
  for (int i = 0; i < CR / 4; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) d[i][q] = 0.f;
  for (int c0 = 0; c0 < R; c0 += 4) {
    f32x4 v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = *reinterpret_cast<const f32x4*>(&sVc[c0 + e][4 * lane]);
#pragma unroll
    for (int i = 0; i < CR / 4; ++i) {
      const f32x4 u = *reinterpret_cast<const f32x4*>(&sUr[wu + 4 * i][c0]);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int q = 0; q < 4; ++q) d[i][q] = fma(u[e], v[e][q], d[i][q]);
    }
  }
#pragma unroll
  for (int i = 0; i < CR / 4; ++i) {
    f32x4 p = *reinterpret_cast<const f32x4*>(&sP[wu + 4 * i][4 * lane]);
#pragma unroll
    for (int q = 0; q < 4; ++q) p[q] += d[i][q];
    __builtin_nontemporal_store(p, reinterpret_cast<f32x4*>(P + (int64_t)(cr0 + wu + 4 * i) * ldp + col0 + 4 * lane));
  }
}

// Float skinny pass.  Tile: about tile_rows x 256 columns of P, chunks of 32
// rows through LDS (the next chunk of P and V_j held in registers meanwhile);
// factor columns padded with zeros to 32 NB (NB <= 2).  The ns row slices of
// a column tile interleave by chunks (slice rt takes chunks rt, rt + ns, ...),
// so the grid streams one band of rows at a time.
//   X: the chunk's 32 x 32 NB outputs with K = 256 split over the waves
//      (wave w: columns [64 w, 64 w + 64)); the four partial sums meet in
//      LDS (over the chunk buffer, no longer read) and are added in wave
//      order; one partial per (row, column tile).
//   Y: as the bfloat16 kernel, wave w owns tile columns [64 w, 64 w + 64).
// A group of four f32 steps covers 8 summation indices: lanes 0-31 supply
// index g + e and lanes 32-63 index g + 4 + e in step e, for both operands.
// `want` selects the products formed (bit 0: X, bit 1: Y; uniform).
template <int NB, bool UPD = false>
__device__ __forceinline__ void skinny_f32_body(const float* __restrict__ P, const int64_t ldp, const int n_pad,
                                                const int tile_rows, const float* __restrict__ Uj,
                                                const float* __restrict__ Vj, const int W, const int R,
                                                float* __restrict__ partX, float* __restrict__ partY,
                                                const int pR, const int want, const int ct, const int rt) {
  const bool wx = (want & kWantX) != 0, wy = (want & kWantY) != 0;
  constexpr int RP = 32 * NB;
  constexpr int CR = 32;           // rows per chunk
  constexpr int FP = 4;            // LDS row padding (floats)
  constexpr int NT = UPD ? 512 : 256;
  static_assert(NB <= 2, "the X exchange buffer must fit in the chunk buffer");
  static_assert(!UPD || NB == 1, "the fused update takes all factor columns in one launch");
  __shared__ __align__(16) float sP[CR][TCB + FP];
  __shared__ __align__(16) float sUt[RP][TCB + FP];
  __shared__ __align__(16) float sVt[RP][CR + FP];
  __shared__ __align__(16) float sVc[UPD ? RP : 1][TCB + FP];
  __shared__ __align__(16) float sUr[UPD ? CR : 1][RP + FP];
  float* xbuf = &sP[0][0];         // [4 waves][NB][16 values][64 lanes]

  const int tid = threadIdx.x;
  const bool mwave = !UPD || tid < 256;   // matrix-core waves (all of them without the update)
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col0 = ct * TCB;
  // interleaved chunks: slice rt of ns takes chunks rt, rt + ns, ...
  const int ns = (n_pad + tile_rows - 1) / tile_rows;
  const int CS = ns * 32;
  const int row0 = rt * 32;
  const int rend = n_pad;
  const int l32 = lane % 32, lh = lane / 32;
  // chunk staging: thread -> rows tid / 64 + 4 i, f32x4 column group tid % 64
  const int srow = tid / 64, sgrp = tid % 64;

  constexpr int VPT = RP * CR / 256;
  f32x4 pre[CR / 4];
  float pv[VPT];
  auto fetch = [&](const int r0) {
    static_for<0, CR / 4>([&](auto i) {
      pre[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(P + (int64_t)(r0 + srow + 4 * i) * ldp + col0 +
                                                                     sgrp * 4));
    });
    static_for<0, VPT>([&](auto i) {
      const int idx = tid + 256 * i;
      const int rr = idx / RP, c = idx % RP;
      pv[i] = fac_clamped(Vj + (int64_t)(r0 + rr) * W, c, R);
    });
  };
  // update waves: the chunk's U_j rows (thread t = tid - 256 holds entries t + 256 i)
  float pu[VPT];
  auto fetch_u = [&](const int r0) {
    static_for<0, VPT>([&](auto i) {
      const int idx = tid - 256 + 256 * i;
      const int rr = idx / RP, c = idx % RP;
      pu[i] = fac_clamped(Uj + (int64_t)(r0 + rr) * W, c, R);
    });
  };
  if (mwave) fetch(row0);
  else if constexpr (UPD) fetch_u(row0);

  if (wx)
    batched_stage<RP * TCB / NT, NT, float>(
        tid, RP * TCB, [&](int idx) { const int c = idx % RP; return fac_or_zero(Uj + (int64_t)(col0 + idx / RP) * W, c, R); },
        [&](int idx, float v) { sUt[idx % RP][idx / RP] = v; });
  if constexpr (UPD)
    batched_stage<RP * TCB / NT, NT, float>(
        tid, RP * TCB, [&](int idx) { const int c = idx % RP; return fac_or_zero(Vj + (int64_t)(col0 + idx / RP) * W, c, R); },
        [&](int idx, float v) { sVc[idx % RP][idx / RP] = v; });

  v16f yacc[NB][2];
#pragma unroll
  for (int a = 0; a < NB; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int v = 0; v < 16; ++v) yacc[a][b][v] = 0.f;

  for (int cr0 = row0; cr0 < rend; cr0 += CS) {
    __syncthreads();   // the previous chunk's exchange buffer has been read
    if (mwave) {
      static_for<0, CR / 4>([&](auto i) { *reinterpret_cast<f32x4*>(&sP[srow + 4 * i][sgrp * 4]) = pre[i]; });
      static_for<0, VPT>([&](auto i) {
        const int idx = tid + 256 * i;
        sVt[idx % RP][idx / RP] = idx % RP < R ? pv[i] : 0.f;
      });
    } else if constexpr (UPD) {
      static_for<0, VPT>([&](auto i) {
        const int idx = tid - 256 + 256 * i;
        sUr[idx / RP][idx % RP] = idx % RP < R ? pu[i] : 0.f;
      });
    }
    __syncthreads();
    if constexpr (UPD) {
      if (!mwave) {
        if (cr0 + CS < rend) fetch_u(cr0 + CS);
        chunk_update<CR, TCB + FP, RP + FP>(const_cast<float*>(P), ldp, col0, cr0, R, sP, sUr, sVc, wave - 4, lane);
        continue;
      }
    }
    if (cr0 + CS < rend) fetch(cr0 + CS);

    if constexpr (NB == 1) {
      // one 32-column factor block: wave w forms the 16 x 16 X tile of rows
      // 16 (w % 2) .. +15 and factor columns 16 (w / 2) .. +15 over the whole
      // tile width on v_mfma_f32_16x16x4f32 (lane l: row / column l % 16,
      // summation index g + 4 (l / 16) + e), so no partial sums cross waves
      if (wx) {
        typedef float v4f __attribute__((ext_vector_type(4)));
        const int l16 = lane % 16, lq = lane / 16;
        const int mb = wave % 2, nbx = wave / 2;
        v4f acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
        for (int g = 0; g < TCB; g += 32) {
          const f32x4 a0 = *reinterpret_cast<const f32x4*>(&sP[mb * 16 + l16][g + 4 * lq]);
          const f32x4 b0 = *reinterpret_cast<const f32x4*>(&sUt[nbx * 16 + l16][g + 4 * lq]);
          const f32x4 a1 = *reinterpret_cast<const f32x4*>(&sP[mb * 16 + l16][g + 16 + 4 * lq]);
          const f32x4 b1 = *reinterpret_cast<const f32x4*>(&sUt[nbx * 16 + l16][g + 16 + 4 * lq]);
          acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.x, b0.x, acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.x, b1.x, acc1, 0, 0, 0);
          acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.y, b0.y, acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.y, b1.y, acc1, 0, 0, 0);
          acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.z, b0.z, acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.z, b1.z, acc1, 0, 0, 0);
          acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0.w, b0.w, acc0, 0, 0, 0);
          acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1.w, b1.w, acc1, 0, 0, 0);
        }
        const int c = nbx * 16 + l16;
        if (c < R) {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            partX[((int64_t)ct * n_pad + cr0 + mb * 16 + 4 * lq + v) * pR + c] = acc0[v] + acc1[v];
        }
      }
    }
    // X partial over this wave's 64 columns (two factor blocks)
    v16f xacc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v = 0; v < 16; ++v) xacc[nb][v] = 0.f;
#pragma unroll
    for (int g = 0; g < (wx && NB > 1 ? 64 : 0); g += 8) {
      const int k0 = wave * 64 + g + 4 * lh;
      const f32x4 a = *reinterpret_cast<const f32x4*>(&sP[l32][k0]);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const f32x4 b = *reinterpret_cast<const f32x4*>(&sUt[nb * 32 + l32][k0]);
        xacc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, xacc[nb], 0, 0, 0);
        xacc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, xacc[nb], 0, 0, 0);
        xacc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, xacc[nb], 0, 0, 0);
        xacc[nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, xacc[nb], 0, 0, 0);
      }
    }

    // Y^T += V_chunk^T P_chunk
#pragma unroll
    for (int g = 0; g < (wy ? CR : 0); g += 8) {
      const int r0 = g + 4 * lh;
#pragma unroll
      for (int cbi = 0; cbi < 2; ++cbi) {
        const int colc = (2 * wave + cbi) * 32 + l32;
        const float b0 = sP[r0][colc], b1 = sP[r0 + 1][colc], b2 = sP[r0 + 2][colc], b3 = sP[r0 + 3][colc];
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          const f32x4 a = *reinterpret_cast<const f32x4*>(&sVt[nb * 32 + l32][r0]);
          yacc[nb][cbi] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b0, yacc[nb][cbi], 0, 0, 0);
          yacc[nb][cbi] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b1, yacc[nb][cbi], 0, 0, 0);
          yacc[nb][cbi] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b2, yacc[nb][cbi], 0, 0, 0);
          yacc[nb][cbi] = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b3, yacc[nb][cbi], 0, 0, 0);
        }
      }
    }

    if (!wx || NB == 1) continue;
    // exchange the X partials (sP is no longer read in this chunk)
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v = 0; v < 16; ++v) xbuf[((wave * NB + nb) * 16 + v) * 64 + lane] = xacc[nb][v];
    __syncthreads();
    // thread -> (v, lane) slots of the 32 x 32 NB outputs
#pragma unroll
    for (int i = 0; i < NB * 4; ++i) {
      const int slot = tid + 256 * i;          // [nb][v][lane]
      const int ln = slot % 64, v = (slot / 64) % 16, nb = slot / 1024;
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) x += xbuf[((w * NB + nb) * 16 + v) * 64 + ln];
      const int c = nb * 32 + ln % 32;
      const int rr = 8 * (v / 4) + 4 * (ln / 32) + (v % 4);
      if (c < R) partX[((int64_t)ct * n_pad + cr0 + rr) * pR + c] = x;
    }
  }

  if (!wy || !mwave) return;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int cbi = 0; cbi < 2; ++cbi) {
      const int col = col0 + (2 * wave + cbi) * 32 + l32;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int c = nb * 32 + 8 * (v / 4) + 4 * lh + (v % 4);
        if (c < R) partY[((int64_t)rt * n_pad + col) * pR + c] = yacc[nb][cbi][v];
      }
    }
}

// Float skinny pass for at most 16 factor columns on v_mfma_f32_16x16x4f32:
// half the matrix-core work of the 32-wide pass at these ranks.  Tiling,
// chunk staging, the X exchange and the partial layouts as skinny_f32_body.
// 16x16x4 layouts: A (16 x 4): lane l holds A[l % 16][l / 16]; B (4 x 16):
// lane l holds B[l / 16][l % 16]; C: element v of lane l is
// C[4 (l / 16) + v][l % 16].  A group of four steps covers 16 summation
// indices: lane l supplies index g + 4 (l / 16) + e in step e, for both
// operands.
template <bool UPD = false>
__device__ __forceinline__ void skinny16_f32_body(const float* __restrict__ P, const int64_t ldp, const int n_pad,
                                                  const int tile_rows, const float* __restrict__ Uj,
                                                  const float* __restrict__ Vj, const int W, const int R,
                                                  float* __restrict__ partX, float* __restrict__ partY,
                                                  const int pR, const int want, const int ct, const int rt) {
  typedef float v4f __attribute__((ext_vector_type(4)));
  const bool wx = (want & kWantX) != 0, wy = (want & kWantY) != 0;
  constexpr int RP = 16;
  constexpr int CR = 32;           // rows per chunk
  constexpr int FP = 4;            // LDS row padding (floats)
  constexpr int NT = UPD ? 512 : 256;
  __shared__ __align__(16) float sP[CR][TCB + FP];
  __shared__ __align__(16) float sUt[RP][TCB + FP];
  __shared__ __align__(16) float sVt[RP][CR + FP];
  __shared__ __align__(16) float sVc[UPD ? RP : 1][TCB + FP];
  __shared__ __align__(16) float sUr[UPD ? CR : 1][RP + FP];
  float* xbuf = &sP[0][0];         // [4 waves][2 row blocks][4 values][64 lanes]

  const int tid = threadIdx.x;
  const bool mwave = !UPD || tid < 256;   // matrix-core waves (all of them without the update)
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col0 = ct * TCB;
  // interleaved chunks: slice rt of ns takes chunks rt, rt + ns, ...
  const int ns = (n_pad + tile_rows - 1) / tile_rows;
  const int CS = ns * 32;
  const int row0 = rt * 32;
  const int rend = n_pad;
  const int l16 = lane % 16, lq = lane / 16;
  const int srow = tid / 64, sgrp = tid % 64;

  constexpr int VPT = RP * CR / 256;
  f32x4 pre[CR / 4];
  float pv[VPT];
  auto fetch = [&](const int r0) {
    static_for<0, CR / 4>([&](auto i) {
      pre[i] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(P + (int64_t)(r0 + srow + 4 * i) * ldp + col0 +
                                                                     sgrp * 4));
    });
    static_for<0, VPT>([&](auto i) {
      const int idx = tid + 256 * i;
      const int rr = idx / RP, c = idx % RP;
      pv[i] = fac_clamped(Vj + (int64_t)(r0 + rr) * W, c, R);
    });
  };
  // update waves: the chunk's U_j rows (thread t = tid - 256 holds entries t + 256 i)
  float pu[VPT];
  auto fetch_u = [&](const int r0) {
    static_for<0, VPT>([&](auto i) {
      const int idx = tid - 256 + 256 * i;
      const int rr = idx / RP, c = idx % RP;
      pu[i] = fac_clamped(Uj + (int64_t)(r0 + rr) * W, c, R);
    });
  };
  if (mwave) fetch(row0);
  else if constexpr (UPD) fetch_u(row0);

  if (wx)
    batched_stage<RP * TCB / NT, NT, float>(
        tid, RP * TCB, [&](int idx) { const int c = idx % RP; return fac_or_zero(Uj + (int64_t)(col0 + idx / RP) * W, c, R); },
        [&](int idx, float v) { sUt[idx % RP][idx / RP] = v; });
  if constexpr (UPD)
    batched_stage<RP * TCB / NT, NT, float>(
        tid, RP * TCB, [&](int idx) { const int c = idx % RP; return fac_or_zero(Vj + (int64_t)(col0 + idx / RP) * W, c, R); },
        [&](int idx, float v) { sVc[idx % RP][idx / RP] = v; });

  v4f yacc[4];
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) yacc[cb] = v4f{0.f, 0.f, 0.f, 0.f};

  for (int cr0 = row0; cr0 < rend; cr0 += CS) {
    __syncthreads();   // the previous chunk's exchange buffer has been read
    if (mwave) {
      static_for<0, CR / 4>([&](auto i) { *reinterpret_cast<f32x4*>(&sP[srow + 4 * i][sgrp * 4]) = pre[i]; });
      static_for<0, VPT>([&](auto i) {
        const int idx = tid + 256 * i;
        sVt[idx % RP][idx / RP] = idx % RP < R ? pv[i] : 0.f;
      });
    } else if constexpr (UPD) {
      static_for<0, VPT>([&](auto i) {
        const int idx = tid - 256 + 256 * i;
        sUr[idx / RP][idx % RP] = idx % RP < R ? pu[i] : 0.f;
      });
    }
    __syncthreads();
    if constexpr (UPD) {
      if (!mwave) {
        if (cr0 + CS < rend) fetch_u(cr0 + CS);
        chunk_update<CR, TCB + FP, RP + FP>(const_cast<float*>(P), ldp, col0, cr0, R, sP, sUr, sVc, wave - 4, lane);
        if (wx) {              // the X exchange below overwrites the chunk: take part in its barriers
          __syncthreads();
          __syncthreads();
        }
        continue;
      }
    }
    if (cr0 + CS < rend) fetch(cr0 + CS);

    // X partial over this wave's 64 columns, two 16-row blocks
    v4f xacc[2] = {v4f{0.f, 0.f, 0.f, 0.f}, v4f{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int g = 0; g < (wx ? 64 : 0); g += 16) {
      const int k0 = wave * 64 + g + 4 * lq;
      const f32x4 b = *reinterpret_cast<const f32x4*>(&sUt[l16][k0]);
#pragma unroll
      for (int mb = 0; mb < 2; ++mb) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(&sP[mb * 16 + l16][k0]);
        xacc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, xacc[mb], 0, 0, 0);
        xacc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, xacc[mb], 0, 0, 0);
        xacc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, xacc[mb], 0, 0, 0);
        xacc[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, xacc[mb], 0, 0, 0);
      }
    }

    // Y^T += V_chunk^T P_chunk for this wave's four 16-column blocks
#pragma unroll
    for (int g = 0; g < (wy ? CR : 0); g += 16) {
      const int r0 = g + 4 * lq;
      const f32x4 a = *reinterpret_cast<const f32x4*>(&sVt[l16][r0]);
#pragma unroll
      for (int cb = 0; cb < 4; ++cb) {
        const int colc = wave * 64 + cb * 16 + l16;
        yacc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, sP[r0][colc], yacc[cb], 0, 0, 0);
        yacc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, sP[r0 + 1][colc], yacc[cb], 0, 0, 0);
        yacc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, sP[r0 + 2][colc], yacc[cb], 0, 0, 0);
        yacc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, sP[r0 + 3][colc], yacc[cb], 0, 0, 0);
      }
    }

    if (!wx) continue;
    // exchange the X partials (sP is no longer read in this chunk)
    __syncthreads();
#pragma unroll
    for (int mb = 0; mb < 2; ++mb)
#pragma unroll
      for (int v = 0; v < 4; ++v) xbuf[((wave * 2 + mb) * 4 + v) * 64 + lane] = xacc[mb][v];
    __syncthreads();
    // thread -> (row block, value, lane) slots of the 32 x 16 outputs
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int slot = tid + 256 * i;          // [mb][v][lane]
      const int ln = slot % 64, v = (slot / 64) % 4, mb = slot / 256;
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < 4; ++w) x += xbuf[((w * 2 + mb) * 4 + v) * 64 + ln];
      const int c = ln % 16;
      const int rr = mb * 16 + 4 * (ln / 16) + v;
      if (c < R) partX[((int64_t)ct * n_pad + cr0 + rr) * pR + c] = x;
    }
  }

  if (!wy || !mwave) return;
#pragma unroll
  for (int cb = 0; cb < 4; ++cb) {
    const int col = col0 + wave * 64 + cb * 16 + l16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int c = 4 * lq + v;
      if (c < R) partY[((int64_t)rt * n_pad + col) * pR + c] = yacc[cb][v];
    }
  }
}

template <bool UPD>
__global__ void __launch_bounds__(UPD ? 512 : 256) k_skinny16_f32(const SkinnyDesc d) {
  skinny16_f32_body<UPD>(static_cast<const float*>(d.src), d.ldp, d.n_pad, d.tile_rows, d.Uj, d.Vj, d.W, d.R,
                         d.partX, d.partY, d.pR, d.want, blockIdx.x, blockIdx.y);
}

template <bool UPD>
__global__ void __launch_bounds__(UPD ? 512 : 256) k_skinny16_f32_multi(const SkinnyDesc* __restrict__ ds, int nd) {
  const SkinnyDesc d = load_desc(ds, find_skinny(ds, nd, (int)blockIdx.x));
  const int local = (int)blockIdx.x - d.block_begin;
  skinny16_f32_body<UPD>(static_cast<const float*>(d.src), d.ldp, d.n_pad, d.tile_rows, d.Uj, d.Vj, d.W, d.R,
                         d.partX, d.partY, d.pR, d.want, local % d.nct, local / d.nct);
}

template <int NB, bool UPD>
__global__ void __launch_bounds__(UPD ? 512 : 256) k_skinny_f32(const SkinnyDesc d) {
  skinny_f32_body<NB, UPD>(static_cast<const float*>(d.src), d.ldp, d.n_pad, d.tile_rows, d.Uj, d.Vj, d.W, d.R,
                           d.partX, d.partY, d.pR, d.want, blockIdx.x, blockIdx.y);
}

template <int NB, bool UPD>
__global__ void __launch_bounds__(UPD ? 512 : 256) k_skinny_f32_multi(const SkinnyDesc* __restrict__ ds, int nd) {
  const SkinnyDesc d = load_desc(ds, find_skinny(ds, nd, (int)blockIdx.x));
  const int local = (int)blockIdx.x - d.block_begin;
  skinny_f32_body<NB, UPD>(static_cast<const float*>(d.src), d.ldp, d.n_pad, d.tile_rows, d.Uj, d.Vj, d.W, d.R,
                           d.partX, d.partY, d.pR, d.want, local % d.nct, local / d.nct);
}

// X-only float pass on the matrix cores: partial X = P U for R <= 16 NB
// factor columns (zero-padded), P streamed from HBM straight into the MFMA
// operand registers: no LDS staging of P, no exchange between waves.
// Block: kXWaves waves over tile_rows rows x 256 columns of P; wave w takes
// the 16-row strips w, w + kXWaves, ..., each read in two halves of 128
// columns, the next half requested before the current one is multiplied.
// v_mfma_f32_16x16x4f32: A (16 x 4): lane l holds A[l % 16][l / 16];
// B (4 x 16): lane l holds B[l / 16][l % 16]; C: element v of lane l is
// C[4 (l / 16) + v][l % 16].  In a 32-column group, lane l reads 4 floats
// of strip row l % 16 at column 4 (l / 16) and 4 at column 16 + 4 (l / 16)
// (each load a contiguous 64-byte segment per row); step e of the group's
// 8 products takes the e-th of these floats as its summation index, and the
// B operand the matching U row.
constexpr int kXWaves = 8;
constexpr int kXRows = 512;   // rows per block where that gives kXBlocks blocks
constexpr int kXBlocks = 512; // else as few (at least a strip per wave) as give so many
inline int xprod_rows(int64_t n_pad) {
  const int64_t nct = n_pad / TCB, ns = (kXBlocks + nct - 1) / nct;
  const int64_t rows = round_up((n_pad + ns - 1) / ns, 16 * kXWaves);
  return rows < kXRows ? (int)rows : kXRows;
}
constexpr int XUS = 4;   // LDS row padding of the U tile (floats): rows 4 apart in distinct banks

template <int NB>
__global__ void __launch_bounds__(64 * kXWaves) k_xprod_f32(const SkinnyDesc d) {
  constexpr int RP = 16 * NB;
  __shared__ float sU[TCB][RP + XUS];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane % 16, lq = lane / 16;
  const int ct = blockIdx.x;
  const int col0 = ct * TCB;
  const int row0 = blockIdx.y * d.tile_rows;
  const int nstrips = (min(row0 + d.tile_rows, d.n_pad) - row0) / 16;
  const float* __restrict__ P = static_cast<const float*>(d.src);

  f32x4 bufA[4][2], bufB[4][2];
  auto load_half = [&](f32x4 (&b)[4][2], const int r, const int h) {
    const float* src = P + (int64_t)(r + l16) * d.ldp + col0 + 128 * h + 4 * lq;
    static_for<0, 4>([&](auto g) {
      b[g][0] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + 32 * g));
      b[g][1] = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src + 32 * g + 16));
    });
  };
  batched_stage<TCB * RP / (64 * kXWaves), 64 * kXWaves, float>(
      tid, TCB * RP,
      [&](int idx) { const int c = idx % RP; return c < d.R ? d.Uj[(int64_t)(col0 + idx / RP) * d.W + c] : 0.f; },
      [&](int idx, float v) { sU[idx / RP][idx % RP] = v; });
  __syncthreads();

  typedef float v4f __attribute__((ext_vector_type(4)));
  v4f acc[NB];
  auto multiply = [&](f32x4 (&b)[4][2], const int h) {
    static_for<0, 4>([&](auto g) {
      static_for<0, 8>([&](auto e) {
        const float a = e < 4 ? b[g][0][e % 4] : b[g][1][e % 4];
        const int k = 128 * h + 32 * g + 4 * lq + (e < 4 ? e : 12 + e);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, sU[k][nb * 16 + l16], acc[nb], 0, 0, 0);
      });
    });
  };

  if (wave < nstrips) load_half(bufA, row0 + 16 * wave, 0);
  for (int st = wave; st < nstrips; st += kXWaves) {
    const int r = row0 + 16 * st;
    // U operands are re-read from LDS in every strip: held in registers across
    // strips (as the compiler would otherwise do) they cost the occupancy
    asm volatile("" ::: "memory");
    load_half(bufB, r, 1);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[nb] = v4f{0.f, 0.f, 0.f, 0.f};
    multiply(bufA, 0);
    if (st + kXWaves < nstrips) load_half(bufA, r + 16 * kXWaves, 0);
    multiply(bufB, 1);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      const int c = nb * 16 + l16;
      if (c < d.R) {
#pragma unroll
        for (int v = 0; v < 4; ++v) d.partX[((int64_t)ct * d.n_pad + r + 4 * lq + v) * d.pR + c] = acc[nb][v];
      }
    }
  }
}

__global__ void __launch_bounds__(256)
k_to_bf16(const float* __restrict__ P, uint16_t* __restrict__ S, int64_t count, const int* __restrict__ gate) {
  if (gate != nullptr && *gate == 0) return;
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= count) return;
  const float4 p = *reinterpret_cast<const float4*>(P + i);
  ushort4 sh;
  sh.x = bf16_rne(p.x); sh.y = bf16_rne(p.y); sh.z = bf16_rne(p.z); sh.w = bf16_rne(p.w);
  *reinterpret_cast<ushort4*>(S + i) = sh;
}

}  // namespace

hipError_t launch_skinny_bf16(int R, const uint16_t* S, int64_t ldp, int64_t n_pad, int tile_rows,
                              const float* slabU, const float* slabV, int W, float* partX, float* partY,
                              hipStream_t s) {
  if (R < 1 || R > kMaxLevelRank || (R > 64 && R % 64 != 0) || n_pad % TCB != 0 || tile_rows % CRB != 0)
    return hipErrorInvalidValue;
  const int nct = (int)(n_pad / TCB);
  const dim3 grid((unsigned)nct, (unsigned)((n_pad + tile_rows - 1) / tile_rows));
  const float* Vj = slabV + (W - R);
  // at most 64 factor columns per launch: two launches of the two-block
  // kernel for R = 128 read the shadow twice but run at twice the occupancy
  // of one four-block launch (whose LDS allows one block per CU)
  const int per = R <= 64 ? R : 64;
  for (int c0 = 0; c0 < R; c0 += per) {
    const SkinnyDesc d{S, ldp, (int)n_pad, tile_rows, slabU + c0, Vj + c0, W, per, partX + c0, partY + c0, R, nct, 0};
    if (skinny_blocks_for(per) == 1)
      hipLaunchKernelGGL((k_skinny_bf16<1>), grid, dim3(256), 0, s, d);
    else
      hipLaunchKernelGGL((k_skinny_bf16<2>), grid, dim3(256), 0, s, d);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_skinny_bf16_multi(int nb, const SkinnyDesc* ds, int nd, int blocks, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  switch (nb) {
    case 1: hipLaunchKernelGGL((k_skinny_bf16_multi<1>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    case 2: hipLaunchKernelGGL((k_skinny_bf16_multi<2>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_fac16(const Fac16Desc& d, hipStream_t s) {
  if (d.cols % 32 != 0 || d.n_pad % 64 != 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_fac16, dim3((unsigned)fac16_blocks(d)), dim3(256), 0, s, d);
  return hipGetLastError();
}

hipError_t launch_fac16_multi(const Fac16Desc* ds, int nd, int blocks, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fac16_multi, dim3((unsigned)blocks), dim3(256), 0, s, ds, nd);
  return hipGetLastError();
}

hipError_t launch_skinny_wide(const uint16_t* S, int64_t ldp, int64_t n_pad, const uint16_t* Ut, const uint16_t* Vt,
                              int R, float* partX, float* partY, hipStream_t s) {
  if (R < kWide16Rank || R > kMaxLevelRank || (R & (R - 1)) != 0 || n_pad % TCB != 0) return hipErrorInvalidValue;
  for (int c0 = 0; c0 < R; c0 += wide_cols(R)) {
    const SkinnyDesc d = wide_desc(S, ldp, n_pad, Ut, Vt, R, c0, partX, partY);
    const dim3 grid((unsigned)wide_blocks(n_pad));
    if (R == 64) hipLaunchKernelGGL((k_skinny_gemm<64>), grid, dim3(256), 0, s, d);
    else hipLaunchKernelGGL((k_skinny_gemm<128>), grid, dim3(256), 0, s, d);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_skinny_wide_multi(int per, const SkinnyDesc* ds, int nd, int blocks, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  switch (per) {
    case 64: hipLaunchKernelGGL((k_skinny_gemm_multi<64>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    case 128: hipLaunchKernelGGL((k_skinny_gemm_multi<128>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_shadow_chain(int R, const ChainDesc& d, int nver, hipStream_t s) {
  if (d.n_pad % TCB != 0 || d.tile_rows % CRB != 0) return hipErrorInvalidValue;
  switch (R) {
    case 1: return shadow_chain_r<1>(d, nver, s);
    case 2: return shadow_chain_r<2>(d, nver, s);
    case 4: return shadow_chain_r<4>(d, nver, s);
    case 8: return shadow_chain_r<8>(d, nver, s);
    case 16: return shadow_chain_r<16>(d, nver, s);
    case 32: return shadow_chain_r<32>(d, nver, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_skinny_f32(int R, const float* P, int64_t ldp, int64_t n_pad, int tile_rows,
                             const float* slabU, const float* slabV, int W, float* partX, float* partY,
                             hipStream_t s, int want, bool update) {
  if (R < 1 || R > kMaxLevelRank || (R > 64 && R % 64 != 0) || n_pad % TCB != 0 || tile_rows % 32 != 0)
    return hipErrorInvalidValue;
  if (update) {
    // one launch over all R columns with the update fused (X and Y both)
    if (!skinny_update_kernel(R) || want != (kWantX | kWantY)) return hipErrorInvalidValue;
    const int nct = (int)(n_pad / TCB);
    const dim3 grid((unsigned)nct, (unsigned)((n_pad + tile_rows - 1) / tile_rows));
    const SkinnyDesc d{P, ldp, (int)n_pad, tile_rows, slabU, slabV + (W - R), W, R, partX, partY, R, nct, 0, want};
    if (R <= 16)
      hipLaunchKernelGGL(k_skinny16_f32<true>, grid, dim3(512), 0, s, d);
    else
      hipLaunchKernelGGL((k_skinny_f32<1, true>), grid, dim3(512), 0, s, d);
    return hipGetLastError();
  }
  if (want == kWantX) {
    // X only: the direct-operand pass (row tiling of its own; the X partials
    // do not depend on it)
    const int nct = (int)(n_pad / TCB);
    const int xrows = xprod_rows(n_pad);
    const dim3 grid((unsigned)nct, (unsigned)((n_pad + xrows - 1) / xrows));
    const int per = R <= 64 ? R : 64;
    for (int c0 = 0; c0 < R; c0 += per) {
      const SkinnyDesc d{P, ldp, (int)n_pad, xrows, slabU + c0, nullptr, W, per, partX + c0, nullptr, R, nct, 0,
                         kWantX};
      if (per <= 16)
        hipLaunchKernelGGL((k_xprod_f32<1>), grid, dim3(64 * kXWaves), 0, s, d);
      else if (per <= 32)
        hipLaunchKernelGGL((k_xprod_f32<2>), grid, dim3(64 * kXWaves), 0, s, d);
      else
        hipLaunchKernelGGL((k_xprod_f32<4>), grid, dim3(64 * kXWaves), 0, s, d);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  const int nct = (int)(n_pad / TCB);
  const dim3 grid((unsigned)nct, (unsigned)((n_pad + tile_rows - 1) / tile_rows));
  const float* Vj = slabV + (W - R);
  // at most 32 factor columns per launch: the one-block kernel (two blocks
  // per CU, no X exchange) twice beats the two-block kernel (one per CU)
  const int per = R <= 32 ? R : 32;
  for (int c0 = 0; c0 < R; c0 += per) {
    const SkinnyDesc d{P, ldp, (int)n_pad, tile_rows, slabU + c0, Vj + c0, W, per, partX + c0, partY + c0, R, nct, 0,
                       want};
    if (skinny_f32_blocks(per) == 0)
      hipLaunchKernelGGL(k_skinny16_f32<false>, grid, dim3(256), 0, s, d);
    else
      hipLaunchKernelGGL((k_skinny_f32<1, false>), grid, dim3(256), 0, s, d);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_skinny_f32_multi(int nb, const SkinnyDesc* ds, int nd, int blocks, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  switch (nb) {
    case 0: hipLaunchKernelGGL(k_skinny16_f32_multi<false>, dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    case 1: hipLaunchKernelGGL((k_skinny_f32_multi<1, false>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    case 2: hipLaunchKernelGGL(k_skinny16_f32_multi<true>, dim3((unsigned)blocks), dim3(512), 0, s, ds, nd); break;
    case 3: hipLaunchKernelGGL((k_skinny_f32_multi<1, true>), dim3((unsigned)blocks), dim3(512), 0, s, ds, nd); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_to_bf16(const float* P, uint16_t* S, int64_t count, hipStream_t s, const int* gate) {
  if (count % 4 != 0) return hipErrorInvalidValue;
  if (count == 0) return hipSuccess;
  hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((count / 4 + 255) / 256)), dim3(256), 0, s, P, S, count, gate);
  return hipGetLastError();
}

}  // namespace lv
