// Internal declarations shared by the HIP translation units of liblinview.
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

namespace lv {

// Every stored power is padded to a multiple of this order; the padding
// rows and columns hold zeros and stay zero under every operation (a zero
// row of P_j or U_j produces zero rows of every product), so no kernel needs
// bounds checks.
constexpr int kPadOrder = 256;
// Largest level rank handled by the register-resident fused pass; larger
// ranks run the skinny products in chunks of this many factor columns.
constexpr int kMaxFusedRank = 16;
// Rows per block of the fused level pass: a wave streams this many rows of
// its 16-byte column group per step (it fixes which wave sums which rows of
// Y, so it is the same at every rank).
constexpr int kFusedRowBlock = 4;
// Memory-side cache of the device (bytes).
constexpr int64_t kCacheBytes = int64_t(256) << 20;
// Largest level of the exponential model (k <= 2^kMaxLevel).
constexpr int kMaxLevel = 10;
// Pipelined batches: at most this many stage streams and factor-slab slots
// (updates in flight).
constexpr int kPipeStreams = 4;
constexpr int kMaxPipeSlots = 24;
// Updates of a batch whose rank is r_pad that go through the levels together
// (a chunk; a level's pass takes up to chain_updates(R) of them at one read
// and write of P), and the chunks in flight.
constexpr int kChainCols = 16;     // factor columns of a pass over several updates
constexpr int kChainUpdates = 8;
constexpr int kPipeChunks = 3;
constexpr int chain_updates(int R) {
  return R >= kChainCols ? 1 : kChainCols / R < kChainUpdates ? kChainCols / R : kChainUpdates;
}
// Work-groups a fused level pass is cut into inside a pipelined batch: one
// per compute unit (the device has 256), so that the passes of two stages
// share every unit instead of one pass filling the device with two
// work-groups per unit.  Returns the work-groups per column tile for nct
// column tiles and ns row slices (each takes ceil(ns / groups) slices;
// never fewer than kPipePassBlocks work-groups in all).
constexpr int kPipePassBlocks = 256;
inline int pipe_slice_groups(int nct, int ns) {
  const int spb = nct * ns / kPipePassBlocks;
  return spb <= 1 ? ns : (ns + spb - 1) / spb;
}

inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// float -> bfloat16 bits, rounding to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint16_t bf16_rne(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

// Columns covered by one tile of the level pass: a wave reads a 1 KiB row
// segment with one 16-byte vector per lane.
template <typename T> constexpr int tile_cols() { return 64 * (16 / (int)sizeof(T)); }
inline __host__ __device__ constexpr int tile_cols_bytes(int elem) { return 64 * (16 / elem); }

// ---- work descriptors ----
// One descriptor per (view, kernel) in a launch.  A single-view launch passes
// one descriptor by value; a multi-view launch passes a device array sorted
// by block_begin (the first work-group of each view) and the work-group
// finds its view by binary search.

// Several updates in one launch: elements from one update's factor slabs and
// partials to the next one's (s: both slabs; x, y, g: partial X, Y and Gram).
struct Strides { int64_t s = 0, x = 0, y = 0, g = 0; };

template <typename T> struct FusedDesc {
  T* P; int64_t ldp; int n_pad; int tile_rows;
  const T* Uj; const T* Vj; int W;      // U_j = Uj[i*W + c], V_j = Vj[i*W + c]
  T* partX; T* partY; double* partG; int pR;
  int nct; int block_begin;             // blocks: nct x ceil(n_pad / tile_rows)
  const T* Ux = nullptr;                // extra X operand (powers' pass of a view with sums)
  T* partX2 = nullptr;                  //   and its partials
  const T* Vy = nullptr;                // Y operand of the passes that update with other factors (row stride
                                        //   Wy); V operand of the Gram in the read-only passes that form it
  const T* Ud = nullptr;                // general form: extra X operand (row stride Wd)
  int Wd = 0, Wy = 0;
  T* partX3 = nullptr;                  //   (Ud) and its partials
};
// (pointers before counts: a round's tables hold one of each per view and level)
template <typename T> struct GramDesc {
  const T* Uj; const T* Vj; double* partG; int W; int n_pad;
  int nrt; int block_begin;             // blocks: nrt x pair chunks (row tiles of gram_rows)
};
template <typename T> struct TailDesc {
  const T* partX; const T* partY; const double* partG; T* slabU; T* slabV;
  int nct; int nrt; int n_pad; int W; int block_begin;   // blocks: ceil(n_pad * R / 256)
  int ng;                                                // Gram partials to add (1: already summed)
};
// Sum of ng Gram partials (count doubles each) into the first.
struct GramSumDesc {
  double* G; int ng; int count; int block_begin;   // blocks: ceil(count / 256)
};
template <typename T> struct UpdateDesc {
  T* P; int64_t ldp; const T* Uj; const T* Vj;
  uint16_t* S;                          // bfloat16 shadow of P rewritten by the pass, or null
  int n_pad; int tile_rows; int W;
  int block_begin;                      // blocks: column tiles x ceil(n_pad / tile_rows)
};
// Products a read-only skinny pass forms.
constexpr int kWantX = 1, kWantY = 2;
// Read-only skinny products of a level on the matrix cores, from the
// bfloat16 shadow of P or from P itself (float): X = P U_j and Y = P^T V_j
// for R columns of the factors (partials with row stride pR, as FusedDesc).
struct SkinnyDesc {
  const void* src; int64_t ldp; int n_pad; int tile_rows;
  const float* Uj; const float* Vj; int W; int R;
  float* partX; float* partY; int pR;
  int nct; int block_begin;             // blocks: nct x ceil(n_pad / tile_rows)
  int want = kWantX | kWantY;           // products formed (float pass only)
  // (products of kWide16Rank and more factor columns from the shadow: Uj and Vj address
  // the factors in bfloat16, transposed, row c = column c, n_pad values)
};
// Factor columns rounded to bfloat16 and transposed: `cols` (a multiple of 32)
// columns of U and of V (row stride W) to the rows of Ut and Vt.
struct Fac16Desc {
  const float* U; uint16_t* Ut;         // first column of U and its row of Ut
  int W; int n_pad; int cols; int dv;   // V's first column is dv columns from U's in the next slab: V = U + n_pad W +
  int block_begin;                      //   dv, Vt = Ut + (W + dv) n_pad; blocks: fac16_blocks
};
inline int fac16_blocks(const Fac16Desc& d) { return d.n_pad / 64 * (d.cols / 32) * 2; }
template <typename T> struct PrepDesc {
  const T* U; int64_t ldu; const T* V; int64_t ldv; int64_t n; T* slabU; T* slabV; int64_t n_pad;
  int r; int r_pad; int W; int block_begin;   // blocks: ceil(n_pad * r_pad / 256)
};

// Descriptor v of a multi-view launch, read through the constant address
// space.  The table is written by the host before the launch and only read
// by it, and the compiler takes pointers loaded from constant memory to
// address global memory: accesses through the descriptor's pointers are then
// global instructions.  Read as ordinary (generic) memory, the pointers would
// be generic too, and their flat accesses count against the LDS wait counter
// as well, so that every wait for an LDS read would also wait for the HBM
// loads in flight.
// (The host pass of the compiler, which only declares the kernels, has no
// address space 4.)
template <typename D> __device__ __forceinline__ D load_desc(const D* ds, int v) {
#if defined(__HIP_DEVICE_COMPILE__)
  return *((const __attribute__((address_space(4))) D*)ds + v);
#else
  return ds[v];
#endif
}

// Tiling of the update pass.  The vector kernel covers tiles of 256 rows x
// (64 lanes x 16 bytes); float storage with rank R >= kMfmaUpdateRank uses
// the matrix-core kernel on 128 x 128 tiles.
constexpr int kUpdateTileRows = 256;
// Level ranks of a plain view run up to kMaxLevelRank (the factors of the
// level below the top; LV_RANK_SWITCH covers 1 .. kMaxLevelRank / 2), the
// top update up to twice that.
constexpr int kMaxLevelRank = 256;
constexpr int kMfmaUpdateRank = 32;
constexpr int kMfmaUpdateTile = 128;
inline __host__ __device__ constexpr bool update_on_mfma(int R, int elem) { return elem == 4 && R >= kMfmaUpdateRank; }
inline int update_tile_rows(int R, int elem) { return update_on_mfma(R, elem) ? kMfmaUpdateTile : kUpdateTileRows; }
// Work-groups a single-view streaming pass aims for, and the rows per
// (interleaved) slice of the vector update pass that give about that many
// for one view of padded order n_pad (several views in one launch keep
// update_tile_rows).
constexpr int kStreamBlocks = 512;
inline int update_slice_rows(int R, int elem, int64_t n_pad) {
  if (update_on_mfma(R, elem)) return kMfmaUpdateTile;
  const int64_t nct = n_pad / tile_cols_bytes(elem);
  int64_t ns = kStreamBlocks / (nct > 0 ? nct : 1);
  const int64_t ns_max = n_pad / (4 * 8);   // at least one 8-row block per wave
  ns = ns < 1 ? 1 : ns > ns_max ? ns_max : ns;
  return (int)((n_pad + ns - 1) / ns);
}
inline __host__ __device__ constexpr int update_tile_cols(int R, int elem) { return update_on_mfma(R, elem) ? kMfmaUpdateTile : tile_cols_bytes(elem); }
// Rows per partial of the stand-alone Gram kernel, and its partial count.
constexpr int kGramRows = 64;
inline int gram_tiles(int64_t n_pad) { return (int)(n_pad / kGramRows); }
// Float storage with level rank R >= kMfmaSkinnyRank forms the skinny
// products on the matrix cores in a read-only pass (then Gram, update);
// smaller ranks use the fused vector pass.
constexpr int kMfmaSkinnyRank = 16;
inline bool skinny_on_mfma(int R, int elem) { return elem == 4 && R >= kMfmaSkinnyRank; }
// Whether the fused pass of rank R forms the Gram partials itself (one per
// row tile); otherwise the stand-alone Gram kernel and its sum provide G.
inline bool gram_in_pass(int R, int elem) { return R <= kMaxFusedRank && !skinny_on_mfma(R, elem); }
// The powers' fused pass of a level with rank R can also form X for Q_j (R
// more columns, views with sums) and for xd columns of a general-form operand
// (xd a power of two up to 8) when the level runs the fused vector pass and
// the X width stays within kFusedXCap columns (one lane per X sum of a block).
constexpr int kFusedXCap = 64 / kFusedRowBlock;
inline bool fused_extra_fits(int R, bool q, int xd) {
  return R <= 8 && (xd == 0 || xd == 1 || xd == 2 || xd == 4 || xd == 8) && R + (q ? R : 0) + xd <= kFusedXCap;
}
inline bool fused_vector_level(int R, int elem, bool shadowed) { return !shadowed && !skinny_on_mfma(R, elem); }
// The sums pass (Y = S^T V_j and the rank update of S in one pass) on the
// vector kernel, below the ranks that run on the matrix cores.
inline bool sums_fused(int R, int elem) { return R <= kMaxFusedRank && !skinny_on_mfma(R, elem); }
// Rows per slice of a level pass of rank R over a matrix of padded order
// n_pad, for a view's tile rows.  The passes take (column tile, row slice)
// work-groups, and 512-row slices leave most of the device idle below
// n_pad = 8192 (128 work-groups at 4096, 4 at 512).  The default height,
// kTileRows, therefore stands for 512 rows or as many as give kFillBlocks
// work-groups (one per compute unit), whichever is less, but not below 8 R rows, so that
// a slice's Y partial stays under 1/16 of the bytes it streams (matrix-core
// passes, `cores`, take 32 columns at a time: not below 256 rows; FP32 rank 64
// at n = 4096, 128 work-groups of 512 rows: 57 us a pass, 256 of 256: 36 us), nor
// below `unit` rows: a block of kFusedRowBlock rows for each of the four waves,
// or a 64-row chunk of the matrix-core passes.  Where 8 R rows leave a vector
// pass fewer than kFillBlocks work-groups, latency and not the partials bounds
// it: down to 2 R rows (FP64 rank-4 update, k = 16: n = 256 174 -> 118 us, 1024
// 173 -> 133 us, 1536 213 -> 194 us; rank 1, n = 512 66 -> 61 us).  A single FP64 update at
// n = 256: 102 us at 512 rows, 46 us so; the read-only float pass at n = 4096
// 38 us and 22 us.  Other heights are taken as they are: rounds over many
// views fill the device anyway and lose by finer slices (32 views of 512 to
// 4096: 2.34 ms with tuned heights, 2.52 ms when every height was cut).
//   Pass and tail of one update by the rule against the best of 64, 128, 256 and
// 512 rows, us: FP32 n = 512 rank 1 13 (14), rank 8 17 (22), rank 32 54 (39);
// n = 2048 17 (17), 23 (23), 61 (53); n = 4096 33 (33), 47 (43), 91 (91); n = 8192
// 96 (97), 111 (113), 227 (228); n = 16384 391 (366), 439 (438), 802 (798); FP64
// ranks 1 to 16 and n = 512 to 8192 within 5%.  The 256-row limit of the
// matrix-core passes costs most, at n <= 2048.
constexpr int kTileRows = 512;      // default rows per tile: the most rows of the default cut
//
// Twice as many work-groups for passes that only read (`reads`) and for 128
// and more bytes of factors per row, whose long row blocks leave one wave per
// SIMD waiting: OLS row change n = 4096 63 -> 60 us, IncrLin n = 5000 1.63 -> 1.56
// ms, FP64 rank-3 batch n = 3001 1.90 -> 1.81 ms; the other updating passes
// lose by it (FP32 update n = 4194 217 -> 228 us).  Matrix-core passes run two
// work-groups per compute unit, so they take at most that many (n = 7168, rank
// 32 from the shadow: 532 of them 40 us, 448 32 us).
constexpr int kFillBlocks = 256;
inline int slice_rows(int64_t n_pad, int elem, int R, bool cores, bool reads = false) {
  const int unit = cores ? 64 : 4 * kFusedRowBlock;
  const int64_t nct = n_pad / tile_cols_bytes(elem);
  const int64_t fill = reads || R * elem >= 128 ? 2 * kFillBlocks : kFillBlocks;
  const int64_t ns = cores ? (fill > nct ? fill / nct : 1) : (fill + nct - 1) / nct;
  int64_t rows = round_up((n_pad + ns - 1) / ns, unit);
  int least = cores && 8 * R > 256 ? 256 : 8 * R;
  if (!cores && R <= kMaxFusedRank && nct * (n_pad / least) < kFillBlocks) least = 2 * R;
  if (rows < least) rows = round_up(least, unit);
  return rows < kTileRows ? (int)rows : kTileRows;
}

// The tail at this level rank: one column per lane and kTailRowsPerThread rows
// per thread.
constexpr int kSlicedTailRank = 16;
constexpr int kTailRowsPerThread = 4;
inline int tail_block_rows(int R) { return 256 / R * kTailRowsPerThread; }
// Lanes per output entry of the tail below kSlicedTailRank.
constexpr int kTailLanes = 8;
// Ranks whose Gram and tail run on the double matrix cores, the 16-column
// blocks that a wave of the tail takes (enough waves for the device at the low
// ranks), the pairs per side of a Gram work-group, and the rows of its tile.
constexpr int kMfmaGramRank = 32;
inline __host__ __device__ constexpr int tail_wave_blocks(int R) { return R < 64 ? 1 : R < 256 ? 2 : 4; }
inline __host__ __device__ constexpr int gram_block(int R) { return R < 64 ? 32 : 64; }
inline __host__ __device__ constexpr int gram_rows(int R) { return R <= 64 ? kGramRows : R; }
inline int gram_count(int64_t n_pad, int R) { return (int)((n_pad + gram_rows(R) - 1) / gram_rows(R)); }
inline int tail_blocks(int64_t n_pad, int R) {
  if (R >= kMfmaGramRank) return (int)(n_pad / 64) * (R / (16 * tail_wave_blocks(R)));
  return R >= kSlicedTailRank ? (int)(n_pad / tail_block_rows(R))
                              : (int)((n_pad * R * kTailLanes + 255) / 256);
}
inline int gram_chunks(int R) {   // work-groups per row tile
  return R >= kMfmaGramRank ? (R / gram_block(R)) * (R / gram_block(R)) : 1;
}

// ---- launchers (stream-ordered; return the launch status) ----

// dst[i*ldd + j] = (i < n && j < n) ? src[i*lds + j] : 0 for i, j < n_pad.
// With a non-null `gate`, the kernel does nothing unless *gate != 0 (read on
// the device, so a decision taken by an earlier kernel needs no host sync).
template <typename Tin, typename Tout>
hipError_t launch_copy_pad(const Tin* src, int64_t lds, int64_t n, Tout* dst, int64_t ldd,
                           int64_t n_pad, hipStream_t s, const int* gate = nullptr);

// Factor slab set-up: slab U columns [0, r_pad) and slab V columns
// [W - r_pad, W) receive U and V (n x r), zero-filled up to r_pad columns and
// n_pad rows.  nver > 1: that many updates, strideU / strideV apart in U and V
// and sstride apart in the slabs.
template <typename T>
hipError_t launch_prep(const T* U, int64_t ldu, const T* V, int64_t ldv, int64_t n, int r,
                       int r_pad, T* slabU, T* slabV, int W, int64_t n_pad, hipStream_t s, int nver = 1,
                       int64_t strideU = 0, int64_t strideV = 0, int64_t sstride = 0);

// Fused level pass for level rank R: partial X = P U_j, partial Y = P^T V_j,
// partial Gram V_j^T U_j (column tile 0 only), and P += U_j V_j^T, in one
// read and one write of P.  slice_groups > 0: that many work-groups per
// column tile, each taking several row slices in turn (same partials, bit
// for bit; see pipe_slice_groups).  nver > 1 (a power of two up to
// chain_updates(R)): nver successive updates in the one read and write, the
// same results as nver launches.
template <typename T>
hipError_t launch_level_fused(int R, T* P, int64_t ldp, int64_t n_pad, int tile_rows,
                              const T* slabU, const T* slabV, int W, T* partX, T* partY,
                              double* partG, hipStream_t s, int slice_groups = 0, int nver = 1,
                              const Strides& vs = {});

// Tail of level j: reduce partials in a fixed order, G = sum of the ng
// partial Grams, U_{j+1} = [U_j, X + U_j G], V_{j+1} = [Y, V_j].
template <typename T>
hipError_t launch_level_tail(int R, const T* partX, const T* partY, const double* partG,
                             int nct, int nrt, int ng, int64_t n_pad, T* slabU, T* slabV, int W,
                             hipStream_t s, int nver = 1, const Strides& vs = {});

// Update-only pass: P += U_j V_j^T for rank R (the top stored power).  With a
// non-null shadow S (float only) the pass also writes S = bf16(P) of the new
// values.  `split` (float, bfloat16-shadow mode) forms the matrix-core ranks
// with split bfloat16 operands (three products) instead of float products.
template <typename T>
hipError_t launch_level_update(int R, T* P, int64_t ldp, int64_t n_pad, const T* slabU,
                               const T* slabV, int W, hipStream_t s, uint16_t* S = nullptr,
                               bool split = false);

// P += U_t V_t^T for nver successive updates (rank R >= 4, slabs sstride
// apart) in one read and one write of P, each delta formed from zero and added
// once: the results of nver launch_level_update calls bit for bit.
template <typename T>
hipError_t launch_level_update_chain(int R, T* P, int64_t ldp, int64_t n_pad, const T* slabU, const T* slabV, int W,
                                     int nver, int64_t sstride, hipStream_t s, bool split = false);

// Gram V_j^T U_j in double: gram_count(n_pad, R) partials of gram_rows(R) rows,
// then their sum in fixed order into partG[0 .. R*R).
template <typename T>
hipError_t launch_level_gram(int R, const T* slabU, const T* slabV, int W, int64_t n_pad, double* partG,
                             hipStream_t s, int nver = 1, const Strides& vs = {});
hipError_t launch_gram_sum_multi(const GramSumDesc* ds, int nd, int blocks, hipStream_t s);

// Skinny products of level rank R (<= kMaxLevelRank) from the bfloat16 shadow S on the
// matrix cores (bf16 x bf16 -> fp32): partial X = S U_j, partial Y = S^T V_j
// over tiles of tile_rows x 256 (partials as for the fused pass, row stride R).
hipError_t launch_skinny_bf16(int R, const uint16_t* S, int64_t ldp, int64_t n_pad, int tile_rows,
                              const float* slabU, const float* slabV, int W, float* partX, float* partY,
                              hipStream_t s);
hipError_t launch_skinny_bf16_multi(int nb, const SkinnyDesc* ds, int nd, int blocks, hipStream_t s);
// Factor blocks of 32 columns the bfloat16 skinny kernel needs for rank R.
inline int skinny_blocks_for(int R) { return R <= 32 ? 1 : 2; }   // R <= 64 per launch

// Level ranks R >= kWide16Rank with shadows: the same products from bfloat16
// factors kept transposed (Ut, Vt: rows are the R factor columns), 64 or 128
// factor columns per launch.  The summation ranges are split wide_splits()
// ways, about two work-groups per compute unit in all and at least 512 rows or
// columns each, with one partial of X and one of Y per split (n_pad / 512 at
// most, fewer than the passes over 2-D tiles leave).  A split has at most
// kWideTerms terms whatever the order: its sum is a float chain (see
// skinny_gemm_body for the bound), while the partials are added in double.
constexpr int kWide16Rank = 64;
constexpr int kWideTerms = 2048;
inline __host__ __device__ int wide_splits(int64_t n_pad) {
  const int64_t tiles = n_pad / 128 * 2;   // X and Y products of a launch
  const int64_t want = (512 + tiles - 1) / tiles, most = n_pad / 512;
  const int64_t least = (n_pad + kWideTerms - 1) / kWideTerms;
  const int64_t s = want < most ? want : most;
  return (int)(s < least ? least : s);
}
inline int wide_cols(int R) { return R < 128 ? R : 128; }
inline int wide_blocks(int64_t n_pad) { return (int)(2 * (n_pad / 128)) * wide_splits(n_pad); }
inline int wide_blocks(const SkinnyDesc& d) { return wide_blocks((int64_t)d.n_pad); }
inline SkinnyDesc wide_desc(const void* S, int64_t ldp, int64_t n_pad, const uint16_t* Ut, const uint16_t* Vt, int R,
                            int c0, float* partX, float* partY) {
  return {S, ldp, (int)n_pad, 0, reinterpret_cast<const float*>(Ut + (int64_t)c0 * n_pad),
          reinterpret_cast<const float*>(Vt + (int64_t)c0 * n_pad), 0, wide_cols(R), partX + c0, partY + c0, R, 0, 0};
}
hipError_t launch_fac16(const Fac16Desc& d, hipStream_t s);
hipError_t launch_fac16_multi(const Fac16Desc* ds, int nd, int blocks, hipStream_t s);
hipError_t launch_skinny_wide(const uint16_t* S, int64_t ldp, int64_t n_pad, const uint16_t* Ut, const uint16_t* Vt,
                              int R, float* partX, float* partY, hipStream_t s);
// Shadowed levels of rank R <= kChain16Rank for nver = 2 or 4 successive
// updates of a batch: the factors' operand forms, then both products
// and the update of each in turn at one read and write of P.  f16, f32:
// chain_factor_bytes(n_pad, R) in all for each update; partials as the single
// updates' ones with row stride R, vs apart; S is rewritten.
constexpr int kChain16Rank = 32;
constexpr int kChain16Updates = 4;   // the larger of the two
constexpr int chain16_updates(int R) { return R < 32 ? 4 : 2; }
struct ChainDesc {
  float* P; uint16_t* S; int64_t ldp; int n_pad; int tile_rows;
  const float* U; const float* V; int W;   // first update's U_j and V_j
  uint16_t* f16; void* f32;
  float* partX; float* partY; Strides vs;
};
inline size_t chain_f16_bytes(int64_t n_pad, int R) { return (size_t)n_pad * 4 * R; }                  // per update
inline size_t chain_f32_bytes(int64_t n_pad, int R) { return (size_t)n_pad * 8 * (R < 4 ? 4 : R); }    // per update
hipError_t launch_shadow_chain(int R, const ChainDesc& d, int nver, hipStream_t s);
hipError_t launch_skinny_wide_multi(int per, const SkinnyDesc* ds, int nd, int blocks, hipStream_t s);

// The same products from the float power P (v_mfma_f32_32x32x2f32, float
// products and accumulation), R <= kMaxLevelRank (32 factor columns per launch; X alone: 64).
// update: also apply P += U_j V_j^T in the same pass (one read and one write
// of P; R = 16 or 32, X and Y both, see skinny_fuses_update).
hipError_t launch_skinny_f32(int R, const float* P, int64_t ldp, int64_t n_pad, int tile_rows,
                             const float* slabU, const float* slabV, int W, float* partX, float* partY,
                             hipStream_t s, int want = kWantX | kWantY, bool update = false);
// nb: the width class below, plus 2 for the update-fused kernels.
hipError_t launch_skinny_f32_multi(int nb, const SkinnyDesc* ds, int nd, int blocks, hipStream_t s);
// Width class of a float skinny launch of at most 32 factor columns (0: the
// 16-wide pass for R <= 16; 1: one 32-column factor block).
inline int skinny_f32_blocks(int R) { return R <= 16 ? 0 : 1; }
// Float level ranks whose skinny pass on the matrix cores also applies the
// rank update (a second pass over P would otherwise follow).  The kernels
// take R = 16 or 32; at 32 the fused block (one per CU by its LDS, one
// 32-row chunk in flight) is slower than the skinny pass plus the update
// pass (839 vs 771 us at n = 16384), so only R = 16 uses it.
inline bool skinny_fuses_update(int R) { return R == 16; }
inline bool skinny_update_kernel(int R) { return R == 16 || R == 32; }

// S = bf16(P) for `count` consecutive floats (count a multiple of 4); with a
// non-null gate only when *gate != 0.
hipError_t launch_to_bf16(const float* P, uint16_t* S, int64_t count, hipStream_t s,
                          const int* gate = nullptr);

// ---- sums of powers (views with LV_WITH_SUMS)

// Read-only pass: partial X = P Uop and, with a non-null partY, Y = P^T Vop for
// R columns (row stride R), P unchanged (fused kernel without its update).
template <typename T>
hipError_t launch_level_readonly(int R, const T* P, int64_t ldp, int64_t n_pad, int tile_rows, const T* Uop,
                                 const T* Vop, int W, T* partX, T* partY, hipStream_t s);
// The powers' fused pass with extra X columns (fused_extra_fits): as
// launch_level_fused for level rank R, and in the same read of P
// X = P Q_j (slabQ non-null; Q_j = columns [0, R) of slabQ, partials to
// partXq, [nct][n_pad][R]) and X = P D (Dop non-null; xd columns with row
// stride ldd, partials to partXd, [nct][n_pad][xd]).
template <typename T>
hipError_t launch_level_fused_x(int R, T* P, int64_t ldp, int64_t n_pad, int tile_rows, const T* slabU,
                                const T* slabV, int W, T* partX, T* partY, double* partG, const T* slabQ, T* partXq,
                                const T* Dop, int ldd, int xd, T* partXd, hipStream_t s);
// The sums pass (R <= 16): partial Y = S^T V_j with the old S (V_j = columns
// [W - R, W) of slabV; partials [nrt][n_pad][R]) and S += Q_j W_j^T, one read
// and one write of S.
template <typename T>
hipError_t launch_sums_fused(int R, T* S, int64_t ldp, int64_t n_pad, int tile_rows, const T* slabQ,
                             const T* slabW, const T* slabV, int W, T* partY, hipStream_t s);
// One launch for a step of the linear and skip models (RY <= 8 columns, R <=
// 16, powers of two, RY <= R): partial X = P_a M and the Gram partials
// V_a^T M (one per slice, RY x RY doubles) with M RY columns of row stride
// Wb; partial Y = P_b^T V_a with the old P_b and P_b += U_b V_b^T (R columns,
// row stride Wb), P_b read and written once.  V_a has row stride Wa; rows_x,
// rows_y are the rows per slice of the two passes.
template <typename T>
hipError_t launch_krylov_step(int R, int RY, const T* Pa, T* Pb, int64_t ldp, int64_t n_pad, int rows_x, int rows_y,
                              const T* M, const T* Ub, const T* Vb, int Wb, const T* Va, int Wa, T* partX, T* partY,
                              double* partG, hipStream_t s);
// Read-only, R <= 8: partial X = P U (row stride W), the Gram partials of
// V^T U (row stride Wv; one per slice, R x R doubles) and, with a non-null
// partY (Wv = W), partial Y = P^T V.
template <typename T>
hipError_t launch_fused_xgram(int R, const T* P, int64_t ldp, int64_t n_pad, int tile_rows, const T* U, int W,
                              const T* V, int Wv, T* partX, T* partY, double* partG, hipStream_t s);
// The next factor block of a model whose products share their left operand
// (U_c = [U_b, f(last wa columns of U_b)], f(M) = P_a M + U_a (V_a^T M); V_c =
// [P_b^T V_a, V_b]): per row, wa columns of X (nct partials [nct][n_pad][wa])
// plus U_a G, with G the sum of ng partials (wa x wa doubles, wa <= 8 if
// ng > 1), go to Uc + wb; with Ub non-null U_b (wb columns) goes before them;
// with Vc non-null wa columns of Y (nrt partials [nrt][n_pad][wa]) go to Vc,
// V_b after them, and zeros to columns wa + wb .. Wc - 1 of Uc and Vc.  Row
// strides: Ua Wa, Ub and Vb Wb, Uc and Vc Wc.
constexpr int kMaxKrylovCols = 8;     // columns that the vector passes of these steps take
template <typename T>
hipError_t launch_krylov_tail(int wa, const T* partX, int nct, const T* partY, int nrt, const double* partG, int ng,
                              const T* Ua, int Wa, const T* Ub, const T* Vb, int Wb, int wb, T* Uc, T* Vc, int Wc,
                              int64_t n_pad, hipStream_t s);

// G = Vop^T Uop (R x R, double) into partG[0 .. R*R), operands given by
// their first columns (row stride W).
template <typename T>
hipError_t launch_gram_cols(int R, const T* Uop, const T* Vop, int W, int64_t n_pad, double* partG, hipStream_t s);
// Factors of the next level's sums (see k_sums_tail): Q_{j+1} = [U_j, X + Q_j],
// W_{j+1} = [Y + W_j G, W_j]; `first` for level 0 (Q_0 = 0, S_0 = I).
template <typename T>
hipError_t launch_sums_tail(int R, const T* partX, const T* partY, const double* G, int nct, int nrt, int64_t n_pad,
                            T* slabQ, T* slabW, const T* slabU, const T* slabV, int W, bool first, hipStream_t s);
// S = I (n x n identity, zero padding to n_pad); dst += src (count elements).
// With a non-null gate only when *gate != 0.
template <typename T>
hipError_t launch_set_identity(T* S, int64_t ld, int64_t n, int64_t n_pad, hipStream_t s, const int* gate = nullptr);
template <typename T>
hipError_t launch_add(T* dst, const T* src, int64_t count, hipStream_t s, const int* gate = nullptr);

// ---- general form T_{i+1} = A T_i + B (hybrid deltas)

// part[0 .. R*p) = A^T B (double) for A n_pad x R (lda), B n_pad x p (ldb):
// 64-row partials, then their fixed-order sum (part holds n_pad / 64 partials).
template <typename T>
hipError_t launch_atb(int R, int p, const T* A, int64_t lda, const T* B, int64_t ldb, int64_t n_pad, double* part,
                      hipStream_t s);
// Several such products (and their sums) in one launch each: the small
// products of a level wait for the same factors, and each alone is shorter
// than a launch.
constexpr int kMaxAtbJobs = 4;
template <typename T> struct AtbJob { int R, p; const T* A; int64_t lda; const T* B; int64_t ldb; double* part; };
template <typename T> struct AtbJobs {
  AtbJob<T> job[kMaxAtbJobs]; int cnt = 0;
  void add(int R, int p, const T* A, int64_t lda, const T* B, int64_t ldb, double* part) {
    job[cnt++] = {R, p, A, lda, B, ldb, part};
  }
};
template <typename T>
hipError_t launch_atb_jobs(const AtbJobs<T>& jobs, int64_t n_pad, hipStream_t s);
// D = sum of nct partials of X + U a (+ Q b if Q is non-null), T += D
// (n_pad x pp; U, Q with row stride W and R columns; a, b R x pp double).
template <typename T>
hipError_t launch_general_tail(const T* partX, int nct, const T* U, const T* Q, int W, int R, const double* a,
                               const double* b, T* D, T* Tm, int64_t n_pad, int pp, hipStream_t s);
// C = A B (+ C0 if non-null), A n_pad x n_pad (lda), B, C, C0 n_pad x pp,
// double; pp in {1, 2, 4, ..., 64}.  With a non-null gate only when *gate != 0.
hipError_t launch_gemm_np(int pp, const double* A, int64_t lda, const double* B, double* C, const double* C0,
                          int64_t n_pad, hipStream_t s, const int* gate = nullptr);
// dst (n_pad x pp, contiguous) = src (n x p, ld lds) zero-padded.
template <typename Tin, typename Tout>
hipError_t launch_copy_rect(const Tin* src, int64_t lds, int64_t n, int p, Tout* dst, int64_t n_pad, int pp,
                            hipStream_t s, const int* gate = nullptr);
// Factored general-form deltas (Delta T_j = Y_j Z_j^T):
// Ynew (n_pad x WYn) = [U_j (R cols, row stride W), sum of nct partials of
// P_j Y_j (width wy, partial row stride pR) + U_j G (G R x ldg double),
// Q_j (R cols, stride W; zero if Q is null), 0 ...].
template <typename T>
hipError_t launch_gfac_y(const T* partX, int nct, int pR, const T* U, const T* Q, int W, int R, const double* G,
                         int ldg, int wy, T* Ynew, int WYn, int64_t n_pad, hipStream_t s);
// Ztnew (WYn x pp, factor-major) = [a (R x pp, double), Zt_j (wy rows),
// b (R x pp, double; zero if null), 0 ...].
template <typename T>
hipError_t launch_gfac_z(const double* a, const T* Zt, int wy, const double* b, int R, T* Ztnew, int WYn, int pp,
                         hipStream_t s);
// Tm (n_pad x pp) += Y (w columns, row stride sy) Zt (w x pp), double sums.
// (jobs: up to kMaxRectJobs such updates of different Tm in one launch.)
// cnt > 1: for i = 0 .. cnt - 1, Tm + i tstride, the first (i + 1) w columns
// of Y, and Zt from row (cnt - 1 - i) w on.
template <typename T>
hipError_t launch_rank_rect(T* Tm, const T* Y, int sy, const T* Zt, int w, int64_t n_pad, int pp, hipStream_t s,
                            int cnt = 1, int64_t tstride = 0);
constexpr int kMaxRectJobs = 16;
template <typename T> struct RectJob { T* Tm; const T* Y; const T* Zt; int sy, w; };
template <typename T> struct RectJobs { RectJob<T> job[kMaxRectJobs]; };
template <typename T>
hipError_t launch_rank_rect_jobs(const RectJobs<T>& jobs, int cnt, int64_t n_pad, int pp, hipStream_t s);
// Z (cnt R x pp, rows in blocks of R): block cnt - 1 - i = V^T T_i for T_i =
// Tm + i tstride (n_pad x pp), V n_pad x R; part holds cnt vtt_tiles(n_pad, R
// pp) R pp doubles.
inline int vtt_rows(int pairs) { return pairs < 256 ? 256 : 64; }
inline int vtt_tiles(int64_t n_pad, int pairs) { return (int)(n_pad / vtt_rows(pairs)); }
template <typename T>
hipError_t launch_vtt(int R, int pp, const T* V, const T* Tm, int64_t tstride, int cnt, int64_t n_pad, double* part,
                      T* Z, hipStream_t s);

// Multi-view launches over device descriptor arrays (nd descriptors,
// `blocks` work-groups in total).  `chunk` selects the read-only skinny pass
// over 16 factor columns used for level ranks above kMaxFusedRank.
template <typename T>
hipError_t launch_fused_multi(int R, bool chunk, const FusedDesc<T>* ds, int nd, int blocks, hipStream_t s);
template <typename T>
hipError_t launch_gram_multi(int R, const GramDesc<T>* ds, int nd, int blocks, hipStream_t s);
template <typename T>
hipError_t launch_tail_multi(int R, const TailDesc<T>* ds, int nd, int blocks, hipStream_t s);
template <typename T>
hipError_t launch_update_multi(int R, bool shadow, bool split, const UpdateDesc<T>* ds, int nd, int blocks,
                               hipStream_t s);
template <typename T>
hipError_t launch_prep_multi(const PrepDesc<T>* ds, int nd, int blocks, hipStream_t s);

// C = A * B for n_pad x n_pad row-major matrices (n_pad a multiple of 256),
// on MFMA (double: 16x16x4 f64; float: 32x32x2 f32).
template <typename T>
hipError_t launch_gemm(const T* A, int64_t lda, const T* B, int64_t ldb, T* C, int64_t ldc,
                       int64_t n_pad, hipStream_t s, const int* gate = nullptr);
// C = A * B for A M x K, B K x N (M, N multiples of 128, K of 16), same kernel;
// splits > 1: that many partial products, M ldc values apart.
template <typename T>
hipError_t launch_gemm_rect(const T* A, int64_t lda, const T* B, int64_t ldb, T* C, int64_t ldc, int64_t M,
                            int64_t N, int64_t K, hipStream_t s, const int* gate = nullptr, int splits = 1);

// ---- drift check (FP64 test of the stored chain P_{j+1} = P_j P_j)

// x = z zero-padded to n_pad (double).
hipError_t launch_vec_pad(const double* z, int64_t n, double* x, int64_t n_pad, hipStream_t s);
hipError_t launch_sign_vector(double* z, int64_t n, int64_t n_pad, unsigned long long seed, hipStream_t s);

// y = P x with double accumulation, P n_pad x n_pad (ld ldp) of type T.
template <typename T>
hipError_t launch_matvec(const T* P, int64_t ldp, int64_t n_pad, const double* x, double* y,
                         hipStream_t s);

// rho_j = max|Pz[j+1] - PPz[j]| / max|Pz[j+1]| for j < m (Pz, PPz: n_pad
// doubles per level); *gate = (some rho_j > tau or not finite); the
// counter is incremented when the gate opens.
hipError_t launch_drift_residual(const double* Pz, const double* PPz, int m, int64_t n_pad,
                                 double tau, double* residuals, int* gate,
                                 unsigned long long* counter, hipStream_t s);

}  // namespace lv
