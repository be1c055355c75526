// Internal view state shared by the C-ABI translation units: workspace
// layout of a view, the view handle, and error helpers.
#pragma once

#include "linview.h"
#include "lv_internal.h"

#include <cstdarg>
#include <cstdio>
#include <vector>

namespace lv {

// Message of the last failure on this host thread (set by fail()).
extern thread_local char g_err[512];
lv_status fail(lv_status st, const char* fmt, ...);

inline bool is_pow2(int64_t x) { return x > 0 && (x & (x - 1)) == 0; }
inline int ilog2(int64_t x) { int m = 0; while ((int64_t(1) << m) < x) ++m; return m; }
inline int64_t next_pow2(int64_t x) { int64_t p = 1; while (p < x) p <<= 1; return p; }

constexpr size_t kAlign = 256;
constexpr int64_t kMaxOrder = 65536;
constexpr int kMaxK = 1024;
constexpr int kMaxWidth = 2 * kMaxLevelRank;   // k * r_pad: width of the top-level factors
// A pass over several updates addresses their factor entries by 32-bit byte
// offsets from the first one's block: the last update's slab pair and a row
// block of it stay below 2^31 (a pair's rows are widest in floats, and as long
// in doubles, whose width stops at kMaxLevelRank).
static_assert(((kChainUpdates - 1) * 2 * kMaxOrder + kFusedRowBlock) * kMaxWidth * (int64_t)sizeof(float) < (int64_t(1) << 31) &&
                  ((kChainUpdates - 1) * 2 * kMaxOrder + kFusedRowBlock) * kMaxLevelRank * (int64_t)sizeof(double) <
                      (int64_t(1) << 31),
              "32-bit offsets of a shared pass");
constexpr int kMinTileRows = 256;   // tile rows a level pass may be set to:
constexpr int kMaxTileRows = 1024;  //   multiples of 64 in [256, 1024]

inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Rows per slice of a pass at the default height: `rows` (slice_rows), or as
// many more, up to the plain kTileRows, as it takes for the partials of ns
// slices, bytes(ns), to fit in room bytes: workspaces hold the partials of
// kTileRows rows, and the finer cut only where idle regions take the rest.
template <typename F>
inline int fitted_rows(int64_t n_pad, int rows, bool cores, size_t room, F bytes) {
  const int unit = cores ? 64 : 4 * kFusedRowBlock;
  while (rows < kTileRows && bytes((n_pad + rows - 1) / rows) > room) rows += unit;
  return rows < kTileRows ? rows : kTileRows;
}

struct Layout {
  int64_t n_pad = 0, ldp = 0;
  int m = 0, r_pad = 0, W = 0, elem = 0, nct = 0;
  size_t P[kMaxLevel + 1] = {};
  size_t slabU = 0, slabV = 0;   // the update's factor slabs (every level's U_j, V_j)
  size_t slot_stride = 0;        // bytes of a slab pair (V follows U directly)
  bool piped = false;            // lv_view_update_batch may pipeline (plain views with m >= 2)
  bool wide16 = false;           // shadows: levels from rank kWide16Rank take transposed bfloat16 factors
  // n_pad x r_pad zeros (set at creation): the factors of the zero updates
  // that lv_view_autotune times (P + 0 0^T = P exactly)
  size_t zfac = 0;
  size_t shadow[kMaxLevel] = {};   // bfloat16 copies of P_0..P_{m-1} (LV_FP32_BF16SHADOW)
  // sums of powers (LV_WITH_SUMS): S_1 = I, S_2, ..., S_k and their factor
  // slabs Q (prefix columns) and W (suffix columns)
  bool sums = false;
  size_t S[kMaxLevel + 1] = {};
  size_t slabQ = 0, slabW = 0;
  // general form T_{i+1} = A T_i + B with hybrid deltas (implies sums): p
  // columns padded to pp, T_1, T_2, ..., T_k and T_0, B (storage type, n_pad x
  // pp), the deltas D (two, ping-pong), FP64 partials of V_j^T T_j and W_j^T B
  bool general = false;
  int p = 0, pp = 0;
  // factored deltas Delta T_j = Y_j Z_j^T instead (LV_GENERAL_FACTORED):
  // p padded to a multiple of 128; Y_j slabs (n_pad x WY[j], true width
  // wy[j]; Y_0 is the prefix of the powers' U slab), Z_j kept transposed
  // (WY[j] x pp), FP64 partials of V_j^T Y_j
  bool gfac = false;
  int wy[kMaxLevel + 1] = {};
  int WY[kMaxLevel + 1] = {};
  size_t Y[kMaxLevel + 1] = {};
  size_t Zt[kMaxLevel + 1] = {};
  size_t atbG = 0;
  // skip-s model (factored deltas only): the powers and sums stop at
  // P_s = P_{2^m}; T_{2s}, T_{3s}, ..., T_{kT} follow T_{js} = P_s T_{(j-1)s} + S_s B
  // (nsk of them, uniform strides), with factor slabs of widths wsk(q)
  int kT = 0, nsk = 0;
  size_t Tsk = 0, Ysk = 0, Ztsk = 0, tstride = 0, ystride = 0, zstride = 0;
  int wsk(int q) const { return wy[m] + q * 2 * (r_pad << m); }
  int WYsk(int q) const { return (int)next_pow2(wsk(q)); }
  size_t T[kMaxLevel + 1] = {};
  size_t T0 = 0, B = 0, D[2] = {}, atbA = 0, atbB = 0;
  size_t probe = 0;  // zpad | Pz (m+1 vectors) | PPz (m vectors) | residuals | gate | counter
  size_t drift_z = 0;  // probe vector of the periodic drift check (n_pad doubles)
  // The rest of the workspace, to its end, is working storage that nothing
  // outlives: creation's and re-anchoring's double matrices (squaring, the
  // sums' and the general form's), an update's partials (lv_view::level_mem) or
  // a batch's slabs and partials (lv_view::plan_batch).  Its smallest size
  // holds the first two side by side, with 256-row tiles, and the slabs of five
  // updates in flight; whatever else a batch or a finer cut asks for has to find
  // room in it.
  size_t work = 0;
  size_t scratch[2] = {}, sscratch[2] = {}, gT[2] = {}, gTmp = 0, gB = 0;
  size_t total = 0;
};

// wide: a plain float view (FP32 or BF16 shadows, no sums, no general form),
// whose top factors may be kMaxWidth wide; other views stop at
// kMaxLevelRank (their level passes take ranks up to kMaxLevelRank / 2).
inline lv_status check_shape(int64_t n, int k, int r_max, lv_mode mode, bool wide = false) {
  if (mode != LV_FP64 && mode != LV_FP32 && mode != LV_FP32_BF16SHADOW)
    return fail(LV_EINVAL, "unknown mode %d", (int)mode);
  if (n < 1 || n > kMaxOrder) return fail(LV_EINVAL, "n = %lld outside [1, %lld]", (long long)n, (long long)kMaxOrder);
  if (!is_pow2(k) || k > kMaxK) return fail(LV_EINVAL, "k = %d is not a power of two in [1, %d]", k, kMaxK);
  if (r_max < 1) return fail(LV_EINVAL, "r_max = %d < 1", r_max);
  const int64_t width = (int64_t)k * next_pow2(r_max);
  const int cap = wide && mode != LV_FP64 ? kMaxWidth : kMaxLevelRank;
  if (width > cap)
    return fail(LV_EINVAL, "k * r_max (rounded up to a power of two) = %lld exceeds %d", (long long)width, cap);
  return LV_OK;
}

constexpr int kMaxGeneralCols = 64;      // p with hybrid deltas (padded to a power of two)
constexpr int kMaxGeneralColsF = 4096;  // p with factored deltas (padded to a multiple of 128)
constexpr int kMaxGeneralWidthF = 128;  // k * r_pad with factored deltas
constexpr int kAtbRows = 64;          // rows per FP64 partial of V^T T and W^T B

// ext_powers: the stored powers live outside the workspace (the caller's
// buffers); the layout then holds only the factor slabs, from offset 0, and
// the working storage of an update.
inline Layout make_layout(int64_t n, int k, int r_max, lv_mode mode, int flags = 0, int p = 0,
                          bool factored = false, int kT = 0, bool ext_powers = false) {
  lv::Layout L;
  L.general = p > 0;
  L.gfac = L.general && factored;
  L.kT = kT > 0 ? kT : k;
  L.nsk = L.gfac ? L.kT / k - 1 : 0;
  L.sums = (flags & LV_WITH_SUMS) != 0 || L.general;
  L.elem = mode == LV_FP64 ? 8 : 4;
  L.n_pad = round_up(n, kPadOrder);
  L.ldp = L.n_pad;
  L.m = ilog2(k);
  L.r_pad = (int)next_pow2(r_max);
  L.W = k * L.r_pad;
  L.nct = (int)(L.n_pad / tile_cols_bytes(L.elem));
  const size_t np = L.n_pad, e = L.elem, ng = gram_tiles(L.n_pad), nrt = np / kMinTileRows;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t at = off; off = align_up(off + bytes); return at; };
  const size_t mat = np * L.ldp * e;
  if (!ext_powers)
    for (int j = 0; j <= L.m; ++j) L.P[j] = take(mat);
  L.slabU = take(np * L.W * e);
  L.slabV = take(np * L.W * e);
  L.slot_stride = off - L.slabU;
  // partials of every level with the smallest tiles, side by side
  auto take_levels = [&]() {
    for (int j = 0; j < L.m; ++j) {
      const size_t R = (size_t)L.r_pad << j;
      take(L.nct * np * R * e);
      take(nrt * np * R * e);
      take(ng * R * R * sizeof(double));
    }
  };
  if (ext_powers) {
    // (what linview.h states for a shape: it decides which the entry point takes)
    L.work = off;
    take_levels();
    L.total = off;
    return L;
  }
  L.piped = !L.sums && L.m >= 2;
  L.zfac = take(np * L.r_pad * e);
  if (mode == LV_FP32_BF16SHADOW) {
    for (int j = 0; j < L.m; ++j) L.shadow[j] = take(np * L.ldp * 2);
    // where the squaring scratch has room for the transposed factors of as many
    // updates as a batch holds at most
    const int chain = chain_updates(L.r_pad), five = L.m + 1 < 5 ? L.m + 1 : 5;
    const int64_t slots = !L.piped ? 1 : chain > 1 && five < kPipeChunks * chain ? kPipeChunks * chain : five;
    L.wide16 = L.m > 0 && (L.r_pad << (L.m - 1)) >= kWide16Rank && slots * 4 * L.W <= 16 * L.n_pad;
  }
  if (L.sums) {
    for (int j = 0; j <= L.m; ++j) L.S[j] = take(mat);
    L.slabQ = take(np * L.W * e);
    L.slabW = take(np * L.W * e);
  }
  size_t wmax = L.r_pad, gmat = 0, gdbl = 0;
  if (L.general) {
    L.p = p;
    L.pp = L.gfac ? (int)round_up(p, 128) : (int)next_pow2(p);
    gmat = np * L.pp * e;
    gdbl = np * L.pp * sizeof(double);
    for (int j = 0; j <= L.m; ++j) L.T[j] = take(gmat);
    L.T0 = take(gmat);
    L.B = take(gmat);
    size_t rmax = (size_t)(L.m > 0 ? L.r_pad << (L.m - 1) : L.r_pad);
    if (L.gfac) {
      L.wy[0] = L.WY[0] = L.r_pad;
      for (int j = 1; j <= L.m; ++j) {
        L.wy[j] = 2 * (L.r_pad << (j - 1)) + L.wy[j - 1];
        L.WY[j] = (int)next_pow2(L.wy[j]);
        if (j < L.m && (size_t)L.WY[j] > wmax) wmax = L.WY[j];
      }
      for (int j = 1; j <= L.m; ++j) L.Y[j] = take(np * L.WY[j] * e);
      for (int j = 0; j <= L.m; ++j) L.Zt[j] = take((size_t)L.WY[j] * L.pp * e);
      if (L.nsk > 0) {
        rmax = (size_t)(L.r_pad << L.m);
        for (int q = 0; q < L.nsk; ++q)
          if ((size_t)L.WYsk(q) > wmax) wmax = L.WYsk(q);   // widths of the P_s passes
        const int wtop = L.WYsk(L.nsk);
        L.tstride = align_up(gmat);
        L.ystride = align_up(np * wtop * e);
        L.zstride = align_up((size_t)wtop * L.pp * e);
        L.Tsk = take(L.nsk * L.tstride);
        L.Ysk = take(L.nsk * L.ystride);
        L.Ztsk = take(L.nsk * L.zstride);
      }
      L.atbG = take(np / kAtbRows * rmax * wmax * sizeof(double));
    } else {
      wmax = L.pp;
      L.D[0] = take(gmat);
      L.D[1] = take(gmat);
    }
    L.atbA = take(np / kAtbRows * rmax * L.pp * sizeof(double));
    L.atbB = take(np / kAtbRows * rmax * L.pp * sizeof(double));
  }
  L.probe = take((size_t)(2 * L.m + 2) * np * sizeof(double) + kMaxLevel * sizeof(double) + 256);
  L.drift_z = take(np * sizeof(double));

  L.work = off;
  const size_t dmat = np * np * sizeof(double);
  if (mode != LV_FP64 && (L.m > 0 || L.general)) {
    for (size_t& at : L.scratch) at = take(dmat);
    if (L.sums)
      for (size_t& at : L.sscratch) at = take(dmat);
  }
  if (L.general) {
    for (size_t& at : L.gT) at = take(gdbl);
    L.gTmp = take(gdbl);
    L.gB = take(gdbl);
    take(L.nct * np * wmax * e);
    take(nrt * np * wmax * e);
  }
  take_levels();
  if (L.sums) take_levels();
  if (L.piped) take((size_t)(L.m + 1 < 5 ? L.m : 4) * L.slot_stride);
  L.total = off;
  return L;
}

template <typename T> T* as(char* p) { return reinterpret_cast<T*>(p); }

// Working storage of one level of an update (or of nver successive updates that
// share the level's passes, vs apart): partials of X, Y and the Gram; of the sums'
// products; of the general form's X; transposed bfloat16 factors of the update's
// slab; operand forms of the shadowed shared passes.
struct LevelMem {
  char *x = nullptr, *y = nullptr, *g = nullptr;
  char *xs = nullptr, *ys = nullptr, *gs = nullptr;
  char* xt = nullptr;
  uint16_t *ut = nullptr, *vt = nullptr;
  char *f16 = nullptr, *f32 = nullptr;
  Strides vs;
};

// Working storage of a pipelined batch: D chunks of C updates in flight, each
// update with a slab pair (and its transposed factors); per level the partials
// of the `most` updates that share its passes.  C = 0: no room for two updates.
struct BatchPlan {
  int C = 0, D = 0;
  size_t bytes = 0;
  char *slabs = nullptr, *fac = nullptr;
  int most[kMaxLevel] = {};
  LevelMem lev[kMaxLevel];
};

// The periodic drift check of a view after an update (no-op unless the
// view's update count is a multiple of its interval); stream-ordered on s.
lv_status periodic_drift(::lv_view* v, hipStream_t s);

inline lv_status hip_check(hipError_t e, const char* what) {
  if (e == hipSuccess) return LV_OK;
  return fail(LV_EDEVICE, "%s: %s", what, hipGetErrorString(e));
}

}  // namespace lv

struct lv_view {
  int64_t n;
  int k;
  int r_max;
  lv_mode mode;
  lv::Layout L;
  char* base;
  size_t ws_bytes;
  int64_t updates;
  int64_t reanchors;
  // periodic drift check: after every drift_every-th update (0: never) with
  // bound drift_tau and the probe vector at L.drift_z; checks enqueued so far
  int64_t drift_every = 0;
  double drift_tau = 0.0;
  int64_t drift_checks = 0;
  // Rows per tile of the level pass of each level below the top (set by the
  // batch autotuner or lv_view_set_tile_rows; kTileRows: the cut of slice_rows;
  // every path uses the same value, which fixes the reduction order of the
  // partial sums).
  int tile_rows[lv::kMaxLevel];
  // rows per slice and slices of the level's pass of rank R.  The default's cut
  // is the one of slice_rows as far as the workspace holds its partials, fixed
  // when the view is created (set_cuts); float views always hold it.
  int cuts[16] = {};
  bool on_cores(int R) const { return shadowed() || lv::skinny_on_mfma(R, L.elem); }
  int rows(int j, int R) const {
    const int t = tile_rows[j];
    return t == lv::kTileRows ? cuts[lv::ilog2(R)] : t == LV_TILE_ROWS_512 ? 512 : t;
  }
  int nrt(int j, int R) const { const int r = rows(j, R); return (int)((L.n_pad + r - 1) / r); }
  // rows per slice of a pass that forms X alone (no partials depend on them)
  int xrows(int R) const { return lv::slice_rows(L.n_pad, L.elem, R, lv::skinny_on_mfma(R, L.elem)); }

  // Kernel timing (diagnostics): event pairs per launch kind, resolved by
  // lv_view_timing.
  bool timing = false;
  struct Pair { hipEvent_t a, b; int kind; };
  std::vector<Pair> pending;
  std::vector<hipEvent_t> pool;

  // Pipelined update_batch (plain views, L.piped): stage streams (stage 0 runs
  // on the caller's stream; created on first use), the events that order the
  // stages (pready: level j's factors of the update in a slot are assembled;
  // pfree: the slot's update is through its top level; of the first pipe_events
  // slots) and fork / join events.  pipeline = false keeps every batch
  // sequential.  lent: working storage for batches beyond the workspace's.
  bool pipeline = true;
  int pipe_nstages = 0, pipe_events = 0;
  char* lent = nullptr;
  size_t lent_bytes = 0;
  hipStream_t pstream[lv::kPipeStreams] = {};
  hipEvent_t pready[lv::kMaxLevel][lv::kMaxPipeSlots] = {};
  int pgroup[lv::kMaxLevel][lv::kMaxPipeSlots] = {};   // last slot of the group that holds a slot's update
  hipEvent_t pfree[lv::kMaxPipeSlots] = {};
  hipEvent_t pfork = nullptr;
  hipEvent_t pjoin[lv::kPipeStreams] = {};

  // stored powers held outside the workspace (set by the allocation-free
  // update entry point; null for views created on a workspace)
  char* pext[lv::kMaxLevel + 1] = {};
  template <typename T> T* P(int j) const { return reinterpret_cast<T*>(pext[j] ? pext[j] : base + L.P[j]); }
  template <typename T> T* slabU() const { return reinterpret_cast<T*>(base + L.slabU); }
  template <typename T> T* slabV() const { return reinterpret_cast<T*>(base + L.slabV); }
  template <typename T> T* S(int j) const { return reinterpret_cast<T*>(base + L.S[j]); }
  template <typename T> T* slabQ() const { return reinterpret_cast<T*>(base + L.slabQ); }
  template <typename T> T* slabW() const { return reinterpret_cast<T*>(base + L.slabW); }
  double* sscratch(int i) const { return reinterpret_cast<double*>(base + L.sscratch[i]); }
  template <typename T> T* Tg(int j) const { return reinterpret_cast<T*>(base + L.T[j]); }
  template <typename T> T* T0() const { return reinterpret_cast<T*>(base + L.T0); }
  template <typename T> T* Bg() const { return reinterpret_cast<T*>(base + L.B); }
  template <typename T> T* D(int i) const { return reinterpret_cast<T*>(base + L.D[i]); }
  double* atbA() const { return reinterpret_cast<double*>(base + L.atbA); }
  double* atbG() const { return reinterpret_cast<double*>(base + L.atbG); }
  template <typename T> T* Yf(int j) const { return reinterpret_cast<T*>(base + L.Y[j]); }
  template <typename T> T* Ztf(int j) const { return reinterpret_cast<T*>(base + L.Zt[j]); }
  // skip-model T_{(q+1)s}, its Y and Z^T slabs (q = 1 .. nsk)
  template <typename T> T* Tskp(int q) const { return reinterpret_cast<T*>(base + L.Tsk + (size_t)(q - 1) * L.tstride); }
  template <typename T> T* Yskp(int q) const { return reinterpret_cast<T*>(base + L.Ysk + (size_t)(q - 1) * L.ystride); }
  template <typename T> T* Ztskp(int q) const { return reinterpret_cast<T*>(base + L.Ztsk + (size_t)(q - 1) * L.zstride); }
  double* atbB() const { return reinterpret_cast<double*>(base + L.atbB); }
  double* gT(int i) const { return reinterpret_cast<double*>(base + L.gT[i]); }
  double* gTmp() const { return reinterpret_cast<double*>(base + L.gTmp); }
  double* gB() const { return reinterpret_cast<double*>(base + L.gB); }
  uint16_t* shadow(int j) const { return reinterpret_cast<uint16_t*>(base + L.shadow[j]); }
  bool shadowed() const { return mode == LV_FP32_BF16SHADOW; }
  // Transposed bfloat16 factors of the levels from rank kWide16Rank (shadow
  // mode): row c holds column c of a slab.
  bool wide16(int R) const { return L.wide16 && R >= lv::kWide16Rank; }
  size_t fac_bytes() const { return L.wide16 ? lv::align_up((size_t)L.n_pad * L.W * 4) : 0; }
  // The columns of a level's factors that the level below has not converted:
  // all of them at the first such level, else the block that its tail added.
  lv::Fac16Desc fac16(int R, bool first, const float* sU, uint16_t* ut) const {
    const int cols = first ? R : R / 2, cu = R - cols, cv = L.W - R;
    // (a float slab of n_pad x W values fills whole 256-byte units: V's follows U's directly)
    return {sU + cu, ut + (int64_t)cu * L.n_pad, L.W, (int)L.n_pad, cols, cv - cu, 0};
  }

  // Places the partials of `most` updates' level of rank R with ns slices from
  // offset off on (of base, which may be null for the size alone); returns the
  // end.
  size_t place(char* at, size_t off, int R, int64_t ns, int most, lv::LevelMem* m) const {
    const size_t n = L.n_pad, e = L.elem, r = R;
    const bool in_pass = lv::fused_vector_level(R, L.elem, shadowed()) && R <= lv::kMaxFusedRank;
    const size_t ng = in_pass ? ns : lv::gram_count(n, R);
    const size_t ny = wide16(R) && lv::wide_splits(n) > ns ? lv::wide_splits(n) : ns;
    auto take = [&](size_t bytes) { char* q = at + off; off = lv::align_up(off + bytes); return q; };
    m->vs = {(int64_t)(L.slot_stride / e), (int64_t)(L.nct * n * r), (int64_t)(ny * n * r), (int64_t)(ng * r * r)};
    m->x = take(most * L.nct * n * r * e);
    m->y = take(most * ny * n * r * e);
    m->g = take(most * ng * r * r * sizeof(double));
    if (shadowed() && most > 1) {
      m->f16 = take(most * lv::chain_f16_bytes(n, R));
      m->f32 = take(most * lv::chain_f32_bytes(n, R));
    }
    if (L.sums) {
      m->xs = take(L.nct * n * r * e);
      m->ys = take(ns * n * r * e);
      m->gs = take(lv::gram_tiles(n) * r * r * sizeof(double));
    }
    // (factored: Y_j, j > 0, has up to 2 R columns; level 0 takes the powers' X)
    if (L.general) m->xt = take(L.nct * n * (!L.gfac ? L.pp : L.m > 1 ? 2 * r : 0) * e);
    return off;
  }
  size_t room() const { return ws_bytes - L.work; }
  // A level's working storage for one update (every level uses the same, one
  // after the other), behind the update's transposed factors.
  lv::LevelMem level_mem(int R, int64_t ns) const {
    lv::LevelMem m;
    place(base + L.work, fac_bytes(), R, ns, 1, &m);
    m.ut = reinterpret_cast<uint16_t*>(base + L.work);
    m.vt = m.ut + (int64_t)L.W * L.n_pad;
    return m;
  }
  // Fixes the default's cuts; with a null base, returns the workspace that
  // holds all of slice_rows'.
  size_t set_cuts() {
    size_t full = L.total;
    lv::LevelMem m;
    for (int R = 1; L.m > 0 && R <= L.r_pad << (L.m - 1); R *= 2) {
      const int want = lv::slice_rows(L.n_pad, L.elem, R, on_cores(R));
      auto bytes = [&](int64_t ns) { return place(nullptr, fac_bytes(), R, ns, 1, &m); };
      cuts[lv::ilog2(R)] = lv::fitted_rows(L.n_pad, want, on_cores(R), room(), bytes);
      const size_t all = L.work + bytes((L.n_pad + want - 1) / want);
      full = all > full ? all : full;
    }
    return full;
  }

  // Updates of padded rank r_pad that a chunk of a batch takes at most.
  int chunk(int r_pad) const {
    if (!shadowed()) return lv::chain_updates(r_pad);
    return r_pad < lv::kChain16Rank ? lv::kChain16Updates : 2;
  }
  // Places a batch's working storage for D chunks of C updates of padded rank
  // r_pad; least_rows > 0: with slices of that many rows where they are more.
  lv::BatchPlan plan_of(char* at, int r_pad, int C, int D, int least_rows = 0) const {
    lv::BatchPlan b;
    b.C = C;
    b.D = D;
    size_t off = 0;
    b.slabs = at;
    off += (size_t)C * D * L.slot_stride;
    b.fac = at + off;
    if (wide16(r_pad << (L.m - 1))) off += (size_t)C * D * fac_bytes();
    for (int j = 0; j < L.m; ++j) {
      const int R = r_pad << j;
      int64_t ns = nrt(j, R);
      if (least_rows > 0 && ns < L.n_pad / least_rows) ns = L.n_pad / least_rows;
      const int shared = shadowed() ? (R <= lv::kChain16Rank ? lv::chain16_updates(R) : 1)
                         : lv::fused_vector_level(R, L.elem, false) ? lv::chain_updates(R) : 1;
      b.most[j] = shared < C ? shared : C;
      off = place(at, off, R, ns, b.most[j], &b.lev[j]);
    }
    b.bytes = off;
    return b;
  }
  // The largest chunks, then the most of them in flight, that fit: three
  // chunks, or an update for each of up to five stages where updates share
  // nothing (more only widen the working set: rank-4 shadow batches n = 8192
  // 23.46 ms with 5 updates in flight, 23.74 ms with 12).
  lv::BatchPlan plan_batch(char* at, size_t bytes, int r_pad) const {
    for (int C = chunk(r_pad); C >= 1; C /= 2)
      for (int D = C > 1 ? lv::kPipeChunks : L.m + 1 < 5 ? L.m + 1 : 5; D >= 2; --D) {
        const lv::BatchPlan b = plan_of(at, r_pad, C, D);
        if (b.bytes <= bytes) return b;
      }
    return {};
  }
  lv::BatchPlan plan_batch(int r_pad) const {
    const lv::BatchPlan own = plan_batch(base + L.work, room(), r_pad);
    if (lent == nullptr) return own;
    const lv::BatchPlan b = plan_batch(lent, lent_bytes, r_pad);
    return b.C > own.C || (b.C == own.C && b.D > own.D) ? b : own;
  }
  // Working storage that gives every batch its full plan; 0 if the workspace does.
  size_t lend_bytes() const {
    size_t most = 0;
    bool fits = true;
    for (int r = 1; L.piped && r <= L.r_pad; r *= 2) {
      const int C = chunk(r), D = C > 1 ? lv::kPipeChunks : L.m + 1 < 5 ? L.m + 1 : 5;
      const size_t need = plan_of(nullptr, r, C, D, lv::kMinTileRows).bytes;
      fits = fits && need <= room();
      most = need > most ? need : most;
    }
    return fits ? 0 : most;
  }
  double* scratch(int i) const { return reinterpret_cast<double*>(base + L.scratch[i]); }
  double* zpad() const { return reinterpret_cast<double*>(base + L.probe); }
  double* drift_z() const { return reinterpret_cast<double*>(base + L.drift_z); }
  double* Pz(int j) const { return zpad() + (size_t)(1 + j) * L.n_pad; }
  double* PPz(int j) const { return zpad() + (size_t)(L.m + 2 + j) * L.n_pad; }
  double* residuals() const { return zpad() + (size_t)(2 * L.m + 2) * L.n_pad; }
  int* gate() const { return reinterpret_cast<int*>(residuals() + lv::kMaxLevel); }
  unsigned long long* drift_counter() const {
    return reinterpret_cast<unsigned long long*>(reinterpret_cast<char*>(residuals() + lv::kMaxLevel) + 64);
  }
};
