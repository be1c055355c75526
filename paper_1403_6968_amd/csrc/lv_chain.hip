// Matrix-power views under the linear, skip-s and exponential iterative
// models (Sec. 3.2, Table 1), maintained by IncrLin / IncrSkip-s / IncrExp
// (App. A).  Every stored P_c is a product P_a P_b of two earlier stored
// matrices (linear: a = 1, b = c - 1; skip-s: a = s, b = c - s beyond s;
// exponential: a = b = c/2), and its delta is factored as
//     U_c = [U_a, P_a U_b + U_a (V_a^T U_b)],   V_c = [P_b^T V_a, V_b]
// from the OLD matrices; and every stored matrix takes P_c += U_c V_c^T.
// Each stored matrix has its own factor slabs (width c * r_pad padded to a
// power of two): in the linear and skip models U_b is transformed, not
// extended, so the prefix layout of the exponential view does not apply.
#include "linview.h"
#include "lv_internal.h"
#include "lv_view_impl.h"

#include <new>
#include <utility>
#include <vector>

using namespace lv;

namespace lv {
namespace {

constexpr int kMaxChainWidth = 128;   // k * r_pad (the read-only passes take up to 128 columns)
constexpr int kMaxChainStored = 128;

// Lanes of eight per (row, column j < wa): the lane group sums the partials of
// X and Y (lane l the partials l, l + 8, ...; a butterfly adds the lane sums in
// double) and writes column wb + j of U_c and column j of V_c; the group of
// j = 0 also copies the row's U_b and V_b and writes the zero columns.
constexpr int kKrylovLanes = 8;
constexpr int kKrylovGramCap = 64;    // Gram partials are summed here up to 8 columns
template <typename T>
__global__ void __launch_bounds__(256)
k_krylov_tail(int wa, const T* __restrict__ partX, int nct, const T* __restrict__ partY, int nrt,
              const double* __restrict__ partG, int ng, const T* __restrict__ Ua, int Wa, const T* __restrict__ Ub,
              const T* __restrict__ Vb, int Wb, int wb, T* Uc, T* Vc, int Wc, int64_t n_pad) {
  constexpr int TL = kKrylovLanes;
  __shared__ double Gs[kKrylovGramCap];
  const int tid = threadIdx.x;
  const double* G = partG;
  if (ng > 1) {
    // wa^2 <= 64 entries, 256 / wa^2 threads each (shuffled together when
    // they share a wave)
    const int cnt = wa * wa, per = 256 / cnt < 32 ? 256 / cnt : 32;
    const int e = tid / per, l = tid % per;
    double g = 0.0;
    if (e < cnt)
      for (int t = l; t < ng; t += per) g += partG[(int64_t)t * cnt + e];
    for (int off = per / 2; off > 0; off >>= 1) g += __shfl_xor(g, off, per);
    if (e < cnt && l == 0) Gs[e] = g;
    __syncthreads();
    G = Gs;
  }
  const int64_t idx = (int64_t)blockIdx.x * (256 / TL) + tid / TL;
  const int sl = tid % TL;
  if (idx >= n_pad * wa) return;   // whole lane groups leave together
  const int64_t row = idx / wa;
  const int j = (int)(idx % wa);
  const int64_t stride = n_pad * wa;
  double x = 0.0, y = 0.0;
#pragma unroll 4
  for (int t = sl; t < nct; t += TL) x += (double)partX[t * stride + idx];
  if (Vc != nullptr) {
#pragma unroll 4
    for (int t = sl; t < nrt; t += TL) y += (double)partY[t * stride + idx];
  }
  for (int d = sl; d < wa; d += TL) x = fma((double)Ua[row * Wa + d], G[d * wa + j], x);
#pragma unroll
  for (int off = TL / 2; off > 0; off >>= 1) {
    x += __shfl_xor(x, off, TL);
    y += __shfl_xor(y, off, TL);
  }
  if (sl == 0) {
    Uc[row * Wc + wb + j] = (T)x;
    if (Vc != nullptr) Vc[row * Wc + j] = (T)y;
  }
  if (Ub != nullptr && j == 0) {
    for (int c = sl; c < wb; c += TL) {
      Uc[row * Wc + c] = Ub[row * Wb + c];
      if (Vc != nullptr) Vc[row * Wc + wa + c] = Vb[row * Wb + c];
    }
    for (int c = wa + wb + sl; Vc != nullptr && c < Wc; c += TL) {
      Uc[row * Wc + c] = T(0);
      Vc[row * Wc + c] = T(0);
    }
  }
}

}  // namespace

template <typename T>
hipError_t launch_krylov_tail(int wa, const T* partX, int nct, const T* partY, int nrt, const double* partG, int ng,
                              const T* Ua, int Wa, const T* Ub, const T* Vb, int Wb, int wb, T* Uc, T* Vc, int Wc,
                              int64_t n_pad, hipStream_t s) {
  if (ng > 1 && wa * wa > kKrylovGramCap) return hipErrorInvalidValue;
  const unsigned blocks = (unsigned)((n_pad * wa * kKrylovLanes + 255) / 256);
  hipLaunchKernelGGL((k_krylov_tail<T>), dim3(blocks), dim3(256), 0, s, wa, partX, nct, partY, nrt, partG, ng, Ua, Wa,
                     Ub, Vb, Wb, wb, Uc, Vc, Wc, n_pad);
  return hipGetLastError();
}
#define LV_INST(T)                                                                                                 \
  template hipError_t launch_krylov_tail<T>(int, const T*, int, const T*, int, const double*, int, const T*, int,  \
                                            const T*, const T*, int, int, T*, T*, int, int64_t, hipStream_t);
LV_INST(float)
LV_INST(double)
#undef LV_INST

}  // namespace lv

struct lv_chain {
  int64_t n, n_pad;
  int k, s, model, r_max, r_pad, elem, nct;
  lv_mode mode;
  std::vector<int> pw;       // stored powers, pw[0] = 1
  std::vector<int> Wd;       // padded slab width of each stored matrix
  // products in evaluation order (indices into pw); of a step's passes, the
  // rows per slice, the slices and the places of the partials
  struct Step { int c, a, b, rows = 0, nrt = 0; size_t x = 0, xd = 0, y = 0, g = 0; };
  std::vector<Step> steps;
  std::vector<int> left_last;   // last step that reads a stored matrix as P_a (-1: none)
  std::vector<char> done;       // matrices that an update's steps have updated already
  std::vector<size_t> P, sU, sV;
  size_t d64[3] = {};
  size_t total = 0;
  char* base = nullptr;
  int64_t updates = 0;

  template <typename T> T* Pm(int i) const { return reinterpret_cast<T*>(base + P[i]); }
  template <typename T> T* U(int i) const { return reinterpret_cast<T*>(base + sU[i]); }
  template <typename T> T* V(int i) const { return reinterpret_cast<T*>(base + sV[i]); }
  template <typename T> T* pX(const Step& q) const { return reinterpret_cast<T*>(base + q.x); }
  template <typename T> T* pXd(const Step& q) const { return reinterpret_cast<T*>(base + q.xd); }   // not wanted
  template <typename T> T* pY(const Step& q) const { return reinterpret_cast<T*>(base + q.y); }
  double* pG(const Step& q) const { return reinterpret_cast<double*>(base + q.g); }
  double* d(int i) const { return reinterpret_cast<double*>(base + d64[i]); }
};

namespace {

// Stored powers and products of a model (Table 1, matrix-powers column).
lv_status plan_chain(lv_chain& c) {
  std::vector<std::pair<int, int>> prods;   // (c, a) with b the previous product
  if (c.model == LV_MODEL_LIN) {
    for (int i = 2; i <= c.k; ++i) prods.push_back({i, 1});
  } else if (c.model == LV_MODEL_EXP) {
    for (int i = 2; i <= c.k; i *= 2) prods.push_back({i, i / 2});
  } else {
    for (int i = 2; i <= c.s; i *= 2) prods.push_back({i, i / 2});
    for (int i = 2 * c.s; i <= c.k; i += c.s) prods.push_back({i, c.s});
  }
  c.pw.assign(1, 1);
  for (auto& p : prods) c.pw.push_back(p.first);
  if ((int)c.pw.size() > kMaxChainStored) return fail(LV_EINVAL, "%d stored matrices exceed %d", (int)c.pw.size(), kMaxChainStored);
  auto index = [&](int power) {
    for (size_t i = 0; i < c.pw.size(); ++i) if (c.pw[i] == power) return (int)i;
    return -1;
  };
  c.steps.clear();
  for (size_t q = 0; q < prods.size(); ++q) {
    const int ci = (int)q + 1, ai = index(prods[q].second), bi = index(prods[q].first - prods[q].second);
    if (ai < 0 || bi != ci - 1) return fail(LV_EINVAL, "internal: product %d has no stored operands", prods[q].first);
    c.steps.push_back({ci, ai, bi});
  }
  c.left_last.assign(c.pw.size(), -1);
  for (size_t q = 0; q < c.steps.size(); ++q) c.left_last[c.steps[q].a] = (int)q;
  return LV_OK;
}

lv_status check_chain(int64_t n, int k, int r_max, lv_mode mode, int model, int s) {
  if (mode != LV_FP64 && mode != LV_FP32) return fail(LV_EINVAL, "chain views take LV_FP64 or LV_FP32, got %d", (int)mode);
  if (n < 1 || n > kMaxOrder) return fail(LV_EINVAL, "n = %lld outside [1, %lld]", (long long)n, (long long)kMaxOrder);
  if (r_max < 1) return fail(LV_EINVAL, "r_max = %d < 1", r_max);
  if (k < 1) return fail(LV_EINVAL, "k = %d < 1", k);
  if (model == LV_MODEL_EXP) {
    if (!is_pow2(k)) return fail(LV_EINVAL, "the exponential model needs k a power of two, got %d", k);
  } else if (model == LV_MODEL_SKIP) {
    if (!is_pow2(s) || s > k || k % s != 0)
      return fail(LV_EINVAL, "the skip model needs s a power of two dividing k, got s = %d, k = %d", s, k);
  } else if (model != LV_MODEL_LIN) {
    return fail(LV_EINVAL, "unknown model %d", model);
  }
  if ((int64_t)k * next_pow2(r_max) > kMaxChainWidth)
    return fail(LV_EINVAL, "k * r_max (rounded up to a power of two) exceeds %d", kMaxChainWidth);
  return LV_OK;
}

// The layout in a workspace of ws_bytes, or of the smallest size; *full (may be
// null) receives the size that holds every slice.
lv_status layout_chain(lv_chain& c, int64_t n, int k, int r_max, lv_mode mode, int model, int s, size_t ws_bytes = 0,
                       size_t* full = nullptr) {
  c.n = n; c.k = k; c.s = model == LV_MODEL_SKIP ? s : 0; c.model = model; c.r_max = r_max; c.mode = mode;
  c.r_pad = (int)next_pow2(r_max);
  c.elem = mode == LV_FP64 ? 8 : 4;
  c.n_pad = round_up(n, kPadOrder);
  c.nct = (int)(c.n_pad / tile_cols_bytes(c.elem));
  lv_status st = plan_chain(c);
  if (st != LV_OK) return st;
  const int ns = (int)c.pw.size();
  c.Wd.resize(ns);
  int maxW = 1;
  for (int i = 0; i < ns; ++i) { c.Wd[i] = (int)next_pow2((int64_t)c.pw[i] * c.r_pad); maxW = c.Wd[i] > maxW ? c.Wd[i] : maxW; }
  size_t maxG = 1;
  for (auto& q : c.steps) { const size_t g = (size_t)c.Wd[q.a] * c.Wd[q.b]; maxG = g > maxG ? g : maxG; }
  size_t off = 0;
  const size_t mat = (size_t)c.n_pad * c.n_pad * c.elem;
  c.P.resize(ns); c.sU.resize(ns); c.sV.resize(ns);
  for (int i = 0; i < ns; ++i) { c.P[i] = off; off = align_up(off + mat); }
  for (int i = 0; i < ns; ++i) {
    const size_t slab = (size_t)c.n_pad * c.Wd[i] * c.elem;
    c.sU[i] = off; off = align_up(off + slab);
    c.sV[i] = off; off = align_up(off + slab);
  }
  // Last the region that an update's partials and creation's double matrices
  // share, sized for both and for whole-width passes over kTileRows rows.
  const size_t work = off, np = c.n_pad, e = c.elem;
  for (size_t cols : {(size_t)c.nct * maxW, (size_t)c.nct * maxW, (np + kTileRows - 1) / kTileRows * maxW})
    off = align_up(off + np * cols * e);
  off = align_up(off + np / kAtbRows * maxG * sizeof(double));
  if (mode == LV_FP32 && ns > 1) {
    for (int i = 0; i < 3; ++i) {
      c.d64[i] = work + i * align_up(np * np * sizeof(double));
      off = align_up(off + np * np * sizeof(double));
    }
  }
  c.total = off;
  const size_t room = (ws_bytes > off ? ws_bytes : off) - work;
  size_t all = off;
  for (auto& q : c.steps) {
    const size_t w = (size_t)c.pw[q.a] * c.r_pad;
    const bool cores = skinny_on_mfma((int)w, c.elem);
    auto place = [&](int64_t nrt) {
      q.nrt = (int)nrt;
      q.x = work;
      q.xd = align_up(q.x + c.nct * np * w * e);
      q.y = align_up(q.xd + c.nct * np * w * e);
      q.g = align_up(q.y + nrt * np * w * e);
      return q.g + (w <= (size_t)kMaxKrylovCols ? nrt : np / kAtbRows) * w * w * sizeof(double) - work;
    };
    const int want = slice_rows(c.n_pad, c.elem, (int)w, cores);
    const size_t bytes = work + place((c.n_pad + want - 1) / want);
    all = bytes > all ? bytes : all;
    q.rows = fitted_rows(c.n_pad, want, cores, room, place);
    place((c.n_pad + q.rows - 1) / q.rows);
  }
  if (full) *full = all;
  return LV_OK;
}

// Creation: the model's products in double precision (float views keep the
// running product and the fixed left operand in double and round each
// stored matrix once).
template <typename T>
lv_status build_chain_model(lv_chain* c, hipStream_t s) {
  const int64_t np = c->n_pad;
  if constexpr (sizeof(T) == 8) {
    for (auto& q : c->steps) {
      lv_status st = hip_check(launch_gemm<double>(c->Pm<double>(q.a), np, c->Pm<double>(q.b), np, c->Pm<double>(q.c),
                                                   np, np, s), "gemm f64");
      if (st != LV_OK) return st;
    }
    return LV_OK;
  } else {
    if (c->steps.empty()) return LV_OK;
    double* prev = c->d(0);
    double* next = c->d(1);
    double* mult = c->d(2);
    const int mult_pw = c->model == LV_MODEL_LIN ? 1 : c->model == LV_MODEL_SKIP ? c->s : -1;
    lv_status st = hip_check(launch_copy_pad<float, double>(c->Pm<float>(0), np, np, prev, np, np, s), "widen A");
    const size_t dbytes = (size_t)np * np * sizeof(double);
    if (st == LV_OK && mult_pw == 1)
      st = hip_check(hipMemcpyAsync(mult, prev, dbytes, hipMemcpyDeviceToDevice, s), "keep A");
    for (auto& q : c->steps) {
      if (st != LV_OK) return st;
      const double* lhs = q.a == q.b ? prev : mult;
      st = hip_check(launch_gemm<double>(lhs, np, prev, np, next, np, np, s), "gemm f64");
      if (st == LV_OK)
        st = hip_check(launch_copy_pad<double, float>(next, np, np, c->Pm<float>(q.c), np, np, s), "round P");
      std::swap(prev, next);
      if (st == LV_OK && c->pw[q.c] == mult_pw && mult_pw != 1)
        st = hip_check(hipMemcpyAsync(mult, prev, dbytes, hipMemcpyDeviceToDevice, s), "keep P_s");
    }
    return st;
  }
}

// One step, the product P_c = P_a P_b, with w = pw[a] r_pad columns of P_a's
// factors: X = P_a M for the last w columns M of U_b (column-tile partials),
// Y = P_b^T V_a (row-slice partials) and the Gram V_a^T M, all from the OLD
// matrices.  Two columns of U_c that apply f(M) = P_a M + U_a (V_a^T M) to
// equal columns are equal, and U_b = [U_a, f(U_a), f(f(U_a)), ...] by induction
// over the steps with this left operand (a = 1 or s, b = a, 2 a, ...), so of
//     U_c = [U_a, f(U_b)] = [U_b, f(M)]
// only f(M) is new: the products take w columns instead of U_b's whole width.
// Up to 8 columns the vector passes run, one read of the matrix when a = b;
// else X and Y in one launch, P_b taking its own update in the pass that
// reads it (*updated) where no later step reads it as P_a.
template <typename T>
lv_status step_products(lv_chain* c, const lv_chain::Step& q, hipStream_t s, int* ng, bool* updated) {
  const int64_t np = c->n_pad;
  const int Wa = c->Wd[q.a], Wb = c->Wd[q.b];
  const int w = c->pw[q.a] * c->r_pad;   // = Wa: the left operands' powers are powers of two
  const T* M = c->U<T>(q.b) + (c->pw[q.b] - c->pw[q.a]) * c->r_pad;
  const T* Va = c->V<T>(q.a);
  *updated = false;
  if (w <= kMaxKrylovCols) {
    *ng = q.nrt;
    if (q.a == q.b)
      return hip_check(launch_fused_xgram<T>(w, c->Pm<T>(q.a), np, np, q.rows, M, Wb, Va, Wa, c->pX<T>(q),
                                             c->pY<T>(q), c->pG(q), s), "P U, P^T V");
    if (Wb <= kMaxFusedRank && c->left_last[q.b] < 0) {
      *updated = true;
      return hip_check(launch_krylov_step<T>(Wb, w, c->Pm<T>(q.a), c->Pm<T>(q.b), np, np, q.rows, q.rows, M,
                                             c->U<T>(q.b), c->V<T>(q.b), Wb, Va, Wa, c->pX<T>(q), c->pY<T>(q), c->pG(q),
                                             s), "P_a U_b, P_b^T V_a, P_b += U_b V_b^T");
    }
    lv_status st = hip_check(launch_fused_xgram<T>(w, c->Pm<T>(q.a), np, np, q.rows, M, Wb, Va, Wa, c->pX<T>(q),
                                                   nullptr, c->pG(q), s), "P_a U_b");
    if (st != LV_OK) return st;
    return hip_check(launch_level_readonly<T>(w, c->Pm<T>(q.b), np, np, q.rows, Va, Va, Wa, c->pXd<T>(q),
                                              c->pY<T>(q), s), "P_b^T V_a");
  }
  // wider: the float matrix cores form only what is asked, the vector pass
  // that forms Y sends X to the discard buffer
  auto pass = [&](const T* P, const T* op1, const T* op2, int W, T* px, T* py, int want) -> hipError_t {
    if (skinny_on_mfma(w, (int)sizeof(T)))
      return launch_skinny_f32(w, reinterpret_cast<const float*>(P), np, np, q.rows,
                               reinterpret_cast<const float*>(op1), reinterpret_cast<const float*>(op2), W,
                               reinterpret_cast<float*>(px), reinterpret_cast<float*>(py), s, want);
    return launch_level_readonly<T>(w, P, np, np, q.rows, op1, op2, W, px, py, s);
  };
  *ng = 1;
  lv_status st = LV_OK;
  if (q.a == q.b) {
    st = hip_check(pass(c->Pm<T>(q.a), M, Va, Wa, c->pX<T>(q), c->pY<T>(q), kWantX | kWantY), "P U, P^T V");
  } else {
    st = hip_check(pass(c->Pm<T>(q.a), M, M, Wb, c->pX<T>(q), nullptr, kWantX), "P_a U_b");
    if (st == LV_OK) st = hip_check(pass(c->Pm<T>(q.b), Va, Va, Wa, c->pXd<T>(q), c->pY<T>(q), kWantY), "P_b^T V_a");
  }
  if (st != LV_OK) return st;
  return hip_check(launch_atb<T>(w, w, Va, Wa, M, Wb, np, c->pG(q), s), "V_a^T U_b");
}

template <typename T>
lv_status chain_update(lv_chain* c, const T* U, const T* V, int r, int64_t ldu, int64_t ldv, hipStream_t s) {
  const int64_t np = c->n_pad;
  lv_status st = hip_check(launch_prep<T>(U, ldu, V, ldv, c->n, r, c->r_pad, c->U<T>(0), c->V<T>(0), c->r_pad, np, s),
                           "prep");
  std::vector<char>& done = c->done;
  done.assign(c->pw.size(), 0);
  for (auto& q : c->steps) {
    if (st != LV_OK) return st;
    const int w = c->pw[q.a] * c->r_pad;
    int ng = 1;
    bool updated = false;
    st = step_products<T>(c, q, s, &ng, &updated);
    if (updated) done[q.b] = 1;
    if (st == LV_OK)
      st = hip_check(launch_krylov_tail<T>(w, c->pX<T>(q), c->nct, c->pY<T>(q), q.nrt, c->pG(q), ng, c->U<T>(q.a),
                                           c->Wd[q.a], c->U<T>(q.b), c->V<T>(q.b), c->Wd[q.b], c->pw[q.b] * c->r_pad,
                                           c->U<T>(q.c), c->V<T>(q.c), c->Wd[q.c], np, s), "chain tail");
  }
  for (size_t i = 0; i < c->pw.size() && st == LV_OK; ++i)
    if (!done[i])
      st = hip_check(launch_level_update<T>(c->Wd[i], c->Pm<T>((int)i), np, np, c->U<T>((int)i), c->V<T>((int)i),
                                            c->Wd[i], s), "P += U V^T");
  return st;
}

}  // namespace

extern "C" {

size_t lv_chain_footprint(int64_t n, int k, int r_max, lv_mode mode, int model, int s) {
  if (check_chain(n, k, r_max, mode, model, s) != LV_OK) return 0;
  lv_chain c;
  if (layout_chain(c, n, k, r_max, mode, model, s) != LV_OK) return 0;
  return c.total;
}

size_t lv_chain_footprint_full(int64_t n, int k, int r_max, lv_mode mode, int model, int s) {
  if (check_chain(n, k, r_max, mode, model, s) != LV_OK) return 0;
  lv_chain c;
  size_t full = 0;
  return layout_chain(c, n, k, r_max, mode, model, s, 0, &full) == LV_OK ? full : 0;
}

lv_status lv_chain_create(const void* A, int64_t n, int64_t lda, int k, int r_max, lv_mode mode, int model, int s,
                          void* workspace, size_t ws_bytes, void* stream, lv_chain** out) {
  g_err[0] = 0;
  if (!out) return fail(LV_EINVAL, "out is NULL");
  *out = nullptr;
  lv_status st = check_chain(n, k, r_max, mode, model, s);
  if (st != LV_OK) return st;
  if (!A || !workspace) return fail(LV_EINVAL, "A or workspace is NULL");
  if (lda < n) return fail(LV_EINVAL, "lda = %lld < n = %lld", (long long)lda, (long long)n);
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
    return fail(LV_ENOMEM, "workspace is not %zu-byte aligned", kAlign);
  lv_chain* c = new (std::nothrow) lv_chain();
  if (!c) return fail(LV_ENOMEM, "host allocation of the chain handle failed");
  st = layout_chain(*c, n, k, r_max, mode, model, s, ws_bytes);
  if (st == LV_OK && ws_bytes < c->total) st = fail(LV_ENOMEM, "workspace has %zu bytes, needs %zu", ws_bytes, c->total);
  if (st != LV_OK) { delete c; return st; }
  c->base = static_cast<char*>(workspace);
  hipStream_t hs = static_cast<hipStream_t>(stream);
  if (mode == LV_FP64) {
    st = hip_check(launch_copy_pad<double, double>(static_cast<const double*>(A), lda, n, c->Pm<double>(0), c->n_pad,
                                                   c->n_pad, hs), "copy A");
    if (st == LV_OK) st = build_chain_model<double>(c, hs);
  } else {
    st = hip_check(launch_copy_pad<float, float>(static_cast<const float*>(A), lda, n, c->Pm<float>(0), c->n_pad,
                                                 c->n_pad, hs), "copy A");
    if (st == LV_OK) st = build_chain_model<float>(c, hs);
  }
  if (st != LV_OK) { delete c; return st; }
  *out = c;
  return LV_OK;
}

lv_status lv_chain_update(lv_chain* c, const void* U, const void* V, int64_t r, int64_t ldu, int64_t ldv,
                          void* stream) {
  g_err[0] = 0;
  if (!c) return fail(LV_EINVAL, "chain is NULL");
  if (!U || !V) return fail(LV_EINVAL, "U or V is NULL");
  if (r < 1 || r > c->r_max) return fail(LV_EINVAL, "rank r = %lld outside [1, %d]", (long long)r, c->r_max);
  if (ldu < r || ldv < r) return fail(LV_EINVAL, "ldu/ldv smaller than r");
  hipStream_t s = static_cast<hipStream_t>(stream);
  const lv_status st =
      c->mode == LV_FP64
          ? chain_update<double>(c, static_cast<const double*>(U), static_cast<const double*>(V), (int)r, ldu, ldv, s)
          : chain_update<float>(c, static_cast<const float*>(U), static_cast<const float*>(V), (int)r, ldu, ldv, s);
  if (st == LV_OK) c->updates += 1;
  return st;
}

lv_status lv_chain_read(const lv_chain* c, int power, void* out, int64_t ldo, void* stream) {
  g_err[0] = 0;
  if (!c || !out) return fail(LV_EINVAL, "chain or out is NULL");
  if (ldo < c->n) return fail(LV_EINVAL, "ldo < n");
  for (size_t i = 0; i < c->pw.size(); ++i)
    if (c->pw[i] == power) {
      const size_t es = c->elem;
      return hip_check(hipMemcpy2DAsync(out, ldo * es, c->base + c->P[i], c->n_pad * es, c->n * es, c->n,
                                        hipMemcpyDeviceToDevice, static_cast<hipStream_t>(stream)),
                       "read");
    }
  return fail(LV_EINVAL, "power %d is not stored by this model", power);
}

int lv_chain_powers(const lv_chain* c, int* powers, int cap) {
  if (!c) return -1;
  const int ns = (int)c->pw.size();
  for (int i = 0; i < ns && i < cap && powers; ++i) powers[i] = c->pw[i];
  return ns;
}

void lv_chain_destroy(lv_chain* c) { delete c; }

}  // extern "C"
