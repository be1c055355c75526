// Fused level pass of the IncrExp update (LINVIEW, App. A exponential model).
//
// For one level j of the exponential model the update needs, with the OLD
// stored power P = A^(2^j) and the level factors U_j, V_j (n x R, R = 2^j r):
//     X = P U_j,   Y = P^T V_j,   G = V_j^T U_j,   P += U_j V_j^T
// and then U_{j+1} = [U_j, X + U_j G], V_{j+1} = [Y, V_j]  (Sec. 4.3, App. A).
//
// k_level_fused does the first four in ONE read and ONE write of P: a tile of
// P is streamed through registers once, in coalesced row segments; Y, X and
// the rank-R update all take the lane's own columns, and X is added over the
// lanes in registers.
// Each tile writes partial X / Y (and the column-tile-0 tiles partial Grams);
// k_level_tail reduces them in a fixed order (deterministic, no float
// atomics) and assembles the next level's factors.  k_level_update is the
// update-only pass of the top stored power.
//
// Layouts (all row-major):
//   P        n_pad x ldp, zero padding beyond n.
//   slab U   n_pad x W; U_j = columns [0, R).
//   slab V   n_pad x W; V_j = columns [W - R, W)  (callers pass the offset base).
//   partX    [nct][n_pad][R]   (nct = n_pad / TC column tiles)
//   partY    [nrt][n_pad][R]   (nrt row tiles)
//   partG    [nrt][R][R] double
#include "lv_device.h"

namespace lv {
namespace {

// ---------------------------------------------------------------- lane sums
//
// x[0 .. N) holds, in every lane, that lane's term of N sums over the wave.
// sum_lanes adds them over the 64 lanes and leaves sum i in the lane(s) with
// sum_index(lane) = i: at each of six steps two lists are merged into one
// (half of the lanes keep one sum, their partners the other), so N sums cost
// about N + 6 additions instead of 6 N.  The steps pair lanes 32, 16 and 8
// apart, mirrored within 8, then 2 and 1 apart, whatever N is: a sum has the
// same bits whichever sums it is merged with.
template <int S> __device__ __forceinline__ unsigned lane_move(unsigned v) {
  // S = 2: row_ror:8, 3: row_half_mirror, 4: quad_perm [2,3,0,1], 5: quad_perm [1,0,3,2]
  constexpr int ctrl = S == 2 ? 0x128 : S == 3 ? 0x141 : S == 4 ? 0x4E : 0xB1;
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, true);
}
template <int S> __device__ __forceinline__ uint2 lane_swap(unsigned a, unsigned b) {
  // the upper half (S = 0) or the odd rows of 16 (S = 1) of a against the
  // lower half or the even rows of b
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  u2 r;
  if constexpr (S == 0) r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  else r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
  return make_uint2(r.x, r.y);
}

// One step: the sums of a (kept by the lanes without bit S) and of b.
template <int S, typename T> __device__ __forceinline__ T merge_lanes(T a, T b, const int lane) {
  if constexpr (S < 2) {
    if constexpr (sizeof(T) == 4) {
      const uint2 r = lane_swap<S>(__builtin_bit_cast(unsigned, a), __builtin_bit_cast(unsigned, b));
      return __builtin_bit_cast(T, r.x) + __builtin_bit_cast(T, r.y);
    } else {
      const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
      const uint2 lo = lane_swap<S>(x.x, y.x), hi = lane_swap<S>(x.y, y.y);
      return __builtin_bit_cast(T, make_uint2(lo.x, hi.x)) + __builtin_bit_cast(T, make_uint2(lo.y, hi.y));
    }
  } else {
    const bool up = (lane >> (5 - S)) & 1;
    const T keep = up ? b : a, send = up ? a : b;
    if constexpr (sizeof(T) == 4) {
      return keep + __builtin_bit_cast(T, lane_move<S>(__builtin_bit_cast(unsigned, send)));
    } else {
      const uint2 x = __builtin_bit_cast(uint2, send);
      return keep + __builtin_bit_cast(T, make_uint2(lane_move<S>(x.x), lane_move<S>(x.y)));
    }
  }
}

template <int S, int N, int END = 6, typename T>
__device__ __forceinline__ T sum_lanes(const T (&x)[N], const int lane) {
  if constexpr (S == END) {
    static_assert(N == 1, "too many sums for the steps");
    return x[0];
  } else {
    T y[(N + 1) / 2];
#pragma unroll
    for (int i = 0; i < (N + 1) / 2; ++i)
      y[i] = merge_lanes<S, T>(x[2 * i], N == 1 ? x[0] : 2 * i + 1 < N ? x[2 * i + 1] : T(0), lane);
    return sum_lanes<S + 1, (N + 1) / 2, END, T>(y, lane);
  }
}
constexpr int log2c(int n) { return n <= 1 ? 0 : 1 + log2c(n / 2); }
__device__ __forceinline__ int sum_index(const int lane) { return (int)(__brev((unsigned)lane) >> 26); }

// ---------------------------------------------------------------- fused pass
//
// Block: 256 threads (4 waves).  Columns: TC = 64 lanes x 16 B.  Rows: the
// matrix is cut into blocks of RB = 4 rows, and the ns = ceil(n_pad /
// tile_rows) row slices of a column tile interleave: slice s owns the row
// blocks b = s, s + ns, s + 2 ns, ... (about tile_rows rows in all), and its
// wave w the i-th of them for i = w, w + 4, w + 8, ...  At any moment the grid
// thus streams one contiguous band of rows rather than ns bands a tile apart,
// which the HBM serves at a markedly higher rate.  A lane holds one 16-byte
// column group: its rows of U_j and V_j and its Y sums stay in registers for
// the whole tile.  Per block a wave forms, from the same registers, the Y
// terms of the lane's columns, the lane's terms of X (summed over the lanes by
// sum_lanes) and the updated rows; the next block is in flight meanwhile.
// The block's own factor rows arrive as one gathered load per 64 entries, go
// to a wave-private LDS block and are read back as broadcasts.  No block-wide
// barrier runs inside the row loop.  The four waves' Y sums meet once at the
// end of the tile.
//
// TT > 1: the factors of TT successive updates are known (a batch, see
// update_batch_pipelined), and one read and one write of P serve them all:
// per block, update t's products are formed from the rows as update t - 1
// left them in registers.  Every sum and every rounding is the one of TT
// passes with TT = 1, so the results are the same bit for bit.  Factors and
// partials of update t lie t * vs.s, t * vs.x, ... further on.  HBM
// bounds the pass up to TT R = 8 (6 TT R flops per element against 8 bytes:
// 0.75 TT R flop/B where the vector units' ridge is 9.8), the vector units
// slightly at 16.
//
// LF: the lane's factor rows (8 TT R values) do not fit the registers beside
// its 4 TT R sums of Y: they stay in LDS, staged once per tile (the four waves
// share the columns), [factor column][lane] so that a wave reads 1 KiB in a
// row, and are read once per block, up to 4 factor columns at a time.
//
// UPD = false gives the read-only variant used for ranks above 16: the
// skinny products of 16 factor columns at a time (partials written with row
// stride pR at the chunk's column offset), the rank update and the Gram done
// by k_level_update and k_gram.
//
// Variants for views that keep the sums of powers or a general form as well
// (one pass over a stored matrix instead of two or three):
//   XE, XD   X is formed for XE + XD more columns: XE taken from Ux (same
//            stride W), XD from Ud (stride Wd), X = P [U_j, Q_j, D_j]; the
//            extra blocks' partials go to partX2 (row stride XE) and partX3
//            (row stride XD).  The powers' pass thus also yields P_j Q_j
//            (sums) and P_j D_j (the general form's delta or factor slab).
//   SP       no X: Y = S^T Vy with the old S for RY columns of another factor
//            Vy, and the rank update S += Uj Vj^T; no Gram.  The sums pass
//            (Uj = Q_j, Vj = W_j, Vy = V_j), and the step of the linear and
//            skip models that forms the next factor from P_b^T V_a and
//            updates P_b.
//   GR       (UPD = false) the Gram Vy^T Uj is formed as well; WY = false: no Y.
template <typename T, int R, int TT, bool UPD, int XE = 0, bool SP = false, int XD = 0, int RY = R, bool GR = UPD && !SP,
          bool WY = true>
__device__ __forceinline__ void fused_body(const FusedDesc<T>& d, const int ct, const int rt, const Strides& vs = {}) {
  constexpr int RB = kFusedRowBlock;
  constexpr int EPL = 16 / (int)sizeof(T);
  constexpr int TC = 64 * EPL;
  constexpr int C = R * TT;                     // factor columns of all the updates
  constexpr int XR = SP ? 1 : R + XE + XD;      // columns of X per update
  constexpr int NX = RB * TT * XR;              // lane sums per block
  constexpr int CY = SP ? RY : C;               // columns of Y
  static_assert(!SP || (UPD && XE == 0 && XD == 0), "the sums pass updates and forms no X");
  static_assert(TT == 1 || (UPD && !SP && XE == 0 && XD == 0), "several updates: the plain pass only");
  static_assert(SP || RY == R, "Y has the factors' columns");
  static_assert(WY || !UPD, "passes without Y read only");
  static_assert(SP || NX <= 64, "one lane per X sum");
  constexpr bool LF = !SP && XE == 0 && XD == 0 && (C > 8 || TT > 1);
  constexpr int CH = R < 4 ? R : 4;             // factor columns read at a time (LF)
  constexpr int YC = CY < 4 ? CY : 4;           // Y columns exchanged at a time
  constexpr int FB = RB * C, FBY = RB * CY;     // factor entries per block: U, and the Y operand
  constexpr int FM = FB > FBY ? FB : FBY;
  constexpr int FN = (FM + 63) / 64;

  __shared__ __align__(16) T facs[4][UPD ? 2 : 1][FM];
  // the lanes' factor rows (LF: U, then V), and the exchange of the Y sums
  constexpr int NF = LF ? (UPD ? 2 : 1) * C * TC : 0;
  __shared__ __align__(16) T lbuf[NF > 4 * TC * YC ? NF : 4 * TC * YC];
  T* const ybuf = lbuf;

  T* __restrict__ P = d.P;
  const int64_t ldp = d.ldp;
  const int n_pad = d.n_pad, W = d.W, pR = d.pR;
  const T* __restrict__ Uj = d.Uj;
  const T* __restrict__ Vj = d.Vj;
  const T* __restrict__ Yop = SP ? d.Vy : d.Vj;
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = wave_id();
  const int col0 = ct * TC;
  const int ns = (n_pad + d.tile_rows - 1) / d.tile_rows;   // row slices
  const int nb_all = n_pad / RB;
  const int nblocks = (nb_all - rt + ns - 1) / ns;          // row blocks of slice rt
  // first row of the slice's i-th row block
  auto blk_row = [&](int i) -> int64_t { return (int64_t)(rt + ns * i) * RB; };
  const int lc = col0 + lane * EPL;

  // entry e = (t TT + v) R + c of a block's factor rows (row t, update v,
  // column c) sits in lane e % 64 of f[e / 64]; foff: byte offset of the
  // lane's entry from the block's first factor row (32 bits: lv_view_impl.h has
  // the bound of the last update's)
  unsigned foff[FN], foffy[SP ? FN : 1];
#pragma unroll
  for (int f = 0; f < FN; ++f) {
    const int e = lane + 64 * f < FB ? lane + 64 * f : 0;
    foff[f] = (unsigned)(((TT > 1 ? (e / R % TT) * vs.s : 0) + (int64_t)(e / C) * W + e % R) * sizeof(T));
    if constexpr (SP) {
      const int ey = lane + 64 * f < FBY ? lane + 64 * f : 0;
      foffy[f] = (unsigned)(((int64_t)(ey / RY) * d.Wy + ey % RY) * sizeof(T));
    }
  }
  // A matrix that is only read is mostly read again soon (A in every step of
  // the linear models): loads that may stay in the 256 MB memory-side cache
  // pay as long as it holds the matrix (IncrLin, rank 1, k = 16: n = 5120 24 ->
  // 19 us per pass, n = 8192 0.80 -> 0.79 ms per update, n = 10240 1.30 -> 1.44).
  // Passes that write the matrix back stream it either way (n = 8192: 487 us
  // per update, 543 with cached accesses).
  const bool cached = (int64_t)n_pad * ldp * (int64_t)sizeof(T) <= kCacheBytes;
  V16<T> p[RB], pn[RB];
  T fy[FN], fu[UPD ? FN : 1], fyn[FN], fun[UPD ? FN : 1];
  auto load_block = [&](V16<T> (&pp)[RB], T (&y)[FN], T (&u)[UPD ? FN : 1], const int64_t r0) {
    if (!UPD && cached) {
#pragma unroll
      for (int t = 0; t < RB; ++t) pp[t] = ld16(P + (r0 + t) * ldp + lc);
    } else {
#pragma unroll
      for (int t = 0; t < RB; ++t) pp[t] = ld16_nt(P + (r0 + t) * ldp + lc);
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      if constexpr (SP) y[f] = *at_byte(Yop + r0 * d.Wy, foffy[f]);
      else if constexpr (WY) y[f] = *at_byte(Yop + r0 * W, foff[f]);
      if constexpr (UPD) u[f] = *at_byte(Uj + r0 * W, foff[f]);
    }
  };
  if (wave < nblocks) load_block(p, fy, fu, blk_row(wave));

  // the lane's factor rows
  T ucol[LF ? 1 : TT][EPL][XR], vcol[LF ? 1 : TT][EPL][UPD ? R : 1], yacc[TT][EPL][SP ? RY : R];
  if constexpr (LF) {
    constexpr int OPS = UPD ? 2 : 1;
#pragma unroll
    for (int i = 0; i < (OPS * TT * TC + 255) / 256; ++i) {
      const int idx = tid + 256 * i, col = idx % TC, v = idx / TC % TT, op = idx / (TC * TT);
      if (OPS * TT * TC % 256 != 0 && idx >= OPS * TT * TC) continue;
      const unsigned g = (unsigned)((col0 + col) * W * (int)sizeof(T));
      T f[R];
      load_row<T, R>(at_byte((op ? Vj : Uj) + v * vs.s, g), f);
#pragma unroll
      for (int c = 0; c < R; ++c) lbuf[(op * C + v * R + c) * TC + col] = f[c];
    }
    __syncthreads();
  }
#pragma unroll
  for (int v = 0; v < TT; ++v)
#pragma unroll
    for (int q = 0; q < EPL; ++q) {
#pragma unroll
      for (int c = 0; c < (SP ? RY : R); ++c) yacc[v][q][c] = T(0);
      if constexpr (LF) continue;
      const unsigned g = (unsigned)((lc + q) * W * (int)sizeof(T));
      load_row<T, UPD ? R : 0>(at_byte(Vj + v * vs.s, g), vcol[v][q]);
      if constexpr (!SP) {
        T u[R];
        load_row<T, R>(at_byte(Uj + v * vs.s, g), u);
#pragma unroll
        for (int c = 0; c < R; ++c) ucol[v][q][c] = u[c];
#pragma unroll
        for (int c = 0; c < XE; ++c) ucol[v][q][R + c] = at_byte(d.Ux, g)[c];
#pragma unroll
        for (int c = 0; c < XD; ++c) ucol[v][q][R + XE + c] = d.Ud[(int64_t)(lc + q) * d.Wd + c];
      }
    }

  // where the lane's X sum of a block goes: sum i = (t TT + v) XR + c
  T* xdst = nullptr;
  int xs = 0;
  if constexpr (!SP) {
    const int i = sum_index(lane);
    const int t = i / (TT * XR), v = i / XR % TT, c = i % XR;
    const int64_t row = (int64_t)ct * n_pad + t;
    if (i < NX) {
      if (c < R) { xs = pR; xdst = d.partX + v * vs.x + row * pR + c; }
      if constexpr (XE > 0)
        if (c >= R && c < R + XE) { xs = XE; xdst = d.partX2 + row * XE + c - R; }
      if constexpr (XD > 0)
        if (c >= R + XE) { xs = XD; xdst = d.partX3 + row * XD + c - R - XE; }
    }
  }

  T* fac_y = facs[wave][0];
  T* fac_u = facs[wave][UPD ? 1 : 0];
  for (int b = wave; b < nblocks; b += 4) {
    const int64_t r0 = blk_row(b);
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      if constexpr (WY)
        if (lane + 64 * f < FBY) fac_y[lane + 64 * f] = fy[f];
      if constexpr (UPD)
        if (lane + 64 * f < FB) fac_u[lane + 64 * f] = fu[f];
    }
    if (b + 4 < nblocks) load_block(pn, fyn, fun, blk_row(b + 4));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    if constexpr (LF) {
      // (re-read in every block: held in registers across blocks, as the
      // compiler would otherwise do, they spill)
      asm volatile("" ::: "memory");
      const T* lu = lbuf + lane * EPL;
      T xs1[RB * TT];   // sums over the lanes of the steps that R columns take
#pragma unroll
      for (int v = 0; v < TT; ++v) {
        T s[RB][EPL], xc[RB][R / CH];
#pragma unroll
        for (int c0 = 0; c0 < R; c0 += CH) {
          V16<T> uc[CH], vc[UPD ? CH : 1];
#pragma unroll
          for (int c = 0; c < CH; ++c) {
            uc[c] = ld16(lu + (v * R + c0 + c) * TC);
            if constexpr (UPD) vc[c] = ld16(lu + (C + v * R + c0 + c) * TC);
          }
#pragma unroll
          for (int t = 0; t < RB; ++t) {
            T vi[CH], x[CH];
            if constexpr (WY) load_row<T, CH>(fac_y + (t * TT + v) * R + c0, vi);
#pragma unroll
            for (int c = 0; c < CH; ++c) {
              if constexpr (WY)
#pragma unroll
                for (int q = 0; q < EPL; ++q) yacc[v][q][c0 + c] = fma(p[t].v[q], vi[c], yacc[v][q][c0 + c]);
              x[c] = p[t].v[0] * uc[c].v[0];
#pragma unroll
              for (int q = 1; q < EPL; ++q) x[c] = fma(p[t].v[q], uc[c].v[q], x[c]);
            }
            xc[t][c0 / CH] = sum_lanes<0, CH, log2c(CH), T>(x, lane);
            if constexpr (UPD) {
              T ui[CH];
              load_row<T, CH>(fac_u + (t * TT + v) * R + c0, ui);
#pragma unroll
              for (int q = 0; q < EPL; ++q) {
                if constexpr (R == 1) {
                  s[t][q] = fma(ui[0], vc[0].v[q], p[t].v[q]);
                } else {
                  s[t][q] = c0 == 0 ? ui[0] * vc[0].v[q] : fma(ui[0], vc[0].v[q], s[t][q]);
#pragma unroll
                  for (int c = 1; c < CH; ++c) s[t][q] = fma(ui[c], vc[c].v[q], s[t][q]);
                }
              }
            }
          }
        }
#pragma unroll
        for (int t = 0; t < RB; ++t) {
          xs1[t * TT + v] = sum_lanes<log2c(CH), R / CH, log2c(R), T>(xc[t], lane);
          if constexpr (UPD) {
#pragma unroll
            for (int q = 0; q < EPL; ++q) p[t].v[q] = R == 1 ? s[t][q] : p[t].v[q] + s[t][q];
          }
        }
        // Y's sums are due here: the compiler would otherwise form them at the
        // block's end and keep (spill) every update's rows until then
        if constexpr (TT > 1) {
#pragma unroll
          for (int q = 0; q < EPL; ++q)
#pragma unroll
            for (int c = 0; c < R; ++c) asm volatile("" : "+v"(yacc[v][q][c]));
        }
      }
      if constexpr (UPD) {
#pragma unroll
        for (int t = 0; t < RB; ++t) st16_nt(P + (r0 + t) * ldp + lc, p[t]);
      }
      const T s = sum_lanes<log2c(R), RB * TT, 6, T>(xs1, lane);
      if (xs != 0) xdst[r0 * xs] = s;
    }
    T x[SP || LF ? 1 : NX];
#pragma unroll
    for (int t = 0; t < (LF ? 0 : RB); ++t) {
#pragma unroll
      for (int v = 0; v < TT; ++v) {
        constexpr int YR = SP ? RY : R;
        if constexpr (WY) {
          T vi[YR];
          load_row<T, YR>(fac_y + (t * TT + v) * YR, vi);
#pragma unroll
          for (int q = 0; q < EPL; ++q)
#pragma unroll
            for (int c = 0; c < YR; ++c) yacc[v][q][c] = fma(p[t].v[q], vi[c], yacc[v][q][c]);
        }
        if constexpr (!SP) {
#pragma unroll
          for (int c = 0; c < XR; ++c) {
            T s = p[t].v[0] * ucol[v][0][c];
#pragma unroll
            for (int q = 1; q < EPL; ++q) s = fma(p[t].v[q], ucol[v][q][c], s);
            x[(t * TT + v) * XR + c] = s;
          }
        }
        if constexpr (UPD) {
          T ui[R];
          load_row<T, R>(fac_u + (t * TT + v) * R, ui);
#pragma unroll
          for (int q = 0; q < EPL; ++q) {
            if constexpr (R == 1) {
              p[t].v[q] = fma(ui[0], vcol[v][q][0], p[t].v[q]);
            } else {
              T s = ui[0] * vcol[v][q][0];
#pragma unroll
              for (int c = 1; c < R; ++c) s = fma(ui[c], vcol[v][q][c], s);
              p[t].v[q] += s;
            }
          }
        }
      }
      if constexpr (UPD) st16_nt(P + (r0 + t) * ldp + lc, p[t]);
    }
    if constexpr (!SP && !LF) {
      const T s = sum_lanes<0, NX, 6, T>(x, lane);
      if (xs != 0) xdst[r0 * xs] = s;
    }
#pragma unroll
    for (int t = 0; t < RB; ++t) p[t] = pn[t];
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      fy[f] = fyn[f];
      if constexpr (UPD) fu[f] = fun[f];
    }
    // the next block's entries overwrite the LDS block only after every
    // lane has read this block's
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }

  // Y partial of this tile: the four waves' sums, YC of the CY columns
  // (update v, column c: v R + c) at a time.
  constexpr int YR = SP ? RY : R;
#pragma unroll
  for (int c0 = 0; c0 < (WY ? CY : 0); c0 += YC) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < EPL; ++q)
#pragma unroll
      for (int c = 0; c < YC; ++c) ybuf[(wave * TC + lane * EPL + q) * YC + c] = yacc[(c0 + c) / YR][q][(c0 + c) % YR];
    __syncthreads();
    for (int idx = tid; idx < TC * YC; idx += 256) {
      const int cc = idx / YC, c = idx % YC;
      const T s = ((ybuf[(0 * TC + cc) * YC + c] + ybuf[(1 * TC + cc) * YC + c]) +
                   ybuf[(2 * TC + cc) * YC + c]) + ybuf[(3 * TC + cc) * YC + c];
      const int v = (c0 + c) / YR;
      d.partY[v * vs.y + ((int64_t)rt * n_pad + col0 + cc) * pR + (c0 + c) % YR] = s;
    }
  }

  // Partial Gram V_j^T U_j over this slice's rows (double accumulation).
  // The TT R^2 pairs are spread over the column tiles (pair p on column tile
  // p mod nct), so no block carries much more work than the others; 32
  // consecutive lanes take a pair, lane g the rows g, g + 32, ... of the slice
  // (counted in slice order), and their sums are added by a butterfly.
  if constexpr (GR) {
    constexpr int NP = R * R;
    const T* __restrict__ Vg = UPD ? Vj : d.Vy;
    const int Wg = UPD ? W : d.Wy;
    const int nct = n_pad / TC;
    const int nsr = nblocks * RB;   // rows of the slice
    const int g0 = tid % 32;
    for (int pair = ct + nct * (tid / 32); pair < TT * NP; pair += 8 * nct) {
      const int v = pair / NP, ab = pair % NP;
      const T* vp = Vg + v * vs.s + ab / R;
      const T* up = Uj + v * vs.s + ab % R;
      double g = 0.0;
#pragma unroll 4
      for (int q = g0; q < nsr; q += 32) {
        const int64_t i = blk_row(q / RB) + q % RB;
        g = fma((double)vp[i * Wg], (double)up[i * W], g);
      }
#pragma unroll
      for (int off = 16; off > 0; off >>= 1) g += __shfl_xor(g, off, 32);
      if (g0 == 0) d.partG[v * vs.g + (int64_t)rt * NP + ab] = g;
    }
  }
}

// Two waves per SIMD for passes over several updates: the widest would
// otherwise take a few registers more than that leaves.
template <int TT> constexpr int fused_min_waves() { return TT > 1 ? 2 : 1; }

template <typename T, int R, int TT, bool UPD>
__global__ void __launch_bounds__(256, (fused_min_waves<TT>())) k_level_fused(const FusedDesc<T> d, const Strides vs) {
  fused_body<T, R, TT, UPD>(d, blockIdx.x, blockIdx.y, vs);
}

// Read-only: X = P Uj alone.
template <typename T, int R>
__global__ void __launch_bounds__(256) k_level_x(const FusedDesc<T> d) {
  fused_body<T, R, 1, false, 0, false, 0, R, false, false>(d, blockIdx.x, blockIdx.y);
}

// The same pass with gridDim.y below the slice count: row slices rt =
// blockIdx.y, blockIdx.y + gridDim.y, ... one after the other (fewer,
// longer-lived work-groups; every slice is summed exactly as with one
// work-group per slice, so the partials are the same bit for bit).
template <typename T, int R, int TT, bool UPD>
__global__ void __launch_bounds__(256) k_level_fused_grouped(const FusedDesc<T> d) {
  const int ns = (d.n_pad + d.tile_rows - 1) / d.tile_rows;
  for (int rt = blockIdx.y; rt < ns; rt += gridDim.y) {
    fused_body<T, R, TT, UPD>(d, blockIdx.x, rt);
    __syncthreads();   // the next slice reuses the LDS blocks
  }
}

// The powers' pass of a view with sums or a general form: X also for Q_j
// (XE = R columns or none) and for D_j (XD columns or none).
template <typename T, int R, int XE, int XD>
__global__ void __launch_bounds__(256) k_level_fused_x(const FusedDesc<T> d) {
  fused_body<T, R, 1, true, XE, false, XD>(d, blockIdx.x, blockIdx.y);
}

// The sums pass: Y = S^T Vy (old S), S += Q_j W_j^T.
template <typename T, int R>
__global__ void __launch_bounds__(256) k_sums_fused(const FusedDesc<T> d) {
  fused_body<T, R, 1, true, 0, true>(d, blockIdx.x, blockIdx.y);
}

// A step of the linear and skip models in one launch: work-groups of the
// first nsx slices form X = P_a M with the Gram (dx, RY columns), the others
// Y = P_b^T V_a and P_b += U_b V_b^T (dy, update rank R).  The two passes are
// independent, and each alone leaves the device half idle at small orders.
template <typename T, int R, int RY>
__global__ void __launch_bounds__(256) k_krylov_step(const FusedDesc<T> dx, const FusedDesc<T> dy, const int nsx) {
  if ((int)blockIdx.y < nsx)
    fused_body<T, RY, 1, false, 0, false, 0, RY, true, false>(dx, blockIdx.x, blockIdx.y);
  else
    fused_body<T, R, 1, true, 0, true, 0, RY>(dy, blockIdx.x, (int)blockIdx.y - nsx);
}

// Read-only: X = P Uj with the Gram Vy^T Uj, and Y = P^T Vj if WY.
template <typename T, int R, bool WY>
__global__ void __launch_bounds__(256) k_fused_xgram(const FusedDesc<T> d) {
  fused_body<T, R, 1, false, 0, false, 0, R, true, WY>(d, blockIdx.x, blockIdx.y);
}

template <typename T, int R, bool UPD>
__global__ void __launch_bounds__(256) k_level_fused_multi(const FusedDesc<T>* __restrict__ ds, int nd) {
  const int v = find_desc(ds, nd, (int)blockIdx.x);
  const FusedDesc<T> d = load_desc(ds, v);
  const int local = (int)blockIdx.x - d.block_begin;
  fused_body<T, R, 1, UPD>(d, local % d.nct, local / d.nct);
}

template <typename T, int R, int TT, bool UPD>
hipError_t fused_launch(const FusedDesc<T>& d, hipStream_t s, int slice_groups = 0, const Strides& vs = {}) {
  const int ns = (d.n_pad + d.tile_rows - 1) / d.tile_rows;
  if constexpr (!UPD) {
    if (d.partY == nullptr) {
      hipLaunchKernelGGL((k_level_x<T, R>), dim3((unsigned)d.nct, (unsigned)ns), dim3(256), 0, s, d);
      return hipGetLastError();
    }
  }
  if constexpr (UPD && R <= 8 && TT == 1) {
    if (slice_groups > 0 && slice_groups < ns) {
      hipLaunchKernelGGL((k_level_fused_grouped<T, R, TT, UPD>), dim3((unsigned)d.nct, (unsigned)slice_groups),
                         dim3(256), 0, s, d);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_level_fused<T, R, TT, UPD>), dim3((unsigned)d.nct, (unsigned)ns), dim3(256), 0, s, d, vs);
  return hipGetLastError();
}

// The fused pass over nver updates (1, 2, 4, ..., up to chain_updates(R)).
template <typename T, int R, int TT>
hipError_t fused_chain(const FusedDesc<T>& d, hipStream_t s, int slice_groups, int nver, const Strides& vs) {
  if (nver == TT) return fused_launch<T, R, TT, true>(d, s, slice_groups, vs);
  if constexpr (2 * TT <= chain_updates(R)) return fused_chain<T, R, 2 * TT>(d, s, slice_groups, nver, vs);
  return hipErrorInvalidValue;
}

// One level with rank R: for R <= 16 the fused pass; above, the skinny
// products in 16-column chunks (read-only passes), the Gram, then the rank-R
// update pass.
template <typename T, int R>
hipError_t fused_r(const FusedDesc<T>& d, hipStream_t s, int slice_groups, int nver, const Strides& vs) {
  if constexpr (R <= kMaxFusedRank) {
    return fused_chain<T, R, 1>(d, s, slice_groups, nver, vs);
  } else {
    if (nver != 1) return hipErrorInvalidValue;
    constexpr int RC = kMaxFusedRank;
    for (int c0 = 0; c0 < R; c0 += RC) {
      FusedDesc<T> c = d;
      c.Uj += c0;
      c.Vj += c0;
      c.partX += c0;
      c.partY += c0;
      c.partG = nullptr;
      hipError_t e = fused_launch<T, RC, 1, false>(c, s);
      if (e != hipSuccess) return e;
    }
    const T* slabV = d.Vj - (d.W - R);
    hipError_t e = launch_level_gram<T>(R, d.Uj, slabV, d.W, d.n_pad, d.partG, s);
    if (e != hipSuccess) return e;
    return launch_level_update<T>(R, d.P, d.ldp, d.n_pad, d.Uj, slabV, d.W, s);
  }
}

template <typename T>
FusedDesc<T> fused_desc(int R, T* P, int64_t ldp, int64_t n_pad, int tile_rows, const T* Uj, const T* Vj, int W,
                        T* partX, T* partY, double* partG) {
  return {P, ldp, (int)n_pad, tile_rows, Uj, Vj, W, partX, partY, partG, R, (int)(n_pad / tile_cols<T>()), 0};
}

}  // namespace

template <typename T>
hipError_t launch_level_fused(int R, T* P, int64_t ldp, int64_t n_pad, int tile_rows,
                              const T* slabU, const T* slabV, int W, T* partX, T* partY,
                              double* partG, hipStream_t s, int slice_groups, int nver, const Strides& vs) {
  const FusedDesc<T> d = fused_desc<T>(R, P, ldp, n_pad, tile_rows, slabU, slabV + (W - R), W, partX, partY, partG);
  LV_RANK_SWITCH(R, return (fused_r<T, RR>(d, s, slice_groups, nver, vs)))
}

// Launch k_level_fused_x for level rank R with XE (0 or R) and xd (0, 1, 2,
// 4 or 8) extra columns, R + XE + xd <= kFusedXCap; the sums of the plain
// pass, so X for U_j, Y, the Gram and the update are bit-identical to it.
template <typename T, int R, int XE>
hipError_t fused_x_launch(int xd, const FusedDesc<T>& d, dim3 grid, hipStream_t s) {
  switch (xd) {
#define LV_FUSED_X_CASE(XD)                                                                   \
    case XD:                                                                                  \
      if constexpr (R + XE + XD <= kFusedXCap) {                                              \
        hipLaunchKernelGGL((k_level_fused_x<T, R, XE, XD>), grid, dim3(256), 0, s, d);        \
        return hipGetLastError();                                                             \
      }                                                                                       \
      return hipErrorInvalidValue;
    LV_FUSED_X_CASE(0)
    LV_FUSED_X_CASE(1)
    LV_FUSED_X_CASE(2)
    LV_FUSED_X_CASE(4)
    LV_FUSED_X_CASE(8)
#undef LV_FUSED_X_CASE
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_level_fused_x(int R, T* P, int64_t ldp, int64_t n_pad, int tile_rows, const T* slabU,
                                const T* slabV, int W, T* partX, T* partY, double* partG, const T* slabQ, T* partXq,
                                const T* Dop, int ldd, int xd, T* partXd, hipStream_t s) {
  if (!fused_extra_fits(R, slabQ != nullptr, xd)) return hipErrorInvalidValue;
  const int nct = (int)(n_pad / tile_cols<T>());
  FusedDesc<T> d{P, ldp, (int)n_pad, tile_rows, slabU, slabV + (W - R), W, partX, partY, partG, R, nct, 0};
  d.Ux = slabQ;
  d.partX2 = partXq;
  d.Ud = Dop;
  d.Wd = ldd;
  d.partX3 = partXd;
  const dim3 grid((unsigned)nct, (unsigned)((n_pad + tile_rows - 1) / tile_rows));
  const bool q = slabQ != nullptr;
  switch (R) {
    case 1: return q ? fused_x_launch<T, 1, 1>(xd, d, grid, s) : fused_x_launch<T, 1, 0>(xd, d, grid, s);
    case 2: return q ? fused_x_launch<T, 2, 2>(xd, d, grid, s) : fused_x_launch<T, 2, 0>(xd, d, grid, s);
    case 4: return q ? fused_x_launch<T, 4, 4>(xd, d, grid, s) : fused_x_launch<T, 4, 0>(xd, d, grid, s);
    case 8: return q ? fused_x_launch<T, 8, 8>(xd, d, grid, s) : fused_x_launch<T, 8, 0>(xd, d, grid, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_sums_fused(int R, T* S, int64_t ldp, int64_t n_pad, int tile_rows, const T* slabQ,
                             const T* slabW, const T* slabV, int W, T* partY, hipStream_t s) {
  const int nct = (int)(n_pad / tile_cols<T>());
  FusedDesc<T> d{S, ldp, (int)n_pad, tile_rows, slabQ, slabW + (W - R), W, nullptr, partY, nullptr, R, nct, 0};
  d.Vy = slabV + (W - R);
  d.Wy = W;
  const dim3 grid((unsigned)nct, (unsigned)((n_pad + tile_rows - 1) / tile_rows));
  switch (R) {
    case 1: hipLaunchKernelGGL((k_sums_fused<T, 1>), grid, dim3(256), 0, s, d); break;
    case 2: hipLaunchKernelGGL((k_sums_fused<T, 2>), grid, dim3(256), 0, s, d); break;
    case 4: hipLaunchKernelGGL((k_sums_fused<T, 4>), grid, dim3(256), 0, s, d); break;
    case 8: hipLaunchKernelGGL((k_sums_fused<T, 8>), grid, dim3(256), 0, s, d); break;
    case 16: hipLaunchKernelGGL((k_sums_fused<T, 16>), grid, dim3(256), 0, s, d); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, int RY>
hipError_t krylov_step_r(int R, const FusedDesc<T>& dx, const FusedDesc<T>& dy, hipStream_t s) {
  const int nsx = (dx.n_pad + dx.tile_rows - 1) / dx.tile_rows, nsy = (dy.n_pad + dy.tile_rows - 1) / dy.tile_rows;
  const dim3 grid((unsigned)dx.nct, (unsigned)(nsx + nsy));
#define LV_STEP_CASE(RR)                                                                      \
  case RR:                                                                                    \
    if constexpr (RR >= RY) {                                                                 \
      hipLaunchKernelGGL((k_krylov_step<T, RR, RY>), grid, dim3(256), 0, s, dx, dy, nsx);     \
      return hipGetLastError();                                                               \
    }                                                                                         \
    return hipErrorInvalidValue;
  switch (R) {
    LV_STEP_CASE(1) LV_STEP_CASE(2) LV_STEP_CASE(4) LV_STEP_CASE(8) LV_STEP_CASE(16)
    default: return hipErrorInvalidValue;
  }
#undef LV_STEP_CASE
}

template <typename T>
hipError_t launch_krylov_step(int R, int RY, const T* Pa, T* Pb, int64_t ldp, int64_t n_pad, int rows_x, int rows_y,
                              const T* M, const T* Ub, const T* Vb, int Wb, const T* Va, int Wa, T* partX, T* partY,
                              double* partG, hipStream_t s) {
  FusedDesc<T> dx = fused_desc<T>(RY, const_cast<T*>(Pa), ldp, n_pad, rows_x, M, nullptr, Wb, partX, nullptr, partG);
  FusedDesc<T> dy = fused_desc<T>(RY, Pb, ldp, n_pad, rows_y, Ub, Vb, Wb, nullptr, partY, nullptr);
  dx.Vy = dy.Vy = Va;
  dx.Wy = dy.Wy = Wa;
  switch (RY) {
    case 1: return krylov_step_r<T, 1>(R, dx, dy, s);
    case 2: return krylov_step_r<T, 2>(R, dx, dy, s);
    case 4: return krylov_step_r<T, 4>(R, dx, dy, s);
    case 8: return krylov_step_r<T, 8>(R, dx, dy, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t launch_fused_xgram(int R, const T* P, int64_t ldp, int64_t n_pad, int tile_rows, const T* U, int W,
                              const T* V, int Wv, T* partX, T* partY, double* partG, hipStream_t s) {
  // P is not written; Y takes the factors' stride, so it needs V beside U
  FusedDesc<T> d = fused_desc<T>(R, const_cast<T*>(P), ldp, n_pad, tile_rows, U, V, W, partX, partY, partG);
  if (partY != nullptr && W != Wv) return hipErrorInvalidValue;
  d.Vy = V;
  d.Wy = Wv;
  const dim3 grid((unsigned)d.nct, (unsigned)((n_pad + tile_rows - 1) / tile_rows));
#define LV_XGRAM_CASE(RR)                                                                                     \
  case RR:                                                                                                    \
    if (partY != nullptr) hipLaunchKernelGGL((k_fused_xgram<T, RR, true>), grid, dim3(256), 0, s, d);         \
    else hipLaunchKernelGGL((k_fused_xgram<T, RR, false>), grid, dim3(256), 0, s, d);                         \
    return hipGetLastError();
  switch (R) {
    LV_XGRAM_CASE(1) LV_XGRAM_CASE(2) LV_XGRAM_CASE(4) LV_XGRAM_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef LV_XGRAM_CASE
}

template <typename T>
hipError_t launch_fused_multi(int R, bool chunk, const FusedDesc<T>* ds, int nd, int blocks, hipStream_t s) {
  if (blocks <= 0) return hipSuccess;
  if (chunk) {
    hipLaunchKernelGGL((k_level_fused_multi<T, kMaxFusedRank, false>), dim3((unsigned)blocks), dim3(256), 0, s,
                       ds, nd);
    return hipGetLastError();
  }
  switch (R) {
    case 1: hipLaunchKernelGGL((k_level_fused_multi<T, 1, true>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    case 2: hipLaunchKernelGGL((k_level_fused_multi<T, 2, true>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    case 4: hipLaunchKernelGGL((k_level_fused_multi<T, 4, true>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    case 8: hipLaunchKernelGGL((k_level_fused_multi<T, 8, true>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    case 16: hipLaunchKernelGGL((k_level_fused_multi<T, 16, true>), dim3((unsigned)blocks), dim3(256), 0, s, ds, nd); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Read-only pass: partial X = P Uop and, with a non-null partY, Y = P^T Vop
// for R columns (row stride R), P unchanged: the fused kernel without its
// update and Gram, in 16-column chunks above 16.
template <typename T>
hipError_t launch_level_readonly(int R, const T* P, int64_t ldp, int64_t n_pad, int tile_rows, const T* Uop,
                                 const T* Vop, int W, T* partX, T* partY, hipStream_t s) {
  // P is not written: UPD = false
  FusedDesc<T> d = fused_desc<T>(R, const_cast<T*>(P), ldp, n_pad, tile_rows, Uop, Vop, W, partX, partY, nullptr);
  switch (R) {
    case 1: return fused_launch<T, 1, 1, false>(d, s);
    case 2: return fused_launch<T, 2, 1, false>(d, s);
    case 4: return fused_launch<T, 4, 1, false>(d, s);
    case 8: return fused_launch<T, 8, 1, false>(d, s);
    default: break;
  }
  if (R % kMaxFusedRank != 0 || R > 128) return hipErrorInvalidValue;
  for (int c0 = 0; c0 < R; c0 += kMaxFusedRank) {
    const hipError_t e = fused_launch<T, kMaxFusedRank, 1, false>(d, s);
    if (e != hipSuccess) return e;
    d.Uj += kMaxFusedRank;
    d.Vj += kMaxFusedRank;
    d.partX += kMaxFusedRank;
    if (d.partY != nullptr) d.partY += kMaxFusedRank;
  }
  return hipSuccess;
}

template hipError_t launch_level_readonly<float>(int, const float*, int64_t, int64_t, int, const float*, const float*,
                                                 int, float*, float*, hipStream_t);
template hipError_t launch_level_readonly<double>(int, const double*, int64_t, int64_t, int, const double*,
                                                  const double*, int, double*, double*, hipStream_t);

template hipError_t launch_level_fused<float>(int, float*, int64_t, int64_t, int, const float*, const float*, int,
                                              float*, float*, double*, hipStream_t, int, int, const Strides&);
template hipError_t launch_level_fused<double>(int, double*, int64_t, int64_t, int, const double*, const double*,
                                               int, double*, double*, double*, hipStream_t, int, int, const Strides&);
template hipError_t launch_level_fused_x<float>(int, float*, int64_t, int64_t, int, const float*, const float*, int,
                                                float*, float*, double*, const float*, float*, const float*, int, int,
                                                float*, hipStream_t);
template hipError_t launch_level_fused_x<double>(int, double*, int64_t, int64_t, int, const double*, const double*,
                                                 int, double*, double*, double*, const double*, double*,
                                                 const double*, int, int, double*, hipStream_t);
template hipError_t launch_sums_fused<float>(int, float*, int64_t, int64_t, int, const float*, const float*,
                                             const float*, int, float*, hipStream_t);
template hipError_t launch_sums_fused<double>(int, double*, int64_t, int64_t, int, const double*, const double*,
                                              const double*, int, double*, hipStream_t);
#define LV_INST(T)                                                                                                \
  template hipError_t launch_krylov_step<T>(int, int, const T*, T*, int64_t, int64_t, int, int, const T*, const T*,    \
                                            const T*, int, const T*, int, T*, T*, double*, hipStream_t);          \
  template hipError_t launch_fused_xgram<T>(int, const T*, int64_t, int64_t, int, const T*, int, const T*, int, T*, T*, \
                                            double*, hipStream_t);
LV_INST(float)
LV_INST(double)
#undef LV_INST
template hipError_t launch_fused_multi<float>(int, bool, const FusedDesc<float>*, int, int, hipStream_t);
template hipError_t launch_fused_multi<double>(int, bool, const FusedDesc<double>*, int, int, hipStream_t);

}  // namespace lv
