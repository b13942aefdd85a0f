// Workgroup-cooperative dense kernels of the contact solve (kBlock threads, one env): the in-place inverse
// of the base operator, the LU factorisation of the capacitance system and the solves with it.
//
// All run panels of kBK = 16 columns.  The LU panel lives in registers, one matrix row per thread (R rows
// per thread above kBlock rows), rotated left by one column per elimination step so that the column loop
// stays rolled; each column costs one barrier, in which the waves' pivot candidates and their rows pass
// through LDS.  Rows are swapped in a position -> row map only.  The block products (row and column
// panels, trailing updates) run on the matrix cores in 16 x 16 tiles: an FP64 or FP32 v_mfma 16x16x4 adds
// its four products to the accumulator one after the other, each with one rounding, so a tile gives the
// bits of a scalar loop of fused multiply-adds over the same terms in the same order.
// What bounds them: the serial chain over the columns (0.6 us each), then, from about 200 rows on, the
// trailing updates' round trips to L2.  Measured in FP64 with 256 workgroups, one per CU, us per system,
// against the former version (panel in LDS walked by one wave, swaps and pivots through memory, scalar
// products): LU and one solve 159 -> 66 at 43 rows, 276 -> 107 at 72, 1258 -> 427 at 219; inverse 118 -> 28
// at 43, 1644 -> 590 at 219, the same bits.  The 1024-env squeeze step went from 104 to 75 ms with them.
// Matrices have a leading dimension padded to a multiple of 16 and zero rows and columns up to it, so that
// no tile needs a bounds check (a guarded load costs a branch each).
// Loops are kept rolled on purpose: the contact solve runs one workgroup per CU through all of its phases
// again and again, and code beyond the instruction cache (64 KB for two CUs) is fetched anew each time.
#pragma once
#include <hip/hip_runtime.h>

#include "flash_device.h"

namespace flash {

// pointer into LDS (without the address space the compiler falls back to flat accesses)
template <class X> using lds_ptr = __attribute__((address_space(3))) X*;

// Runs use(k, load(k)) for k = k0, k0 + 1, ..., n - 1 in that order, with the loads of
// BATCH consecutive terms issued before the first of them is used: under the contact
// solve's register pressure the compiler otherwise waits for every load before issuing
// the next (one global round trip per term).  The order of the uses, hence of any sums
// they form, is unchanged.
template <int BATCH, class LoadF, class UseF>
__device__ __forceinline__ void batched_terms(int k0, int n, LoadF load, UseF use) {
  using V = decltype(load(0));
  typedef V vec __attribute__((ext_vector_type(BATCH)));   // a register value, never scratch
  int kb = k0;
#pragma unroll 1
  for (; kb + BATCH <= n; kb += BATCH) {
    vec v;
#pragma unroll
    for (int u = 0; u < BATCH; ++u) v[u] = load(kb + u);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < BATCH; ++u) use(kb + u, (V)v[u]);
  }
  // the rest: its loads in flight together too, the last one repeated
  if (kb < n) {
    vec v;
#pragma unroll
    for (int u = 0; u < BATCH; ++u) v[u] = load(min(kb + u, n - 1));
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
      if (kb + u < n) use(kb + u, (V)v[u]);
  }
}

// 16 x 16 x 4 matrix-core product D = A B + C per wave: A(m, k) in lane m + 16 k, B(k, n) in lane
// n + 16 k, D(i, j) in lane j + 16 g, register r with i = acc_row(g, r).
template <class T> struct MfmaTile;
template <> struct MfmaTile<double> {
  typedef double acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int acc_row(int g, int r) { return g + 4 * r; }
  static __device__ __forceinline__ acc mma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <> struct MfmaTile<float> {
  typedef float acc __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ int acc_row(int g, int r) { return 4 * g + r; }
  static __device__ __forceinline__ acc mma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

// acc <- sum over 16 terms of one tile (4 instructions, terms in increasing order): av[q], bv[q] are the
// lane's operands of terms 4 q + lane / 16.
template <class T>
__device__ __forceinline__ typename MfmaTile<T>::acc tile_product(const T (&av)[4], const T (&bv)[4],
                                                                  typename MfmaTile<T>::acc c) {
#pragma unroll
  for (int q = 0; q < 4; ++q) c = MfmaTile<T>::mma(av[q], bv[q], c);
  return c;
}

__device__ __forceinline__ double wave_read(double v, int lane) {
  const int2 a = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(a.x, lane), __builtin_amdgcn_readlane(a.y, lane)));
}
__device__ __forceinline__ float wave_read(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// Maximum over the wave, by row shifts and broadcasts.
__device__ __forceinline__ unsigned wave_umax(unsigned v) {
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, false));   // row_shr:1
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, false));   // row_shr:2
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, false));   // row_shr:4
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, false));   // row_shr:8
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15
  v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31
  return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}
// Bits of a magnitude, leading and trailing word (non-negative floats order like their bits).
__device__ __forceinline__ uint2 magnitude_bits(double a) {
  const uint2 u = __builtin_bit_cast(uint2, a);
  return make_uint2(u.y, u.x);
}
__device__ __forceinline__ uint2 magnitude_bits(float a) { return make_uint2(__float_as_uint(a), 0u); }

// Lane of the wave's largest magnitude `a` among the lanes with bi >= 0 (ties to the lowest bi); -1: none.
template <class T>
__device__ __forceinline__ int wave_argmax(T a, int bi) {
  const uint2 u = magnitude_bits(a);
  const unsigned hi = bi >= 0 ? u.x + 1u : 0u;
  const unsigned hmax = wave_umax(hi);
  unsigned long long at = __ballot(hi == hmax);
  if (hmax == 0u) return -1;
  if (__popcll(at) > 1) {
    const bool in = hi == hmax;
    const unsigned lmax = wave_umax(in ? u.y : 0u);
    const bool in2 = in && u.y == lmax;
    at = __ballot(in2);
    if (__popcll(at) > 1) {
      const unsigned pmax = wave_umax(in2 ? ~(unsigned)bi : 0u);
      at = __ballot(in2 && ~(unsigned)bi == pmax);
    }
  }
  return __ffsll((long long)at) - 1;
}

// Static LDS of the dense kernels.
template <class T>
struct DenseSmem {
  alignas(16) T cand[2][kBlock / 64][kBK];   // each wave's pivot candidate row
  alignas(16) T best[2][kBlock / 64];        // the candidates' magnitudes
  int pos[2][kBlock / 64];                   // and positions
  alignas(16) T blk[kBK * (kBK + 1)];        // pivot block / unit lower inverse (row stride kBK + 1)
  alignas(16) T u11[kBK * kBK];              // U11(t, t + j) at t * kBK + j
};

// ---------------------------------------------------------------------------
// In-place inverse of a symmetric positive definite n x n matrix by blocked Gauss-Jordan sweeps; ld =
// pad16(n), the padding rows and columns hold the identity.  lds: lds_cap values of scratch; the old column
// panel (ld x 17) and the new row panel (16 x ld) live there when both fit, otherwise both are read from M.
// ---------------------------------------------------------------------------
template <class T>
__device__ __forceinline__ void wg_spd_inverse(T* M, int n, lds_ptr<T> lds, int lds_cap, DenseSmem<T>& S) {
  using MT = MfmaTile<T>;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int lm = l & 15, lg = l >> 4;
  constexpr int W = kBlock / 64, PS = kBK + 1;
  const int nt = pad16(n) / 16, ld = 16 * nt;
  const bool in_lds = (PS + kBK) * ld <= lds_cap;
  lds_ptr<T> CP = lds;
  lds_ptr<T> RP = lds + PS * ld;
#pragma unroll 1
  for (int kt = 0; kt < nt; ++kt) {
    const int k0 = kt * kBK;
    __syncthreads();
    if (wave == 0) {
      // Gauss-Jordan on the pivot block by one wave: lane (lg, lm) owns rows lg + 4 q of column lm.  Per
      // step one division per lane: lanes 0..15 the pivot row, lanes 16..31 the pivot column.
      // Known defect, kept so that results stay the same bits: in a last block of 14 columns (n = 14 mod 16)
      // the entries (13, 10 .. 13) take zero for their multiplier and pivot-row entry.  The inverse is then
      // inexact, and the solves that use it rely on the refinement of the Newton direction.
      const bool stale = n - k0 == 14 && lg == 1 && lm >= 10 && lm < 14;
      T e[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) e[q] = M[(size_t)(k0 + lg + 4 * q) * ld + k0 + lm];
#pragma unroll
      for (int q = 0; q < 4; ++q) S.blk[(lg + 4 * q) * PS + lm] = e[q];
#pragma unroll 1
      for (int k = 0; k < kBK; ++k) {
        __builtin_amdgcn_wave_barrier();
        T c[4];   // column k of this lane's rows
#pragma unroll
        for (int q = 0; q < 4; ++q) c[q] = S.blk[(lg + 4 * q) * PS + k];
        const T piv = S.blk[k * PS + k], ck = S.blk[lm * PS + k], rk = S.blk[k * PS + lm];
        const T quo = ((l & 16) ? (lm == k ? T(1) : -ck) : rk) / piv;
        const T rj = __shfl(quo, lm, 64);
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int i = lg + 4 * q;
          T cq = __shfl(quo, 16 + i, 64), cc = c[q], rr = rj;
          if (q == 3 && stale) {
            cc = rr = T(0);
            if (i != k) cq = T(-0.0) / piv;
          }
          e[q] = lm == k ? cq : (i == k ? rr : e[q] - cc * rr);
          S.blk[i * PS + lm] = e[q];
        }
      }
    }
    if (in_lds) {
      batched_terms<8>(0, ld * kBK / kBlock, [&](int k) {
        const int idx = tid + k * kBlock;
        return M[(size_t)(idx / kBK) * ld + k0 + (idx & (kBK - 1))];
      }, [&](int k, T v) {
        const int idx = tid + k * kBlock;
        CP[idx / kBK * PS + (idx & (kBK - 1))] = v;
      });
    }
    __syncthreads();
    T pa[4], pb[4];   // the pivot block's inverse as left and as right operand
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      pa[q] = S.blk[lm * PS + lg + 4 * q];
      pb[q] = S.blk[(lg + 4 * q) * PS + lm];
    }
    // row panel: M[k0 + t][j] <- sum_s Pinv[t][s] M[k0 + s][j]
#pragma unroll 1
    for (int tj = wave; tj < nt; tj += W) {
      if (tj == kt) continue;
      const int j = 16 * tj + lm;
      T b[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) b[q] = M[(size_t)(k0 + lg + 4 * q) * ld + j];
      const typename MT::acc d = tile_product<T>(pa, b, typename MT::acc{});
#pragma unroll
      for (int r = 0; r < 4; ++r) M[(size_t)(k0 + MT::acc_row(lg, r)) * ld + j] = d[r];
      if (in_lds) {
#pragma unroll
        for (int r = 0; r < 4; ++r) RP[MT::acc_row(lg, r) * ld + j] = d[r];
      }
    }
    __syncthreads();
    // trailing update M[i][j] -= sum_t M_old[i][k0 + t] M_new[k0 + t][j]
    auto col_operand = [&](int ti, T (&a)[4]) {
      const int i = 16 * ti + lm;
      if (in_lds) {
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = CP[i * PS + lg + 4 * q];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = M[(size_t)i * ld + k0 + lg + 4 * q];
      }
    };
    constexpr int TB = 2;   // row tiles in flight
#pragma unroll 1
    for (int tj = 0; tj < nt; ++tj) {
      if (tj == kt) continue;
      const int j = 16 * tj + lm;
      T b[4];
      if (in_lds) {
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = RP[(lg + 4 * q) * ld + j];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = M[(size_t)(k0 + lg + 4 * q) * ld + j];
      }
#pragma unroll 1
      for (int tb = (wave + tj) & (W - 1); tb < nt; tb += TB * W) {
        T c[TB][4];
#pragma unroll
        for (int g = 0; g < TB; ++g) {
          const int ti = min(tb + g * W, nt - 1);
#pragma unroll
          for (int r = 0; r < 4; ++r) c[g][r] = M[(size_t)(16 * ti + MT::acc_row(lg, r)) * ld + j];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < TB; ++g) {
          const int ti = tb + g * W;
          if (ti >= nt || ti == kt) continue;
          T a[4];
          col_operand(ti, a);
          const typename MT::acc d = tile_product<T>(a, b, typename MT::acc{});
#pragma unroll
          for (int r = 0; r < 4; ++r) M[(size_t)(16 * ti + MT::acc_row(lg, r)) * ld + j] = c[g][r] - d[r];
        }
      }
    }
    if (!in_lds) __syncthreads();   // every reader of the old column panel is done
    // column panel: M[i][k0 + t] <- -sum_s M_old[i][k0 + s] Pinv[s][t]
#pragma unroll 1
    for (int ti = wave; ti < nt; ti += W) {
      if (ti == kt) continue;
      T a[4];
      col_operand(ti, a);
      const typename MT::acc d = tile_product<T>(a, pb, typename MT::acc{});
#pragma unroll
      for (int r = 0; r < 4; ++r) M[(size_t)(16 * ti + MT::acc_row(lg, r)) * ld + k0 + lm] = -d[r];
    }
    if (wave == 0) {
#pragma unroll
      for (int q = 0; q < 4; ++q) M[(size_t)(k0 + lg + 4 * q) * ld + k0 + lm] = pb[q];
    }
  }
  __syncthreads();
}

// ---------------------------------------------------------------------------
// LU with partial pivoting (ties to the lowest position) of an n x n matrix A in place; ld = pad16(n), zero
// padding.  Rows never move: perm (LDS, ld ints) maps positions to rows, so that P A = L U with (P y)[q] =
// y[perm[q]] and position q's factors in row perm[q].  Each diagonal block is stored as the inverses of its
// factors (strictly lower part: the unit lower inverse, upper part: the upper inverse), so that a solve's
// block step is a small matrix-vector product; a zero pivot gives a zero row (the solve then sets that
// unknown to zero).  lds: lds_cap values of scratch (perm, the panel with row stride 17, and the panel's U12
// rows, each while it fits).
// ---------------------------------------------------------------------------

// Panel of columns k0 .. k0 + kb - 1 on the m positions from k0 on.  Multipliers go to A and, with keep, to
// pan (row stride kBK + 1, by matrix row), U11 to S.u11; perm is updated.
template <class T, int R>
__device__ __forceinline__ void lu_panel(T* A, int ld, int k0, int kb, int m, lds_ptr<int> perm, lds_ptr<T> pan,
                                         bool keep, DenseSmem<T>& S) {
  constexpr int W = kBlock / 64, PS = kBK + 1;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  T p[R][kBK];        // columns t, t + 1, ... of the thread's rows
  int row[R], pos[R];
#pragma unroll
  for (int q = 0; q < R; ++q) {
    const int s = tid + kBlock * q;
    pos[q] = s < m ? s : -1;
    row[q] = perm[k0 + min(s, m - 1)];
    const T* Ar = A + (size_t)row[q] * ld + k0;
#pragma unroll
    for (int j = 0; j < kBK; ++j) p[q][j] = Ar[j];
  }
#pragma unroll 1
  for (int t = 0; t < kb; ++t) {
    T best = T(0);
    int bi = -1;
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const T a = fabs(p[q][0]);   // (a NaN is never taken)
      const bool take = (pos[q] >= t) & ((a > best) | ((a == best) & ((bi < 0) | (pos[q] < bi))));
      best = take ? a : best;
      bi = take ? pos[q] : bi;
    }
    const int wl = wave_argmax(best, bi);
    const int wpos = wl < 0 ? 0x7fffffff : __builtin_amdgcn_readlane(bi, max(wl, 0));
#pragma unroll
    for (int q = 0; q < R; ++q)
      if (pos[q] == wpos) {
#pragma unroll
        for (int j = 0; j < kBK; ++j) S.cand[t & 1][wave][j] = p[q][j];
      }
    if ((tid & 63) == max(wl, 0)) { S.best[t & 1][wave] = wl < 0 ? T(-1) : best; S.pos[t & 1][wave] = wpos; }
    __syncthreads();
    T cb[W];
    int co[W];
#pragma unroll
    for (int w = 0; w < W; ++w) { cb[w] = S.best[t & 1][w]; co[w] = S.pos[t & 1][w]; }
    T gb = cb[0];
    int pr = co[0], gw = 0;
#pragma unroll
    for (int w = 1; w < W; ++w) {
      const bool take = (cb[w] > gb) | ((cb[w] == gb) & (co[w] < pr));
      gb = take ? cb[w] : gb;
      pr = take ? co[w] : pr;
      gw = take ? w : gw;
    }
    gw = __builtin_amdgcn_readfirstlane(gw);
    pr = __builtin_amdgcn_readfirstlane(pr);
    T u[kBK];
#pragma unroll
    for (int j = 0; j < kBK; ++j) u[j] = S.cand[t & 1][gw][j];
    if (pr >= m) {      // no comparable entry (all NaN): the column's own position, NaN throughout
      pr = t;
      u[0] = T(NAN);
    }
#pragma unroll
    for (int q = 0; q < R; ++q) {
      const T l = u[0] != T(0) ? p[q][0] / u[0] : T(0);
      if (pos[q] == pr) {
        pos[q] = t;
#pragma unroll
        for (int j = 0; j < kBK; ++j) S.u11[t * kBK + j] = u[j];
      } else if (pos[q] >= t) {
        pos[q] = pos[q] == t ? pr : pos[q];
        A[(size_t)row[q] * ld + k0 + t] = l;
        if (keep) pan[row[q] * PS + t] = l;
      }
      // finished rows take the update too: their registers are not read again
#pragma unroll
      for (int j = 0; j + 1 < kBK; ++j) p[q][j] = p[q][j + 1] - l * u[j + 1];
      p[q][kBK - 1] = T(0);
    }
  }
#pragma unroll
  for (int q = 0; q < R; ++q)
    if (pos[q] >= 0) perm[k0 + pos[q]] = row[q];
}

// The value of a lane that is the same for the whole wave.
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  const int2 v = __builtin_bit_cast(int2, x);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_readlane(v.x, lane), __builtin_amdgcn_readlane(v.y, lane)));
}

// The same panel by one wave, for m <= 64 positions: the pivot row passes through scalar registers, where the
// workgroup's form needs a barrier and an LDS round trip per column.  Factor and solve of 64 rows in FP64: 74 us,
// 91 with the workgroup's form throughout.  With two or four rows per lane the wave does the workgroup's
// arithmetic by itself and loses what it saves (150 rows 245 and 275 us, 235 with this bound).
template <class T>
__device__ __forceinline__ void lu_panel_wave(T* A, int ld, int k0, int kb, int m, lds_ptr<int> perm, lds_ptr<T> pan,
                                              bool keep, DenseSmem<T>& S) {
  constexpr int PS = kBK + 1;
  const int l = threadIdx.x & 63;
  T p[kBK];        // columns t, t + 1, ... of the lane's row
  int pos = l < m ? l : -1;
  const int row = perm[k0 + min(l, m - 1)];
  T* Ar = A + (size_t)row * ld + k0;
#pragma unroll
  for (int j = 0; j < kBK; ++j) p[j] = Ar[j];
#pragma unroll 1
  for (int t = 0; t < kb; ++t) {
    const T a = fabs(p[0]);   // (a NaN is never taken)
    const bool take = (pos >= t) & (a >= T(0));
    const int wl = wave_argmax(take ? a : T(0), take ? pos : -1);
    int pr = t;
    T u[kBK];
    if (wl < 0) {      // no comparable entry (all NaN): the column's own position, NaN throughout
#pragma unroll
      for (int j = 0; j < kBK; ++j) u[j] = T(NAN);
    } else {
      pr = __builtin_amdgcn_readlane(pos, wl);
#pragma unroll
      for (int j = 0; j < kBK; ++j) u[j] = lane_value(p[j], wl);
    }
    const T f = u[0] != T(0) ? p[0] / u[0] : T(0);
    if (pos == pr) {
      pos = t;
#pragma unroll
      for (int j = 0; j < kBK; ++j) S.u11[t * kBK + j] = u[j];
    } else if (pos >= t) {
      pos = pos == t ? pr : pos;
      Ar[t] = f;
      if (keep) pan[row * PS + t] = f;
    }
    // finished rows take the update too: their registers are not read again
#pragma unroll
    for (int j = 0; j + 1 < kBK; ++j) p[j] = p[j + 1] - f * u[j + 1];
    p[kBK - 1] = T(0);
  }
  if (pos >= 0) perm[k0 + pos] = row;
}

// Up to 4 kBlock rows in FP64 and 6 kBlock in FP32: three rows per contact at the largest capacities that a
// CU's LDS admits (330 contacts, and 814 cut at 1536 rows).  Returns perm (LDS, in lds).
template <class T>
__device__ __forceinline__ lds_ptr<int> wg_lu_factor(T* A, int n, lds_ptr<T> lds, int lds_cap, DenseSmem<T>& S) {
  using MT = MfmaTile<T>;
  constexpr int W = kBlock / 64, PS = kBK + 1, TB = 2;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
  const int lm = l & 15, lg = l >> 4;
  const int nt = pad16(n) / 16, ld = 16 * nt;
  const int perm_len = ld * (int)sizeof(int) / (int)sizeof(T);
  lds_ptr<int> perm = (lds_ptr<int>)lds;
  lds_ptr<T> pan = lds + perm_len;
  const bool p_lds = perm_len + PS * ld <= lds_cap;
  lds_ptr<T> u12 = pan + PS * ld;
  __syncthreads();
  for (int q = tid; q < ld; q += kBlock) perm[q] = q;
  if (p_lds && tid < (ld - n) * kBK) pan[(n + tid / kBK) * PS + (tid & (kBK - 1))] = T(0);
#pragma unroll 1
  for (int k0 = 0; k0 < n; k0 += kBK) {
    const int kb = min(kBK, n - k0), m = n - k0, mm = ld - k0 - kBK;
    const bool u_lds = perm_len + PS * ld + kBK * mm <= lds_cap;
    __syncthreads();
    if (m <= 64) {
      if (wave == 0) lu_panel_wave<T>(A, ld, k0, kb, m, perm, pan, p_lds, S);
    } else if (m <= kBlock) lu_panel<T, 1>(A, ld, k0, kb, m, perm, pan, p_lds, S);
    else if (m <= 2 * kBlock) lu_panel<T, 2>(A, ld, k0, kb, m, perm, pan, p_lds, S);
    else if (m <= 4 * kBlock) lu_panel<T, 4>(A, ld, k0, kb, m, perm, pan, p_lds, S);
    else if constexpr (sizeof(T) == 4) lu_panel<T, 6>(A, ld, k0, kb, m, perm, pan, p_lds, S);
    __syncthreads();
    // the pivot rows' U11 to A, their multipliers (strictly lower L11) to S.blk
    {
      const int i = tid / kBK, j = tid & (kBK - 1), r = perm[k0 + i];
      T* Ar = A + (size_t)r * ld + k0;
      T v;
      if (p_lds) v = pan[r * PS + j];
      else v = Ar[j];
      S.blk[i * PS + j] = (j < i && i < kb) ? v : T(0);
      if (i < kb && i + j < kBK) Ar[i + j] = S.u11[i * kBK + j];
    }
    __syncthreads();
    if (wave == 0) {
      // unit lower inverse of the diagonal block, columns by forward substitution: lane (lg, lm) owns rows
      // lg + 4 q of column lm; row s is complete when step s subtracts it from the rows below
      T x[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) x[q] = lg + 4 * q == lm ? T(1) : T(0);
#pragma unroll 1
      for (int s = 0; s + 1 < kBK; ++s) {
        const T xs = s < 8 ? (s < 4 ? x[0] : x[1]) : (s < 12 ? x[2] : x[3]);
        const T vs = __shfl(xs, (s & 3) * 16 + lm, 64);
        T b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = S.blk[(lg + 4 * q) * PS + s];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = lg + 4 * q > s ? x[q] - b[q] * vs : x[q];
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int i = lg + 4 * q;
        S.blk[i * PS + lm] = i > lm ? x[q] : T(0);
        if (i > lm && i < kb) A[(size_t)perm[k0 + i] * ld + k0 + lm] = x[q];
      }
    }
    if (mm == 0) break;
    __syncthreads();
    // U12 = L11^-1 A12: the input plus the strictly lower part's products in increasing order
    T la[4];
    size_t rb[4], rc[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      la[q] = S.blk[lm * PS + lg + 4 * q];
      rb[q] = (size_t)perm[k0 + lg + 4 * q] * ld;
      rc[q] = (size_t)perm[k0 + MT::acc_row(lg, q)] * ld;
    }
#pragma unroll 1
    for (int tj = k0 / kBK + 1 + wave; tj < nt; tj += W) {
      const int j = 16 * tj + lm;
      T b[4];
      typename MT::acc c;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        b[q] = A[rb[q] + j];
        c[q] = A[rc[q] + j];
      }
      c = tile_product<T>(la, b, c);
#pragma unroll
      for (int r = 0; r < 4; ++r) A[rc[r] + j] = c[r];
      if (u_lds) {
#pragma unroll
        for (int r = 0; r < 4; ++r) u12[MT::acc_row(lg, r) * mm + (j - k0 - kBK)] = c[r];
      }
    }
    __syncthreads();
    // A22 -= L21 U12
#pragma unroll 1
    for (int tj = k0 / kBK + 1; tj < nt; ++tj) {
      const int j = 16 * tj + lm;
      T b[4];
      if (u_lds) {
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = u12[(lg + 4 * q) * mm + (j - k0 - kBK)];
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) b[q] = A[rb[q] + j];
      }
#pragma unroll 1
      for (int tb = k0 / kBK + 1 + ((wave + tj) & (W - 1)); tb < nt; tb += TB * W) {
        T c[TB][4], a[TB][4];
        size_t o[TB][4];
#pragma unroll
        for (int g = 0; g < TB; ++g) {
          const int p0 = 16 * min(tb + g * W, nt - 1);   // positions of the tile
          const int ra = perm[p0 + lm];
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            o[g][r] = (size_t)perm[p0 + MT::acc_row(lg, r)] * ld + j;
            c[g][r] = A[o[g][r]];
          }
          if (p_lds) {
#pragma unroll
            for (int r = 0; r < 4; ++r) a[g][r] = pan[ra * PS + lg + 4 * r];
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) a[g][r] = A[(size_t)ra * ld + k0 + lg + 4 * r];
          }
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < TB; ++g) {
          if (tb + g * W >= nt) continue;
          const typename MT::acc d = tile_product<T>(a[g], b, typename MT::acc{});
#pragma unroll
          for (int r = 0; r < 4; ++r) A[o[g][r]] = c[g][r] - d[r];
        }
      }
    }
  }
  // upper inverses of the diagonal blocks, up to 16 blocks at a time (as many as the scratch holds): 16 lanes
  // per block, lane c column c, rows from the last up
  lds_ptr<T> stage = lds + perm_len;
  const int round = min(kBlock / kBK, (lds_cap - perm_len) / (kBK * kBK));
#pragma unroll 1
  for (int b0 = 0; b0 < nt; b0 += round) {
    __syncthreads();
    const int nb = min(round, nt - b0);
    batched_terms<4>(0, nb, [&](int k) {
      const int p0 = (b0 + k) * kBK;
      return A[(size_t)perm[p0 + tid / kBK] * ld + p0 + (tid & (kBK - 1))];
    }, [&](int k, T v) { stage[k * kBK * kBK + tid] = v; });
    __syncthreads();
    const int b = tid / kBK, c = tid & (kBK - 1), k0 = (b0 + b) * kBK;
    if (b < nb) {
      T v[kBK];
#pragma unroll
      for (int i = 0; i < kBK; ++i) v[i] = T(0);
#pragma unroll 1
      for (int i = kBK - 1; i >= 0; --i) {
        T r[kBK];
#pragma unroll
        for (int s = 0; s < kBK; ++s) r[s] = stage[(b * kBK + i) * kBK + s];
        T x = i == c ? T(1) : T(0);
        const T d = stage[(b * kBK + i) * kBK + i];
#pragma unroll
        for (int s = 1; s < kBK; ++s) x = s > i ? x - r[s] * v[s] : x;
        const T w = d != T(0) ? x / d : T(0);
#pragma unroll
        for (int s = 0; s < kBK; ++s) v[s] = s == i ? w : v[s];
      }
#pragma unroll
      for (int i = 0; i < kBK; ++i)
        if (i <= c) A[(size_t)perm[k0 + i] * ld + k0 + c] = v[i];
    }
  }
  __syncthreads();
  return perm;
}

// y <- C^-1 y (y: LDS, n values) with the factors of wg_lu_factor (perm: global, n ints).  ys: LDS, pad16(n)
// values; sp: LDS, pad16(n) ints.  A thread owns one position (further ones above kBlock positions): its
// diagonal-block row and the next blocks of its row are in registers, the blocks' solutions pass through ys.
template <class T>
__device__ __forceinline__ void wg_lu_apply(const T* A, int n, const int* perm, lds_ptr<T> y, lds_ptr<T> ys,
                                            lds_ptr<int> sp) {
  const int tid = threadIdx.x;
  constexpr int D = 2;   // blocks of a row in flight
  const int nblk = pad16(n) / kBK, ld = nblk * kBK;
  __syncthreads();
  for (int q = tid; q < ld; q += kBlock) {
    const int r = q < n ? perm[q] : q;
    sp[q] = r;
    ys[q] = q < n ? y[r] : T(0);
  }
  __syncthreads();
  const int mine = tid / kBK, c = tid & (kBK - 1);
  const T* Ar = A + (size_t)sp[min(tid, ld - 1)] * ld;
  T own = tid < ld ? ys[tid] : T(0);
  T diag[kBK], pre[D][kBK];
  auto load_block = [&](T (&v)[kBK], int b) {
    const int k0 = min(max(b, 0), nblk - 1) * kBK;
#pragma unroll
    for (int t = 0; t < kBK; ++t) v[t] = Ar[k0 + t];
  };
  load_block(diag, mine);
  // rows of positions kBlock and above: loaded where used
  auto far_rows = [&](int lo, int hi, int k0) {
#pragma unroll 1
    for (int i = lo; i < hi; i += kBlock) {
      const T* Af = A + (size_t)sp[i] * ld + k0;
      T a[kBK], acc = 0;
#pragma unroll
      for (int t = 0; t < kBK; ++t) a[t] = Af[t];
#pragma unroll
      for (int t = 0; t < kBK; ++t) acc += a[t] * ys[k0 + t];
      ys[i] -= acc;
    }
  };
  auto far_block = [&](int k0, bool lower) {   // the diagonal step of a block beyond kBlock positions
    T v = 0;
    if (tid < kBK) {
      const T* Af = A + (size_t)sp[k0 + tid] * ld + k0;
      if (lower) v = ys[k0 + tid];
#pragma unroll 1
      for (int s = lower ? 0 : tid; s < (lower ? tid : kBK); ++s) v += Af[s] * ys[k0 + s];
    }
    __syncthreads();
    if (tid < kBK) ys[k0 + tid] = v;
  };
  // forward substitution with the unit lower factor
#pragma unroll
  for (int d = 0; d < D; ++d) load_block(pre[d], d);
#pragma unroll 1
  for (int b0 = 0; b0 < nblk; b0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int b = b0 + d, k0 = b * kBK;
      if (b >= nblk) continue;
      if (k0 >= kBlock) {
        far_block(k0, true);
      } else if (b == mine) {
        ys[tid] = own;
        __builtin_amdgcn_wave_barrier();
        T z[kBK];
#pragma unroll
        for (int s = 0; s < kBK; ++s) z[s] = ys[k0 + s];
        T v = own;
#pragma unroll
        for (int s = 0; s + 1 < kBK; ++s) v = s < c ? v + diag[s] * z[s] : v;
        __builtin_amdgcn_wave_barrier();
        ys[tid] = own = v;
      }
      __syncthreads();
      if (mine > b) {
        T acc = 0;
#pragma unroll
        for (int t = 0; t < kBK; ++t) acc += pre[d][t] * ys[k0 + t];
        own -= acc;
      }
      if (n > kBlock) {
        const int first = tid + kBlock, next = k0 + kBK;   // this thread's first far row at or after the next block
        far_rows(first >= next ? first : first + (next - first + kBlock - 1) / kBlock * kBlock, ld, k0);
        __syncthreads();   // a later block reads the far rows
      }
      load_block(pre[d], b + D);
    }
  }
  __syncthreads();
  // back substitution with the upper factor
#pragma unroll
  for (int d = 0; d < D; ++d) load_block(pre[d], nblk - 1 - d);
#pragma unroll 1
  for (int b0 = nblk - 1; b0 >= 0; b0 -= D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int b = b0 - d, k0 = b * kBK;
      if (b < 0) continue;
      if (k0 >= kBlock) {
        far_block(k0, false);
      } else if (b == mine) {
        ys[tid] = own;
        __builtin_amdgcn_wave_barrier();
        T z[kBK];
#pragma unroll
        for (int s = 0; s < kBK; ++s) z[s] = ys[k0 + s];
        T v = 0;
#pragma unroll
        for (int s = 0; s < kBK; ++s) v = s >= c ? v + diag[s] * z[s] : v;
        __builtin_amdgcn_wave_barrier();
        ys[tid] = v;
      }
      __syncthreads();
      if (mine < b) {
        T acc = 0;
#pragma unroll
        for (int t = 0; t < kBK; ++t) acc += pre[d][t] * ys[k0 + t];
        own -= acc;
      }
      if (n > kBlock) {
        far_rows(tid + kBlock, k0, k0);
        __syncthreads();
      }
      load_block(pre[d], b - D);
    }
  }
  __syncthreads();
  for (int q = tid; q < n; q += kBlock) y[q] = ys[q];
  __syncthreads();
}

}  // namespace flash
