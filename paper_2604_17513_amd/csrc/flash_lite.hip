// Lightweight contact update in global memory (Alg. 1 with the inertia-only metric of Eq. 10)
// for contact counts beyond what one CU's LDS holds.
//
// Each update reads the current displacement u = z + h^2 Gbar H^T lambda (the position update
// of Alg. 1, formed by the explicit-inverse product over the contact rows), evaluates Phi and its
// generalized-Jacobian blocks at Y = F^T u per contact, and takes lambda <- lambda + delta with
// (K W~ + E) delta = -Phi per vertex, W~ = h^2 H M^-1 H^T.  The metric couples only the contacts
// of one vertex, so every vertex group is updated by one thread from global memory.  The contact displacement
// follows lambda through the global product instead of the contact-space Delassus operator, so no cap x cap
// matrix exists.
//
// An update is two launches, the product and k_lite_update, because one launch costs about as long as the
// product's own work on a small batch.  k_lite_update adds up the product's partial sums itself, folds its
// contacts' residuals into the env's slot of this update, and forms the next multipliers before the env's
// residual is known: they go to the other of two buffers, and the next product and update leave an env alone
// whose last residual met the tolerance.  k_lite_end then counts, sums u for every vertex, and brings the
// multipliers of the update an env stopped at back to the first buffer.
#include <hip/hip_runtime.h>

#include <type_traits>
#include <utility>

#include "flash_contact.h"
#include "flash_device.h"
#include "flash_launch.h"

namespace flash {

namespace {

__device__ __forceinline__ double wg_max(double v, double* sh) {
  for (int d = 32; d > 0; d >>= 1) v = fmax(v, __shfl_xor(v, d, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  double m = sh[0];
  for (int w = 1; w < kBlock / 64; ++w) m = fmax(m, sh[w]);
  __syncthreads();
  return m;
}

// Residual of contact j at (u of its vertex, lambda lj), FP64, at the residual scale s = h^2 / m_v.
template <class T, class CT>
__device__ __forceinline__ double lite_residual(const DevBatch<T>& B, size_t cb, int j, const CT* F, const T (&u)[3],
                                                const double* lj, CT mu) {
  const double uw0 = (double)u[0], uw1 = (double)u[1], uw2 = (double)u[2];
  double Y[3];
  for (int a = 0; a < 3; ++a) Y[a] = (double)F[3 * a] * uw0 + (double)F[3 * a + 1] * uw1 + (double)F[3 * a + 2] * uw2;
  const double s = (double)B.cs[cb + j];
  const double cnd = B.cd0d[cb + j] + Y[0];
  const double ut1 = Y[1] - (double)B.cdob[2 * (cb + j)], ut2 = Y[2] - (double)B.cdob[2 * (cb + j) + 1];
  const bool att = B.cobs[cb + j] >= kMaxObs;
  const double pn = att ? cnd : fmin(cnd, s * lj[0]);
  const double z1 = lj[1] - ut1 / s, z2 = lj[2] - ut2 / s;
  const double nz = sqrt(z1 * z1 + z2 * z2);
  const double rh = (double)mu * fmax(lj[0], 0.0);
  double q1 = z1, q2 = z2;
  if (!att && nz > rh) { const double f = nz > 0 ? rh / nz : 0.0; q1 = f * z1; q2 = f * z2; }
  const double t1 = s * (lj[1] - q1), t2 = s * (lj[2] - q2);
  const double rj = fmax(fabs(pn), sqrt(t1 * t1 + t2 * t2));
  return rj == rj ? rj : INFINITY;
}

template <class T, class CT>
__device__ __forceinline__ const CT* lite_frames(const DevBatch<T>& B, size_t cb) {
  if constexpr (std::is_same<CT, T>::value) return B.cframe + 9 * cb;
  else return B.cframe64 + 9 * cb;
}

// Multipliers and world forces before (0) and after an odd number of updates of a local-global iteration.
template <class T>
__device__ __forceinline__ double* lite_lambda(const DevBatch<T>& B, int it) { return it & 1 ? B.lite_lam : B.clam; }
template <class T>
__device__ __forceinline__ T* lite_force(const DevBatch<T>& B, int it) { return it & 1 ? B.lite_force : B.cforce; }

__device__ __forceinline__ int lite_slots(int lg_iterations, int max_newton) { return lg_iterations * (max_newton + 1); }

// Whether env e had stopped by the update of `slot` (its residual met the tolerance; slots of later updates
// stay zero, so it stays stopped).
template <class T>
__device__ __forceinline__ bool lite_stopped(const DevBatch<T>& B, int e, int slot) {
  const unsigned long long r = B.lite_r[(size_t)e * lite_slots(B.lg_iterations, B.max_newton) + slot];
  return __longlong_as_double((long long)r) <= B.tol;
}

// An env's product at a vertex: its row-split partials in split order, kSumBatch loads per component in flight.
constexpr int kSumBatch = 8;
template <class T>
__device__ __forceinline__ void split_sum(const T* P, int ns, int n, int col, T (&s)[3]) {
  s[0] = s[1] = s[2] = 0;
  for (int s0 = 0; s0 < ns; s0 += kSumBatch) {
    T v[kSumBatch][3];
#pragma unroll
    for (int q = 0; q < kSumBatch; ++q)
#pragma unroll
      for (int k = 0; k < 3; ++k) v[q][k] = P[((size_t)min(s0 + q, ns - 1) * 3 + k) * n + col];
#pragma unroll
    for (int q = 0; q < kSumBatch; ++q)
#pragma unroll
      for (int k = 0; k < 3; ++k) s[k] = s0 + q < ns ? s[k] + v[q][k] : s[k];
  }
}
// u = z + h^2 s.  The roundings are fixed (components 0 and 2 fused, 1 not), so that both kernels that form u, and
// any compiler, give the same bits; these are the bits the step has always had.
template <class T>
__device__ __forceinline__ T displaced(T z, T hh, T s, int k) {
#pragma clang fp contract(off)
  if (k == 1) {
    const T p = hh * s;
    return z + p;
  }
  return __builtin_elementwise_fma(hh, s, z);
}
template <class T>
__device__ __forceinline__ int split_count(const DevBatch<T>& B, int n, int nrows) {
  const int R = split_rows(split_cover(n, B.cap));
  return (nrows + R - 1) / R;
}

// Once per step, after detection: world forces F lambda of the warm start (the first position
// update reads them); the env's residual slots cleared.  Grid: (chunks of kBlock contacts, envs).
template <class T, class CT>
__global__ void __launch_bounds__(kBlock) k_lite_prepare(DevBatch<T> B) {
  const int e = blockIdx.y;
  const int c = B.ccount[e];
  const size_t cb = (size_t)e * B.cap;
  const CT* Fr = lite_frames<T, CT>(B, cb);
  const int j = blockIdx.x * kBlock + threadIdx.x;
  if (j < c) {
    const CT* F = Fr + 9 * j;
    const double* lj = B.clam + 3 * (cb + j);
    const CT l0 = (CT)lj[0], l1 = (CT)lj[1], l2 = (CT)lj[2];
    for (int k = 0; k < 3; ++k) B.cforce[3 * (cb + j) + k] = (T)(F[k] * l0 + F[3 + k] * l1 + F[6 + k] * l2);
  }
  if (blockIdx.x == 0) {
    const int ns = lite_slots(B.lg_iterations, B.max_newton);
    for (int q = threadIdx.x; q < ns; q += kBlock) B.lite_r[(size_t)e * ns + q] = 0ull;
  }
}

// Residual and update `it` of every env that has not stopped; partial: the product's partial sums.  Grid:
// (chunks of kBlock contacts, envs).  Each workgroup folds its contacts' maximum into the env's slot
// (non-negative doubles order like their bits, so an integer atomic maximum gives the exact maximum whatever
// the order); every vertex group whose first contact lies in the chunk takes one update, except with it =
// max_newton, which only evaluates.  Latency bound (one chain of dependent loads per contact): 7 us for 4104
// contacts, where the sum of partials, the residual and the update took a launch each, 5 us apiece.
template <class T, class CT>
__global__ void __launch_bounds__(kBlock) k_lite_update(DevBatch<T> B, const T* mu_env, int slot, int it,
                                                        const T* partial, const int64_t* poff) {
  __shared__ double sh_red[kBlock / 64];
  const int e = blockIdx.y;
  const int c = B.ccount[e];
  const int j0 = blockIdx.x * kBlock;
  if (j0 >= c || (it > 0 && lite_stopped(B, e, slot - 1))) return;
  const size_t cb = (size_t)e * B.cap;
  const CT* Fr = lite_frames<T, CT>(B, cb);
  const int v0 = B.voff[e];
  const int n = B.voff[e + 1] - v0;
  const CT mu = (CT)mu_env[e];
  const int j = j0 + threadIdx.x;
  const int* cv = B.cvert + cb;
  const double* lam_in = lite_lambda(B, it);
  T u[3] = {0, 0, 0};
  double rloc = 0.0;
  if (j < c) {
    T s[3];
    split_sum(partial + poff[e], split_count(B, n, c), n, cv[j], s);
    const T hh = (T)(B.h * B.h);
    for (int k = 0; k < 3; ++k) u[k] = displaced(B.z[(size_t)k * B.NV + v0 + cv[j]], hh, s[k], k);
    rloc = lite_residual<T, CT>(B, cb, j, Fr + 9 * j, u, lam_in + 3 * (cb + j), mu);
  }
  const double r = wg_max(rloc, sh_red);
  if (threadIdx.x == 0)
    atomicMax(&B.lite_r[(size_t)e * lite_slots(B.lg_iterations, B.max_newton) + slot],
              (unsigned long long)__double_as_longlong(r));
  if (it >= B.max_newton || j >= c) return;
  if (j > 0 && cv[j - 1] == cv[j]) return;   // not the first contact of its vertex
  double* lam_out = lite_lambda(B, it + 1);
  T* force = lite_force(B, it + 1);
  const int* cobs = B.cobs + cb;
  const double dmaxf = B.max_force;
  int m = 1;
  while (j + m < c && cv[j + m] == cv[j] && m < kCacheSlots) ++m;
  const CT uw0 = (CT)u[0], uw1 = (CT)u[1], uw2 = (CT)u[2];
  CT Y[3 * kCacheSlots], d0[kCacheSlots], dob[2 * kCacheSlots], dl[3 * kCacheSlots];
  double lam[3 * kCacheSlots];
  for (int q = 0; q < m; ++q) {
    const CT* F = Fr + 9 * (j + q);
    for (int a = 0; a < 3; ++a) {
      Y[3 * q + a] = F[3 * a] * uw0 + F[3 * a + 1] * uw1 + F[3 * a + 2] * uw2;
      lam[3 * q + a] = lam_in[3 * (cb + j + q) + a];
    }
    d0[q] = (CT)B.cd0[cb + j + q];
    dob[2 * q] = (CT)B.cdob[2 * (cb + j + q)];
    dob[2 * q + 1] = (CT)B.cdob[2 * (cb + j + q) + 1];
  }
  const CT sp = (CT)B.cs[cb + j];
  if (m == 1) {
    CT ph[3], K[3][3], E[3][3];
    lite_contact(sp, mu, d0[0], dob[0], dob[1], Y, lam, cobs[j] >= kMaxObs, ph, K, E);
    // Z = sp K + E = [sp 0 0; E_tn sp I]
    const CT dn = -ph[0] / sp;
    dl[0] = dn;
    dl[1] = (-ph[1] - E[1][0] * dn) / sp;
    dl[2] = (-ph[2] - E[2][0] * dn) / sp;
  } else {
    lite_group_solve<CT>(m, sp, mu, Fr + 9 * j, d0, dob, Y, lam, cobs + j, dl);
  }
  for (int q = 0; q < m; ++q) {
    const CT* F = Fr + 9 * (j + q);
    double ln[3];
    for (int a = 0; a < 3; ++a) {
      ln[a] = fmin(fmax(lam[3 * q + a] + (double)dl[3 * q + a], -dmaxf), dmaxf);
      lam_out[3 * (cb + j + q) + a] = ln[a];
    }
    const CT l0 = (CT)ln[0], l1 = (CT)ln[1], l2 = (CT)ln[2];
    for (int k = 0; k < 3; ++k) force[3 * (cb + j + q) + k] = (T)(F[k] * l0 + F[3 + k] * l1 + F[6 + k] * l2);
  }
}

// End of a local-global iteration whose updates have the slots from slot0 on: u = z + h^2 Gbar H^T lambda for
// every vertex, the multipliers and forces of an odd number of updates back in the first buffer, and the
// counters and flags.  Grid: (chunks of kBlock vertices or contacts, envs).
template <class T>
__global__ void __launch_bounds__(kBlock) k_lite_end(DevBatch<T> B, int slot0, int first_lg, const T* partial,
                                                     const int64_t* poff) {
  const int e = blockIdx.y;
  const int c = B.ccount[e];
  const int v0 = B.voff[e];
  const int n = B.voff[e + 1] - v0;
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (blockIdx.x * kBlock >= max(n, c)) return;
  int it = 0;
  while (it < B.max_newton && !lite_stopped(B, e, slot0 + it)) ++it;
  if (i < n) {
    T s[3];
    split_sum(partial + poff[e], split_count(B, n, c), n, i, s);
    const T hh = (T)(B.h * B.h);
    for (int k = 0; k < 3; ++k) {
      const size_t o = (size_t)k * B.NV + v0 + i;
      B.u[o] = displaced(B.z[o], hh, s[k], k);
    }
  }
  if ((it & 1) && i < c) {
    const size_t o = 3 * ((size_t)e * B.cap + i);
    for (int k = 0; k < 3; ++k) {
      B.clam[o + k] = B.lite_lam[o + k];
      B.cforce[o + k] = B.lite_force[o + k];
    }
  }
  if (i == 0) {
    const bool open = !lite_stopped(B, e, slot0 + it);
    B.iters[e] += it;
    if (B.phase) {
      unsigned long long* cnt = B.phase + (size_t)B.n_envs * 8 + 8 * e;
      cnt[3] += open ? 1 : 0;
      cnt[6] += it;
      cnt[7] += 1;
    }
    if (c > 0 && open) B.flags[e] |= 2; else B.flags[e] &= ~2;
    if (first_lg && B.ws_state) B.ws_state[e] &= ~5;
  }
}

// Partial sums of one row split of env e's explicit-inverse product for one column tile.
// ROWS = false: rows 0..n-1 with the right-hand side b (z = Gbar b); ROWS = true: the contact
// rows with their world forces (Gbar H^T lambda).  Gbar is symmetric, so rows are
// read along their length (VW columns per lane, non-temporal: each row is read once per product).
// Few envs are bound by latency, not bandwidth: a wave reads its 128 rows of a split in batches of UNROLL, two
// batches in flight.  One env of 4096 vertices (128 workgroups of 16-byte lanes): 25 us at 4 rows a batch, 15 us
// with 4-byte lanes (four times the workgroups) and 16 rows.
template <class T, bool ROWS, int VW, int UNROLL>
__global__ void __launch_bounds__(kBlock) k_gemv_split(DevBatch<T> B, const int4* items, const T* force, int slot,
                                                       T* partial, const int64_t* poff) {
  constexpr int TILE = 64 * VW;
  constexpr int WS = kBlock / 64;
  typedef T vec_t __attribute__((ext_vector_type(VW)));
  typedef T f4_t __attribute__((ext_vector_type(4)));
  __shared__ f4_t s_vec[kSplitRows];   // (b0, b1, b2, 0) per staged row
  __shared__ int s_row[kSplitRows];
  __shared__ T s_red[(WS - 1) * 3 * TILE];
  const int4 item = items[blockIdx.x];
  const int e = item.x, tile0 = item.y, split = item.z;
  if (e < 0 || (slot >= 0 && lite_stopped(B, e, slot))) return;   // padding item, or an env that has stopped
  const int v0 = B.voff[e];
  const int n = B.voff[e + 1] - v0;
  const int ld = B.gld[e];
  const int nrows = ROWS ? B.ccount[e] : n;
  const int R = split_rows(split_cover(n, B.cap));
  const int r0 = split * R;
  if (r0 >= nrows) return;   // the merge reads only the splits that hold rows
  const int r1 = min(r0 + R, nrows);
  const T* G = B.G + B.goff[e];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int col0 = tile0 + lane * VW;
  T acc[VW][3];
  for (int q = 0; q < VW; ++q) acc[q][0] = acc[q][1] = acc[q][2] = 0;
  // the split's rows in chunks of kSplitRows staged in LDS, summed in row order per wave
  for (int c0 = r0; c0 < r1; c0 += kSplitRows) {
  const int nr = min(kSplitRows, r1 - c0);
  __syncthreads();
  for (int r = threadIdx.x; r < nr; r += kBlock) {
    f4_t f;
    if (ROWS) {
      const size_t j = (size_t)e * B.cap + c0 + r;
      s_row[r] = B.cvert[j];
      f[0] = force[3 * j]; f[1] = force[3 * j + 1]; f[2] = force[3 * j + 2];
    } else {
      s_row[r] = c0 + r;
      f[0] = B.b[v0 + c0 + r]; f[1] = B.b[B.NV + v0 + c0 + r]; f[2] = B.b[2 * B.NV + v0 + c0 + r];
    }
    f[3] = 0;
    s_vec[r] = f;
  }
  __syncthreads();
  if (col0 < ld) {   // ld is a multiple of 32 columns: a lane's VW columns lie inside the row
    // Row indices are the same over the wave (scalar registers): the UNROLL loads go out
    // together, and the next UNROLL rows' loads before this iteration's FMAs (double buffer);
    // rows past the staged ones load the last staged row, unused.
    const int wsc = __builtin_amdgcn_readfirstlane(wid);
    auto load_rows = [&](int rb, vec_t* g) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const int q = __builtin_amdgcn_readfirstlane(s_row[min(rb + WS * u, nr - 1)]);
        g[u] = __builtin_nontemporal_load(reinterpret_cast<const vec_t*>(G + (size_t)q * ld + col0));
      }
    };
    vec_t gn[UNROLL];
    if (wsc < nr) load_rows(wsc, gn);
    for (int rb = wsc; rb < nr; rb += WS * UNROLL) {
      vec_t g[UNROLL];
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) g[u] = gn[u];
      if (rb + WS * UNROLL < nr) load_rows(rb + WS * UNROLL, gn);
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const int r = rb + WS * u;
        if (r < nr) {
          const f4_t b = s_vec[r];
#pragma unroll
          for (int q = 0; q < VW; ++q) {
            acc[q][0] += g[u][q] * b[0];
            acc[q][1] += g[u][q] * b[1];
            acc[q][2] += g[u][q] * b[2];
          }
        }
      }
    }
  }
  }
  // fixed-order reduction over the waves
  if (wid > 0)
    for (int q = 0; q < VW; ++q)
      for (int k = 0; k < 3; ++k) s_red[((wid - 1) * 3 + k) * TILE + lane * VW + q] = acc[q][k];
  __syncthreads();
  if (wid == 0) {
    T* P = partial + poff[e];
    for (int q = 0; q < VW; ++q) {
      const int col = col0 + q;
      if (col >= n) continue;
      for (int k = 0; k < 3; ++k) {
        T s = acc[q][k];
        for (int w = 0; w < WS - 1; ++w) s += s_red[(w * 3 + k) * TILE + lane * VW + q];
        P[((size_t)split * 3 + k) * n + col] = s;
      }
    }
  }
}

// k_gemv_split for a chunk of up to kTwinChunk envs that share one inverse.  A lane's inverse row
// vector, loaded once, serves every env of the chunk that reads that row at that position of the
// split: all of them in the apply, and in the position update wherever their contact rows
// coincide (identical envs in identical states); where they differ, each env loads its own row.
// Rows are staged kTwinRows at a time, a multiple of the wave count, so every row stays on the wave
// k_gemv_split gives it; with its per-wave row order and its fixed-order reduction over the waves,
// every env gets the bits it gets from k_gemv_split.  Loads are ordinary (cached): the other chunks
// of a group read the same rows on the same XCD close in time.  166-180 VGPRs (3 waves per SIMD in
// FP32, 2 in FP64).
constexpr int kTwinRows = 128;
template <class T, bool ROWS>
__device__ __forceinline__ void twins_vector(const DevBatch<T>& B, const int* envs, int w, int tile0, int split,
                                             const T* force, int slot, T* partial, const int64_t* poff) {
  constexpr int VW = (int)(16 / sizeof(T));
  constexpr int TILE = 64 * VW;
  constexpr int UNROLL = 4;
  constexpr int WS = kBlock / 64;
  constexpr int EB = kTwinChunk;
  constexpr int SR = kTwinRows;
  static_assert(kSplitRows % SR == 0 && SR % (WS * UNROLL) == 0, "staging must keep every row on its wave");
  static_assert(UNROLL == 4, "a wave reads its rows' shared indices as one int4");
  static_assert(EB % 4 == 0, "right-hand sides are read 4 envs at a time");
  // s_one holds row r at perm_row(r): a wave's UNROLL rows rb + WS * u (rb = wave + WS * UNROLL * k)
  // lie side by side from perm_row(rb) on
  auto perm_row = [](int r) { return r / (WS * UNROLL) * (WS * UNROLL) + r % WS * UNROLL + r / WS % UNROLL; };
  typedef T vec_t __attribute__((ext_vector_type(VW)));
  typedef T f4_t __attribute__((ext_vector_type(4)));
  __shared__ f4_t s_vec[SR * EB];   // [row][env] the env's right-hand side at this position, 0 if none
  __shared__ int s_row[SR * EB];    // [row][env] inverse row the env reads at this position, -1 if none
  __shared__ __align__(16) int s_one[SR];   // the row every reading env reads (rows permuted, below)
  __shared__ int s_mixed;           // some position has envs reading different rows
  __shared__ T s_red[(WS - 1) * 3 * TILE];
  __shared__ int s_e[EB], s_r1[EB];
  __syncthreads();   // the LDS may still be read for the workgroup's previous envs
  const int e0 = envs[0];
  const int n = B.voff[e0 + 1] - B.voff[e0];   // the same mesh, inverse and split size for the chunk
  const int ld = B.gld[e0];
  const int R = split_rows(split_cover(n, B.cap));
  const int r0 = split * R;
  if (threadIdx.x < EB) {
    int e = -1, r1 = r0;
    if ((int)threadIdx.x < w) {
      e = envs[threadIdx.x];
      const int nrows = ROWS ? B.ccount[e] : n;
      if (!(slot >= 0 && lite_stopped(B, e, slot)) && r0 < nrows) r1 = min(r0 + R, nrows);
    }
    s_e[threadIdx.x] = e;
    s_r1[threadIdx.x] = r1;
  }
  __syncthreads();
  int r1m = r0;
  for (int t = 0; t < EB; ++t) r1m = max(r1m, s_r1[t]);
  if (r1m == r0) return;   // no env of the chunk reads rows in this split (uniform over the block)
  const T* G = B.G + B.goff[e0];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int col0 = tile0 + lane * VW;
  T acc[EB][VW][3];
#pragma unroll
  for (int t = 0; t < EB; ++t)
#pragma unroll
    for (int q = 0; q < VW; ++q) acc[t][q][0] = acc[t][q][1] = acc[t][q][2] = 0;
  for (int c0 = r0; c0 < r1m; c0 += SR) {
    const int nrm = min(SR, r1m - c0);
    __syncthreads();
    if (threadIdx.x == 0) s_mixed = 0;
    // all SR x EB slots are written: an env that reads no row at a position (past its rows, past
    // the chunk's envs) gets row -1 and a zero right-hand side
    for (int idx = threadIdx.x; idx < SR * EB; idx += kBlock) {
      const int r = idx / EB, t = idx - r * EB;
      const int e = s_e[t];
      int row = -1;
      f4_t f = {0, 0, 0, 0};
      if (e >= 0 && r < nrm && c0 + r < s_r1[t]) {
        if (ROWS) {
          const size_t j = (size_t)e * B.cap + c0 + r;
          row = B.cvert[j];
          f[0] = force[3 * j]; f[1] = force[3 * j + 1]; f[2] = force[3 * j + 2];
        } else {
          const int vb = B.voff[e] + c0 + r;
          row = c0 + r;
          f[0] = B.b[vb]; f[1] = B.b[B.NV + vb]; f[2] = B.b[2 * B.NV + vb];
        }
      }
      s_row[idx] = row;
      s_vec[idx] = f;
    }
    __syncthreads();
    // the row every env that reads at this position reads (row 0 where none does); s_mixed is set
    // where envs read different rows
    for (int r = threadIdx.x; r < SR; r += kBlock) {
      int one = -1;
      bool same = true;
      for (int t = 0; t < EB; ++t) {
        const int q = s_row[r * EB + t];
        if (q < 0) continue;
        if (one < 0) one = q;
        else if (q != one) same = false;
      }
      s_one[perm_row(r)] = one < 0 ? 0 : one;
      if (!same) s_mixed = 1;
    }
    __syncthreads();
    // One pass with one load per row for the whole chunk, or, where the envs read different rows
    // somewhere in these rows, one pass per env over its own rows (its row indices written to
    // s_one first, a scalar env mask selecting its sums).
    const bool mixed = __builtin_amdgcn_readfirstlane(s_mixed) != 0;   // the same over the block
    const int npass = mixed ? w : 1;
    const int wsc = __builtin_amdgcn_readfirstlane(wid);
    for (int p = 0; p < npass; ++p) {
      if (mixed) {
        __syncthreads();
        for (int r = threadIdx.x; r < SR; r += kBlock) {
          const int q = s_row[r * EB + p];
          s_one[perm_row(r)] = q < 0 ? 0 : q;
        }
        __syncthreads();
      }
      const unsigned mask = mixed ? (1u << p) : ((1u << w) - 1u);
      if (col0 < ld) {   // ld is a multiple of 32 columns: a lane's VW columns lie inside the row
        // Row indices are the same over the wave (scalar registers), so the UNROLL loads go out
        // together, and the next UNROLL rows' loads go out before this iteration's FMAs (double
        // buffer).  An env's sum takes g * b at every row of the wave; where it reads nothing b
        // is zero and g * 0 leaves the sum as it is (the sums start at +0 and the inverse is
        // finite), so each env adds exactly its own rows in k_gemv_split's order.  The rows
        // rb + WS * u stay below SR (SR is a multiple of WS * UNROLL).
        auto load_rows = [&](int rb, vec_t* g) {
          const int4 o4 = *reinterpret_cast<const int4*>(s_one + perm_row(rb));
          const int ones[4] = {o4.x, o4.y, o4.z, o4.w};
#pragma unroll
          for (int u = 0; u < UNROLL; ++u)
            g[u] = *reinterpret_cast<const vec_t*>(G + (size_t)__builtin_amdgcn_readfirstlane(ones[u]) * ld + col0);
        };
        vec_t gn[UNROLL];
        if (wsc < nrm) load_rows(wsc, gn);
        for (int rb = wsc; rb < nrm; rb += WS * UNROLL) {
          vec_t g[UNROLL];
#pragma unroll
          for (int u = 0; u < UNROLL; ++u) g[u] = gn[u];
          if (rb + WS * UNROLL < nrm) load_rows(rb + WS * UNROLL, gn);
#pragma unroll
          for (int u = 0; u < UNROLL; ++u) {
            // right-hand sides read 4 envs at a time (one LDS wait per 4 envs); 4 x 4 values live
#pragma unroll
            for (int t0 = 0; t0 < EB; t0 += 4) {
              if (!((mask >> t0) & 0xFu)) continue;   // none of these 4 envs takes the row
              f4_t bb[4];
#pragma unroll
              for (int i = 0; i < 4; ++i) bb[i] = s_vec[(rb + WS * u) * EB + t0 + i];
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                if (!((mask >> (t0 + i)) & 1u)) continue;
#pragma unroll
                for (int q = 0; q < VW; ++q) {
                  acc[t0 + i][q][0] += g[u][q] * bb[i][0];
                  acc[t0 + i][q][1] += g[u][q] * bb[i][1];
                  acc[t0 + i][q][2] += g[u][q] * bb[i][2];
                }
              }
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
      }
    }
  }
  // per env, k_gemv_split's fixed-order reduction over the waves
#pragma unroll
  for (int t = 0; t < EB; ++t) {
    const int e = s_e[t];
    if (e < 0 || s_r1[t] <= r0) continue;   // uniform over the block
    __syncthreads();
    if (wid > 0)
      for (int q = 0; q < VW; ++q)
        for (int k = 0; k < 3; ++k) s_red[((wid - 1) * 3 + k) * TILE + lane * VW + q] = acc[t][q][k];
    __syncthreads();
    if (wid == 0) {
      T* P = partial + poff[e];
      for (int q = 0; q < VW; ++q) {
        const int col = col0 + q;
        if (col >= n) continue;
        for (int k = 0; k < 3; ++k) {
          T s = acc[t][q][k];
          for (int w2 = 0; w2 < WS - 1; ++w2) s += s_red[(w2 * 3 + k) * TILE + lane * VW + q];
          P[((size_t)split * 3 + k) * n + col] = s;
        }
      }
    }
  }
}

template <class T, bool ROWS>
__global__ void __launch_bounds__(kBlock) k_gemv_split_twins(DevBatch<T> B, const int4* items, const int* envs,
                                                             const T* force, int slot, T* partial, const int64_t* poff) {
  const int4 item = items[blockIdx.x];
  if (item.w > 0) twins_vector<T, ROWS>(B, envs + item.x, item.w, item.y, item.z, force, slot, partial, poff);
}

// The FP32 products of a chunk of up to kWideChunk envs on the matrix cores: NT tiles of 16 columns hold the
// chunk's 3 right-hand sides per env, the left operand is the inverse (16 of its columns, 4 of a wave's rows per
// instruction).  v_mfma_f32_16x16x4_f32 adds its four products as a chain of FMAs in row order, and a wave takes
// its rows in k_gemv_split's order, so every env gets k_gemv_split's bits.  Bound by the matrix cores (140 TFLOP/s
// measured for this instruction; a wave's inverse rows are loaded three steps ahead, the next block's right-hand
// sides during the products): 256 sheets of 4096 vertices 330 us a product, 25 of a workgroup's 39 us in the
// products, the rest before the first and in the sum over the waves; the vector form took 456 us.
// Where the envs of a chunk read different rows somewhere in the split, the vector form takes the whole split.
typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int kWideTile = 256;                              // columns of a workgroup
constexpr int kWideRows = 128;                              // rows staged at a time
constexpr int kWideRed = 65;                                // padded rows of the reduction area
constexpr int wide_stride(int nt) { return 16 * nt + 4; }   // a wave's rows, 4 apart, fall on different banks
constexpr size_t wide_smem(int nt) {
  const int rhs = 2 * kWideRows * wide_stride(nt), red = kBlock / 64 * kWideTile / 16 * 4 * kWideRed;
  return sizeof(float) * (rhs > red ? rhs : red);
}
template <bool ROWS, int NT>
__global__ void __launch_bounds__(kBlock) k_gemv_split_wide(DevBatch<float> B, const int4* items, const int* envs,
                                                            const float* force, int slot, float* partial,
                                                            const int64_t* poff) {
  constexpr int WS = kBlock / 64, SR = kWideRows, TILE = kWideTile;
  constexpr int BS = wide_stride(NT);
  constexpr int CT = TILE / 16;     // column tiles of a wave
  constexpr int RS = kWideRed;
  constexpr int NB = 4;             // steps whose inverse rows are in flight or in use
  constexpr int EB = kWideChunk * SR / kBlock;   // envs whose right-hand side a thread stages, one row each
  static_assert(SR % (4 * WS * NB) == 0 && kBlock % SR == 0, "staging and steps cover whole blocks");
  extern __shared__ __align__(16) float s_buf[];   // two blocks of right-hand sides [row][BS], then the reduction
  __shared__ int s_one[2][SR];                     // and the rows they multiply
  __shared__ int s_mixed;
  __shared__ int s_e[kWideChunk], s_r1[kWideChunk];
  __shared__ int64_t s_off[kWideChunk];
  const int4 item = items[blockIdx.x];
  const int w = item.w, tile0 = item.y, split = item.z;
  if (w <= 0) return;   // padding item
  const int* chunk = envs + item.x;
  const int e0 = chunk[0];
  const int n = B.voff[e0 + 1] - B.voff[e0];   // the same mesh, inverse and split size for the chunk
  const int ld = B.gld[e0];
  const int R = split_rows(split_cover(n, B.cap));
  const int r0 = split * R;
  const int tid = threadIdx.x;
  if (tid < kWideChunk) {
    const int e = chunk[min(tid, w - 1)];
    int r1 = r0;
    if (tid < w) {
      const int nrows = ROWS ? B.ccount[e] : n;
      if (!(slot >= 0 && lite_stopped(B, e, slot)) && r0 < nrows) r1 = min(r0 + R, nrows);
    }
    s_e[tid] = e;
    s_r1[tid] = r1;
    s_off[tid] = poff[e] + (int64_t)split * 3 * n;
  }
  if (tid == 0) s_mixed = 0;
  for (int r = tid; r < 2 * SR; r += kBlock)   // columns past the chunk's stay zero
    for (int q = 3 * w; q < 16 * NT; ++q) s_buf[r * BS + q] = 0.f;
  __syncthreads();
  int r1m = r0, el = e0;   // the most rows an env of the chunk reads, and such an env
  for (int t = 0; t < w; ++t)
    if (s_r1[t] > r1m) { r1m = s_r1[t]; el = s_e[t]; }
  if (r1m == r0) return;   // no env of the chunk reads rows in this split (uniform over the block)
  if (ROWS) {
    // does every env that reads at a position read that env's row?
    bool same = true;
    for (int p = r0 + tid; p < r1m; p += kBlock) {
      const int one = B.cvert[(size_t)el * B.cap + p];
#pragma unroll
      for (int t = 0; t < kWideChunk; ++t)   // (past the chunk: its last env, reading nothing)
        same &= (B.cvert[(size_t)s_e[t] * B.cap + min(p, max(s_r1[t] - 1, 0))] == one) | (p >= s_r1[t]);
    }
    if (!same) s_mixed = 1;
    __syncthreads();
    if (s_mixed) {
      for (int t = 0; t < w; t += kTwinChunk)
        twins_vector<float, ROWS>(B, chunk + t, min(kTwinChunk, w - t), tile0, split, force, slot, partial, poff);
      return;
    }
  }
  const float* G = B.G + B.goff[e0];
  const int l = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lm = l & 15, lk = l >> 4;
  const float* Gl[4];   // this lane's four columns of each 64 (past the row: its last four, not stored)
#pragma unroll
  for (int c = 0; c < 4; ++c) Gl[c] = G + min(tile0 + 64 * c + 4 * lm, ld - 4);
  // a block's right-hand sides and rows: to registers, and from there to LDS once the block before is done
  const int sr = tid % SR, st = tid / SR * EB;
  float f[EB][3];
  int one = 0;
  auto fetch = [&](int c0) {
    const int p = c0 + sr;
    if (ROWS) one = B.cvert[(size_t)el * B.cap + min(p, r1m - 1)];
    else one = min(p, r1m - 1);
#pragma unroll
    for (int i = 0; i < EB; ++i) {
      const int e = s_e[st + i], q = min(p, max(s_r1[st + i] - 1, 0));
#pragma unroll
      for (int k = 0; k < 3; ++k)
        f[i][k] = ROWS ? force[3 * ((size_t)e * B.cap + q) + k] : B.b[(size_t)k * B.NV + B.voff[e] + q];
    }
  };
  auto stage = [&](int c0, int buf) {
    if (tid < SR) s_one[buf][sr] = one;
#pragma unroll
    for (int i = 0; i < EB; ++i)
      if (st + i < w) {
        const bool reads = c0 + sr < s_r1[st + i];
#pragma unroll
        for (int k = 0; k < 3; ++k) s_buf[(buf * SR + sr) * BS + 3 * (st + i) + k] = reads ? f[i][k] : 0.f;
      }
  };
  floatx4 acc[CT][NT];
#pragma unroll
  for (int c = 0; c < CT; ++c)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[c][t] = floatx4{};
  const int rl = wave + WS * lk;   // this lane's row of a step
  fetch(r0);
  for (int c0 = r0, buf = 0; c0 < r1m; c0 += SR, buf ^= 1) {
    stage(c0, buf);
    __syncthreads();
    if (c0 + SR < r1m) fetch(c0 + SR);
    __builtin_amdgcn_sched_barrier(0);
    // whole rounds of NB steps: rows past the last have zero right-hand sides
    const int steps = (min(SR, r1m - c0) + 4 * WS * NB - 1) / (4 * WS * NB) * NB;
    const int* rows = s_one[buf] + rl;
    const float* rhs = s_buf + (buf * SR + rl) * BS + lm;
    auto load = [&](int i, floatx4 (&a)[4]) {
      const size_t o = (size_t)rows[min(i, steps - 1) * 4 * WS] * ld;
#pragma unroll
      for (int c = 0; c < 4; ++c) a[c] = *reinterpret_cast<const floatx4*>(Gl[c] + o);
    };
    floatx4 an[NB][4];
#pragma unroll
    for (int p = 0; p < NB; ++p) {
      load(p, an[p]);
      __builtin_amdgcn_sched_barrier(0);   // in the order of their use, so that the first wait is for the first only
    }
#pragma unroll 1
    for (int i = 0; i < steps; i += NB)
#pragma unroll
      for (int p = 0; p < NB; ++p) {
        float b[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) b[t] = rhs[(i + p) * 4 * WS * BS + 16 * t];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int t = 0; t < NT; ++t)
              acc[4 * c + q][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(an[p][c][q], b[t], acc[4 * c + q][t], 0, 0, 0);
        load(i + p + NB, an[p]);
        __builtin_amdgcn_sched_barrier(0);   // the loads stay NB - 1 steps ahead of their use
      }
  }
  // k_gemv_split's fixed-order sum over the waves, one tile of right-hand sides at a time.  Tile 4 c + q,
  // register r, lane lm + 16 g hold column 64 c + 16 g + 4 r + q of right-hand side lm.
  const int at = ((l & 3) * 4 + ((l >> 2) & 3)) * RS + 16 * (l >> 4);
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_buf[((wave * CT + c) * 4 + r) * RS + l] = acc[c][t][r];
    __syncthreads();
#pragma unroll 1
    for (int j = wave; j < 16; j += WS) {   // a right-hand side per wave and turn
      const int en = (16 * t + j) / 3, k = 16 * t + j - 3 * en;
      if (en >= w || s_r1[en] <= r0) continue;
      float* P = partial + s_off[en] + (int64_t)k * n + tile0 + l;
      float v[4][WS];
#pragma unroll
      for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int u = 0; u < WS; ++u) v[c][u] = s_buf[(u * CT + 4 * c) * 4 * RS + at + j];
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (tile0 + 64 * c + l < n) P[64 * c] = ((v[c][0] + v[c][1]) + v[c][2]) + v[c][3];
    }
  }
}

// Adds each env's row-split partials in split order: z = sum.
template <class T>
__global__ void __launch_bounds__(kBlock) k_gemv_merge(DevBatch<T> B, const T* partial, const int64_t* poff) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= B.NV) return;
  const int e = B.vert_env[i];
  const int v0 = B.voff[e];
  const int n = B.voff[e + 1] - v0;
  T s[3];
  split_sum(partial + poff[e], split_count(B, n, n), n, i - v0, s);
  for (int k = 0; k < 3; ++k) B.z[(size_t)k * B.NV + i] = s[k];
}

template <class T, bool ROWS>
void launch_split_product(const DevBatch<T>& B, const SplitSchedule& S, const T* force, int slot, hipStream_t s) {
  T* P = static_cast<T*>(S.partial);
  if (S.n_items > 0) {
    const dim3 g((unsigned)S.n_items), blk(kBlock);
    constexpr int V16 = (int)(16 / sizeof(T)), V8 = (int)(8 / sizeof(T));
    if (S.vw == V16)
      hipLaunchKernelGGL((k_gemv_split<T, ROWS, V16, 8>), g, blk, 0, s, B, S.items, force, slot, P, S.poff);
    else if (S.vw == V8)
      hipLaunchKernelGGL((k_gemv_split<T, ROWS, V8, 16>), g, blk, 0, s, B, S.items, force, slot, P, S.poff);
    else
      hipLaunchKernelGGL((k_gemv_split<T, ROWS, 1, 16>), g, blk, 0, s, B, S.items, force, slot, P, S.poff);
  }
  if (S.n_twin_items > 0) {
    const dim3 g((unsigned)S.n_twin_items), blk(kBlock);
    if constexpr (std::is_same<T, float>::value) {
      auto go = [&](auto kernel, int nt) {
        hipLaunchKernelGGL(kernel, g, blk, wide_smem(nt), s, B, S.twin_items, S.twin_envs, force, slot, P, S.poff);
      };
      if (3 * S.max_chunk <= 16) go(k_gemv_split_wide<ROWS, 1>, 1);
      else if (3 * S.max_chunk <= 32) go(k_gemv_split_wide<ROWS, 2>, 2);
      else go(k_gemv_split_wide<ROWS, 3>, 3);
    } else {
      hipLaunchKernelGGL((k_gemv_split_twins<T, ROWS>), g, blk, 0, s, B, S.twin_items, S.twin_envs, force, slot, P,
                         S.poff);
    }
  }
}

}  // namespace

hipError_t prepare_lite() {
  const std::pair<const void*, int> kernels[] = {
      {(const void*)k_gemv_split_wide<false, 1>, 1}, {(const void*)k_gemv_split_wide<true, 1>, 1},
      {(const void*)k_gemv_split_wide<false, 2>, 2}, {(const void*)k_gemv_split_wide<true, 2>, 2},
      {(const void*)k_gemv_split_wide<false, 3>, 3}, {(const void*)k_gemv_split_wide<true, 3>, 3}};
  hipError_t st = hipSuccess;
  for (const auto& k : kernels) {
    const hipError_t e = hipFuncSetAttribute(k.first, hipFuncAttributeMaxDynamicSharedMemorySize, (int)wide_smem(k.second));
    if (st == hipSuccess) st = e;
  }
  return st;
}

template <class T>
void launch_split_apply(const DevBatch<T>& B, const SplitSchedule& S, hipStream_t s) {
  launch_split_product<T, false>(B, S, nullptr, -1, s);
  hipLaunchKernelGGL(k_gemv_merge<T>, dim3((unsigned)((B.NV + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, B,
                     (const T*)S.partial, S.poff);
}

template <class T>
void launch_split_correct(const DevBatch<T>& B, const SplitSchedule& S, int k, int it, hipStream_t s) {
  launch_split_product<T, true>(B, S, it & 1 ? B.lite_force : B.cforce, it > 0 ? k * (B.max_newton + 1) + it - 1 : -1, s);
}

template <class T>
void launch_lite_prepare(const DevBatch<T>& B, hipStream_t s) {
  const dim3 g((unsigned)((B.cap + kBlock - 1) / kBlock), (unsigned)B.n_envs), blk(kBlock);
  if (B.csp64) hipLaunchKernelGGL((k_lite_prepare<T, double>), g, blk, 0, s, B);
  else hipLaunchKernelGGL((k_lite_prepare<T, T>), g, blk, 0, s, B);
}

template <class T>
void launch_lite_update(const DevBatch<T>& B, const SplitSchedule& S, const T* mu_env, int k, int it, hipStream_t s) {
  const dim3 g((unsigned)((B.cap + kBlock - 1) / kBlock), (unsigned)B.n_envs), blk(kBlock);
  const int slot = k * (B.max_newton + 1) + it;
  const T* P = static_cast<const T*>(S.partial);
  if (B.csp64) hipLaunchKernelGGL((k_lite_update<T, double>), g, blk, 0, s, B, mu_env, slot, it, P, S.poff);
  else hipLaunchKernelGGL((k_lite_update<T, T>), g, blk, 0, s, B, mu_env, slot, it, P, S.poff);
}

template <class T>
void launch_lite_end(const DevBatch<T>& B, const SplitSchedule& S, int k, hipStream_t s) {
  const int most = S.max_n > B.cap ? S.max_n : B.cap;
  hipLaunchKernelGGL(k_lite_end<T>, dim3((unsigned)((most + kBlock - 1) / kBlock), (unsigned)B.n_envs), dim3(kBlock), 0,
                     s, B, k * (B.max_newton + 1), k == 0 ? 1 : 0, (const T*)S.partial, S.poff);
}

#define FLASH_LITE(T)                                                                                              \
  template void launch_split_apply<T>(const DevBatch<T>&, const SplitSchedule&, hipStream_t);                      \
  template void launch_split_correct<T>(const DevBatch<T>&, const SplitSchedule&, int, int, hipStream_t);          \
  template void launch_lite_prepare<T>(const DevBatch<T>&, hipStream_t);                                           \
  template void launch_lite_update<T>(const DevBatch<T>&, const SplitSchedule&, const T*, int, int, hipStream_t);  \
  template void launch_lite_end<T>(const DevBatch<T>&, const SplitSchedule&, int, hipStream_t);
FLASH_LITE(float)
FLASH_LITE(double)
#undef FLASH_LITE

}  // namespace flash
