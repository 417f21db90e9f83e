// Single-workgroup ReLU-QP kernel for small problems (n + m <= 128): every iteration, check and
// penalty switch of Algorithm 1 (online stage) in one launch of one workgroup.
//
// The iteration is the compact layer of the persistent kernel (Sec. III-A with OSQP
// over-relaxation): w = [sigma x - q ; rho z - y], one product with
// Wc_j = [D_j, D_j A'; A D_j, A D_j A'] gives xt and A xt, and the relaxation, the clamp
// (eq. clamp) and the dual update are row-local. At these sizes an iteration is a few hundred
// multiply-adds, so its time is set by latency, not by bandwidth: a persistent grid would spend
// it on the cross-workgroup exchange of w. Here Wc_j lives in registers for the whole solve
// (reloaded when the penalty changes), w is exchanged through LDS, and one workgroup barrier per
// iteration is the only synchronisation.
//
// Layout: row r of Wc_j is split over S = 8 consecutive lanes; lane s of the row holds and multiplies
// the columns (i S + s) V .. + V - 1 (V entries: 16 bytes), i < NI, and DPP lane moves sum the S partials,
// leaving the row's value in all S lanes. Waves that hold no row skip the product. Bound by the chain of
// one LDS round trip, the sums, the update and the barrier for the smallest, and by the bytes LDS returns
// (L^2 values per iteration at 128 bytes per clock) for the largest: 0.26 / 0.28 / 0.34 / 0.45 us per FP64
// iteration at 38 / 60 / 90 / 126 rows (0.30 / 0.30 / 0.47 / 0.77 with one 8-byte read per column and a
// single chain), 0.23 / 0.24 / 0.28 / 0.31 in FP32 (0.23 / 0.25 / 0.32 / 0.43). One lane per row, a wave
// that iterates alone with w broadcast, took 0.27 us at 38 FP64 rows and 0.44 at 60, and its checks twice
// as long.
//
// Every check_interval iterations (Sec. III-C) the rows of [P, A'; A, 0] [x; y] (P x + A'y and
// A x) are formed with FP64 accumulation from the check matrix, held in LDS for the whole
// launch, and the seven inf-norms are reduced as ordered bit patterns (exact and
// NaN-propagating). The stopping test (eqs. primal, dual) and
// the penalty rule (eq. rho_update, nearest grid value) are those of the persistent kernel.
#include "small_kernel.h"

#include "device_common.h"

namespace rqp {
namespace {

constexpr int SB = kSmallBlock;
constexpr int SWAVES = SB / kWave;
constexpr int S = 8;  // lanes per row
constexpr int kRhoMax = 64;  // the host accepts at most 64 penalty values

enum { S_RUNNING = 0, S_SOLVED = 1, S_MAX_ITER = 2, S_NONFINITE = 3, S_ABORTED = 4 };
enum { K_RP = 0, K_RD, K_AX, K_Z, K_PX, K_ATY, K_Q, K_NORMS };

// 16-byte vectors of the layer input and the rows.
template <typename T>
struct Vec;
template <>
struct Vec<float> {
  static constexpr int V = 4;
  typedef float4 type;
};
template <>
struct Vec<double> {
  static constexpr int V = 2;
  typedef double2 type;
};
template <typename T>
__device__ __forceinline__ void load_vec(const T* p, T (&v)[Vec<T>::V]) {
  const typename Vec<T>::type t = *reinterpret_cast<const typename Vec<T>::type*>(p);
  v[0] = t.x;
  v[1] = t.y;
  if constexpr (Vec<T>::V == 4) {
    v[2] = t.z;
    v[3] = t.w;
  }
}
// Sum of the products of NI vectors of a row with vectors (i S + s) of w, in two chains.
template <typename T, int NI>
__device__ __forceinline__ T row_product(const T (&wst)[NI][Vec<T>::V], const T* w, int s) {
  constexpr int V = Vec<T>::V;
  T acc[2] = {(T)0, (T)0};
  T x[NI][V];
#pragma unroll
  for (int i = 0; i < NI; ++i) load_vec(w + (i * S + s) * V, x[i]);
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int e = 0; e < V; ++e) acc[(i * V + e) & 1] = fma(wst[i][e], x[i][e], acc[(i * V + e) & 1]);
  return acc[0] + acc[1];
}

// Sum over the 8 lanes of a row (consecutive and aligned) with DPP lane moves (VALU, no LDS round
// trip): swaps of neighbours and of pairs within a quad, then the half-row mirror. Every lane of the
// row ends with the same sum (each step adds the same two partial sums, in either order).
template <typename T>
__device__ __forceinline__ T row_sum(T v) {
  v = dpp_add<0xb1, 0xf>(v);          // quad_perm [1,0,3,2]
  v = dpp_add<0x4e, 0xf>(v);          // quad_perm [2,3,0,1]
  return dpp_add<0x141, 0xf>(v);      // row_half_mirror
}

// This lane's vectors of row r of a matrix of ldw columns (a multiple of 4, zero past L): zero for rows
// or columns past L.
template <typename T, int NI>
__device__ __forceinline__ void load_row(const T* M, const LayerArgs& a, bool row, int r, int s,
                                         T (&w)[NI][Vec<T>::V]) {
  constexpr int V = Vec<T>::V;
  const T* const p = M + (long)(row ? r : 0) * a.ldw;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = (i * S + s) * V;
    if (row && c < a.L) {
      load_vec(p + c, w[i]);
    } else {
#pragma unroll
      for (int e = 0; e < V; ++e) w[i][e] = (T)0;
    }
  }
}

// Products of this lane's part of its row of the check matrix with cv over its columns below cend,
// FP64, split at column n (the P or A part and the A' part), accumulated in ascending column order,
// with the sums of their absolute values (alo, ahi: the rounding bound of the check); columns out of
// range contribute zero.
template <typename T, int NI>
__device__ __forceinline__ void check_products(const LayerArgs& a, const T* Cl, int NT, int s, int cend, const T* cv,
                                               double& lo, double& hi, double& alo, double& ahi) {
  constexpr int V = Vec<T>::V;
  lo = 0.0;
  hi = 0.0;
  alo = 0.0;
  ahi = 0.0;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    T cval[V], xval[V];
    load_vec(Cl + (i * NT + threadIdx.x) * V, cval);
    load_vec(cv + (i * S + s) * V, xval);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      const int c = (i * S + s) * V + e;
      const double v = c < cend ? (double)cval[e] * (double)xval[e] : 0.0;
      if (c < a.n) {
        lo += v;
        alo += fabs(v);
      } else {
        hi += v;
        ahi += fabs(v);
      }
    }
  }
}

template <typename T, int NI>
__global__ void __launch_bounds__(SB) small_kernel(LayerArgs a) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  T* Cl = reinterpret_cast<T*>(dyn_lds);  // the check matrix, NI * NT * V entries
  __shared__ __align__(16) T wb[2][kSmallRows];  // layer input w, two parities
  __shared__ __align__(16) T cv[kSmallRows];     // [x; y] for the check and z = A x of a warm start
  __shared__ T upd[kSmallRows][2];  // q, l, u from an initial state
  __shared__ uint64_t nrm[SWAVES][8];  // the waves' norm maxima
  __shared__ double grid_s[kRhoMax], mid_s[kRhoMax];

  const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n = a.n, L = a.L;
  const int r = tid / S, s = tid - r * S;  // this lane's row and column lane
  const bool wave_rows = wave * (kWave / S) < L;  // the wave holds at least one row
  const int NT = (L * S + kWave - 1) / kWave * kWave;  // threads of the waves that hold rows
  const bool row = r < L, own = row && s == 0, xrow = r < n;
  const bool seq = row && !xrow && a.eq[r - n] != 0;

  if (tid < a.n_rho) grid_s[tid] = a.grid[tid];
  if (tid < a.n_rho - 1) mid_s[tid] = a.mid[tid];
  // entries past L are read as columns of the zero padding; keep them finite
  if (tid < kSmallRows && tid >= L) wb[0][tid] = wb[1][tid] = cv[tid] = (T)0;
  // the check matrix [P, A'; A, 0] straight to LDS, vector i of thread t at (i NT + t) V, in flight during
  // the first solve's update; lanes without a row and vectors past the last column copy other entries,
  // which no sum takes
  if (wave * kWave < NT) {
    const T* const Cr = static_cast<const T*>(a.C) + (long)(row ? r : 0) * a.ldw;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = (i * S + s) * Vec<T>::V;
      lds_copy16(Cr + (c < L ? c : 0), Cl + (i * NT + wave * kWave) * Vec<T>::V);
    }
  }

  const int ci = a.check_interval, max_iter = a.max_iter;
  const T alpha = (T)a.alpha, oma = (T)(1.0 - a.alpha), sigma = (T)a.sigma;
  // rounding bound of the check (FP32 iterations): |computed - FP64| <= kappa * sum |a_ij v_j|
  // per row, with the stored matrices and the outputs rounded to FP32 and FP64 accumulation over
  // at most L terms on both sides; an FP64 handle computes the FP64 residual itself
  const double kappa = sizeof(T) == sizeof(double) ? 0.0 : 1.01 * (2.0 * 0x1p-24 + 2.0 * (double)(L + 8) * 0x1p-53);
  const double ut = sizeof(T) == sizeof(double) ? 0.0 : 1.01 * 0x1p-24;
  // the state of row r, held by all S lanes of the row (they compute the same values); ax is
  // the last check's (A x)_r of a constraint row
  T sx = 0, sz = 0, sy = 0, sq = 0, sl = 0, su = 0;
  double ax = 0.0;
  int j = a.warm ? *a.js : a.j0;
  int held_j = -1;
  T wst[NI][Vec<T>::V];  // this lane's entries of its row of the layer matrix, for penalty held_j

  for (int sv = 0; sv < a.count; ++sv) {
    const bool warm = sv == 0 ? a.warm != 0 : a.chain != 0;
    if (!warm) j = a.j0;
    if (j != held_j) {  // in flight during the update
      load_row<T, NI>(static_cast<const T*>(a.W) + (long)j * a.w_stride, a, row, r, s, wst);
      held_j = j;
    }
    __syncthreads();  // upd[] of the previous solve has been read

    // update from an initial state (Sec. IV): q = F x0, l = lo - E x0, u = hi - E x0, FP64
    // products, one wave per row; written back to the handle's q, l, u
    if (a.x0) {
      const double* x0 = a.x0 + (long)sv * a.nx;
      // (UB rows of a wave at a time, their loads and lane sums interleaved)
      constexpr int UB = 4;
      for (int rb = wave * UB; rb < L; rb += SWAVES * UB) {
        double du[UB];
        const double* ar[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int rr = rb + u < L ? rb + u : rb;
          ar[u] = rr < n ? a.F + (long)rr * a.nx : a.E + (long)(rr - n) * a.nx;
          du[u] = 0.0;
        }
        for (int c = lane; c < a.nx; c += kWave) {
          const double xv = x0[c];
#pragma unroll
          for (int u = 0; u < UB; ++u) du[u] = fma(ar[u][c], xv, du[u]);
        }
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1)
#pragma unroll
          for (int u = 0; u < UB; ++u) du[u] += __shfl_xor(du[u], off, kWave);
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int rr = rb + u;
          if (rr >= L || lane != 0) continue;
          const double dv = du[u];
          if (rr < n) {
            upd[rr][0] = (T)dv;
            static_cast<T*>(const_cast<void*>(a.q))[rr] = (T)dv;
          } else {
            const int i = rr - n;
            upd[rr][0] = (T)(a.plo[i] - dv);
            upd[rr][1] = (T)(a.phi[i] - dv);
            static_cast<T*>(const_cast<void*>(a.l))[i] = upd[rr][0];
            static_cast<T*>(const_cast<void*>(a.u))[i] = upd[rr][1];
          }
        }
      }
    }
    __syncthreads();

    // cold start (zero state, start penalty), or warm from the handle (first solve) or from the
    // previous solve of this launch
    if (row) {
      if (xrow) {
        sq = a.x0 ? upd[r][0] : static_cast<const T*>(a.q)[r];
        if (!warm) sx = (T)0;
        else if (sv == 0) sx = static_cast<const T*>(a.xs)[r];
      } else {
        const int i = r - n;
        sl = a.x0 ? upd[r][0] : static_cast<const T*>(a.l)[i];
        su = a.x0 ? upd[r][1] : static_cast<const T*>(a.u)[i];
        if (!warm) sy = (T)0;
        else if (sv == 0) sy = static_cast<const T*>(a.ys)[i];
        ax = 0.0;
        sz = (T)0;
      }
    }
    T srho = (T)(grid_s[j] * (seq ? a.rho_eq_scale : 1.0));
    T rinv = (T)1 / srho;  // y / rho as y * (1 / rho): one rounding more, no division per iteration
    if (sv == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the check matrix, before a barrier

    // warm start (Sec. II-B): z = A x with FP64 accumulation
    if (warm) {
      if (own) cv[r] = xrow ? sx : sy;
      __syncthreads();
      double p = 0.0, unused, unused2, unused3;
      if (wave_rows) {
        check_products<T, NI>(a, Cl, NT, s, n, cv, p, unused, unused2, unused3);
        p = row_sum(p);
      }
      if (row && !xrow) {
        sz = (T)p;
        ax = p;
      }
    }
    if (own) wb[1][r] = xrow ? sigma * sx - sq : srho * sz - sy;
    __syncthreads();  // w_1

    int k = 0, nchk = 0;
    const long hoff = (long)sv * a.max_checks;
    while (true) {
      const int kend = (k / ci + 1) * ci < max_iter ? (k / ci + 1) * ci : max_iter;
      // the part of the update that does not wait for the product
      T pre = xrow ? oma * sx : fma(sy, rinv, oma * sz);
      while (k < kend) {
        ++k;
        // layer matvec: row r of Wc_j times w_k, then the row-local update
        if (wave_rows) {
          const T v = row_sum(row_product<T, NI>(wst, wb[k & 1], s));
          if (row) {
            const T t = fma(alpha, v, pre);
            T wn;
            if (xrow) {
              sx = t;
              wn = sigma * sx - sq;
            } else {
              sz = box_clamp(t, sl, su);
              sy = srho * (t - sz);
              wn = srho * sz - sy;
            }
            if (own && k < kend) wb[(k + 1) & 1][r] = wn;
            pre = xrow ? oma * sx : fma(sy, rinv, oma * sz);
          }
        }
        __syncthreads();
      }

      // check at iteration k: rows of [P, A'; A, 0] [x; y], FP64 accumulation: P x + A'y for
      // the x rows (dual side), A x for the constraint rows (primal side). In FP32 the published
      // residuals are upper bounds and the norms lower bounds of the FP64 values of a CPU
      // evaluation of the returned x, z, y with the caller's P, q, A (kappa), so SOLVED implies
      // that the FP64 test passes.
      if (own) cv[r] = xrow ? sx : sy;
      __syncthreads();
      double pr = 0.0, ar = 0.0, apr = 0.0, aar = 0.0;
      if (wave_rows) {
        check_products<T, NI>(a, Cl, NT, s, L, cv, pr, ar, apr, aar);
        pr = row_sum(pr);
        ar = row_sum(ar);
        apr = row_sum(apr);
        aar = row_sum(aar);
      }
      if (row && !xrow) ax = pr;
      // lane i of a row takes norm i (7: the host's abort flag), the wave its rows' maxima, and after one
      // barrier every wave reduces the waves' maxima and decides for itself: no broadcast
      double nv = 0.0;
      if (row) {
        // a Ruiz-scaled problem weights each row's terms so that the norms are the original
        // problem's: 1 / (c D_r) on the dual side, 1 / E_i on the primal side (1 otherwise)
        if (xrow) {
          const double qv = (double)sq, f = a.sc_dual ? a.sc_dual[r] : 1.0;
          const double dpx = kappa * apr, daty = kappa * aar, dq = ut * fabs(qv);
          if (s == K_RD) nv = f * (fabs(pr + qv + ar) + dpx + daty + dq);
          if (s == K_PX) nv = f * lower_bound(fabs(pr), dpx);
          if (s == K_ATY) nv = f * lower_bound(fabs(ar), daty);
          if (s == K_Q) nv = f * lower_bound(fabs(qv), dq);
        } else {
          const double e = a.sc_prim ? a.sc_prim[r - n] : 1.0;
          const double ds = kappa * apr, zv = (double)sz, dz = ut * fabs(zv);
          if (s == K_RP) nv = e * (fabs(pr - zv) + ds + dz);
          if (s == K_AX) nv = e * lower_bound(fabs(pr), ds);
          if (s == K_Z) nv = e * lower_bound(fabs(zv), dz);
        }
      }
      uint64_t nb = abs_bits(nv);
      if (tid == K_NORMS) {
        // the host-mapped flag costs a PCIe round trip, so it is read at every kAbortEvery-th
        // check only
        const bool ab = (nchk % kAbortEvery) == kAbortEvery - 1 && a.abort_flag &&
                        __hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
        nb = ab ? 1u : 0u;
      }
      nb = max_over_groups(nb);
      if (lane < 8) nrm[wave][lane] = nb;
      __syncthreads();
      static_assert(SWAVES == 16, "two waves' maxima per lane");
      const uint64_t m0 = nrm[lane / 8][lane % 8], m1 = nrm[8 + lane / 8][lane % 8];
      nb = max_over_groups(m0 > m1 ? m0 : m1);
      uint64_t fin[K_NORMS + 1];
      bool nonfinite = false;
#pragma unroll
      for (int i = 0; i <= K_NORMS; ++i) {
        const uint32_t flo = __builtin_amdgcn_readlane((uint32_t)nb, i);
        const uint32_t fhi = __builtin_amdgcn_readlane((uint32_t)(nb >> 32), i);
        fin[i] = (uint64_t)flo | ((uint64_t)fhi << 32);
        if (i < K_NORMS) nonfinite |= fin[i] >= kInfBits;
      }
      const double rp = bits_to_double(fin[K_RP]), rd = bits_to_double(fin[K_RD]);
      const double nax = bits_to_double(fin[K_AX]), nz = bits_to_double(fin[K_Z]);
      const double npx = bits_to_double(fin[K_PX]), naty = bits_to_double(fin[K_ATY]);
      const double nq = bits_to_double(fin[K_Q]);
      int st = S_RUNNING;
      if (nonfinite) {
        st = S_NONFINITE;
      } else if (a.terminate) {
        const double eps_p = a.eps_abs + a.eps_rel * fmax(nax, nz);
        const double eps_d = a.eps_abs + a.eps_rel * fmax(fmax(npx, naty), nq);
        if (rp <= eps_p && rd <= eps_d) st = S_SOLVED;
      }
      if (st == S_RUNNING && k == max_iter) st = S_MAX_ITER;
      if (st == S_RUNNING && fin[K_NORMS] == 1) st = S_ABORTED;
      int jn = j;
      if (st == S_RUNNING && a.n_rho > 1 && rp > 0.0 && rd > 0.0) {
        const double num = rp * fmax(fmax(npx, naty), fmax(nq, 1e-4));
        const double den = rd * fmax(fmax(nax, nz), 1e-4);
        const double rh = grid_s[j] * sqrt(num / den);
        // lane i compares with midpoint i; the midpoints rise, so the count of those below is the index
        jn = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < a.n_rho - 1 && rh > mid_s[lane]));
      }
      st = __builtin_amdgcn_readfirstlane(st);
      if (tid == 0) {
        if (a.rho_hist) a.rho_hist[hoff + nchk] = jn;
        if (a.prim_res) a.prim_res[hoff + nchk] = rp;
        if (a.dual_res) a.dual_res[hoff + nchk] = rd;
      }
      ++nchk;
      if (st != S_RUNNING) {
        if (own) {
          // the handle keeps the (scaled) iterates; the outputs are in original units
          if (xrow) {
            static_cast<T*>(a.xs)[r] = sx;
            static_cast<T*>(a.xo)[(long)sv * n + r] = a.un_x ? (T)(a.un_x[r] * (double)sx) : sx;
          } else {
            const int i = r - n;
            static_cast<T*>(a.zs)[i] = sz;
            static_cast<T*>(a.ys)[i] = sy;
            a.axs[i] = ax;
            static_cast<T*>(a.zo)[(long)sv * a.m + i] = a.sc_prim ? (T)(a.sc_prim[i] * (double)sz) : sz;
            static_cast<T*>(a.yo)[(long)sv * a.m + i] = a.un_y ? (T)(a.un_y[i] * (double)sy) : sy;
          }
        }
        if (tid == 0) {
          a.iterations[sv] = k;
          a.status[sv] = st;
          a.rho_index[sv] = j;
          *a.js = j;
        }
        break;  // next solve of the sequence
      }
      if (jn != j) {
        j = jn;
        srho = (T)(grid_s[j] * (seq ? a.rho_eq_scale : 1.0));
        rinv = (T)1 / srho;
        load_row<T, NI>(static_cast<const T*>(a.W) + (long)j * a.w_stride, a, row, r, s, wst);
        held_j = j;
      }
      if (own) wb[(k + 1) & 1][r] = xrow ? sigma * sx - sq : srho * sz - sy;
      __syncthreads();  // w_{k+1}
    }
  }
}

// NI vectors per lane reach the last column.
struct Shape {
  const void* fn;
  size_t lds;  // the check matrix: at most 128 KB (FP64, 128 rows)
};
template <typename T, int NI>
Shape shape(int L) {
  const int nt = (L * S + kWave - 1) / kWave * kWave;
  return Shape{reinterpret_cast<const void*>(&small_kernel<T, NI>), (size_t)NI * nt * 16};
}
template <typename T>
Shape shape_for(int L) {
  constexpr int C = S * Vec<T>::V;  // columns per vector of a row's lanes
  if (L <= C) return shape<T, 1>(L);
  if (L <= 2 * C) return shape<T, 2>(L);
  if (L <= 3 * C) return shape<T, 3>(L);
  if (L <= 4 * C) return shape<T, 4>(L);
  if constexpr (sizeof(T) == sizeof(double)) {
    if (L <= 5 * C) return shape<T, 5>(L);
    if (L <= 6 * C) return shape<T, 6>(L);
    if (L <= 7 * C) return shape<T, 7>(L);
    return shape<T, 8>(L);
  }
  return shape<T, 4>(L);
}

}  // namespace

template <typename T>
hipError_t prepare_small(int L) {
  if (L < 1 || L > kSmallRows) return hipErrorInvalidValue;
  const Shape sh = shape_for<T>(L);
  return hipFuncSetAttribute(sh.fn, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
}

template <typename T>
hipError_t launch_small(const LayerArgs& a, hipStream_t st) {
  if (a.L < 1 || a.L > kSmallRows || a.Ad || a.n_rho > kRhoMax) return hipErrorInvalidValue;
  const Shape sh = shape_for<T>(a.L);
  LayerArgs arg = a;
  void* args[] = {&arg};
  return hipLaunchKernel(sh.fn, dim3(1), dim3(SB), args, sh.lds, st);
}

template hipError_t prepare_small<float>(int);
template hipError_t prepare_small<double>(int);
template hipError_t launch_small<float>(const LayerArgs&, hipStream_t);
template hipError_t launch_small<double>(const LayerArgs&, hipStream_t);

}  // namespace rqp
