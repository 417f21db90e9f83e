// Persistent ReLU-QP layer kernel for gfx950: every iteration, check and penalty switch of
// Algorithm 1 (online stage) in one cooperative launch. Device code, instantiated per precision
// and variant by layer_{f32,f32x,f64,f64x}.hip.
//
// Iteration (Sec. III-A; OSQP over-relaxation alpha; alpha = 1 is the paper's layer). With
// w = [sigma x - q ; rho z - y] and the compact layer matrix
//     Wc_j = [I; A] D_j [I, A'] = [D_j, D_j A'; A D_j, A D_j A'],   D_j = (P + sigma I + A' rho_j A)^-1,
// one matvec gives both xt = D_j (sigma x - q + A'(rho z - y)) and s = A xt. Then
//     x <- alpha xt + (1 - alpha) x
//     t  = alpha s + (1 - alpha) z + y / rho,   z <- clamp(t, l, u),   y <- rho (t - z)
// are row-local, and the next w is row-local too. This is the paper's "v <- clamp(W v + b)"
// (eq. gpu_update) with an (n+m)^2 weight instead of its (n+2m)^2 one: the paper's W also
// precomputes the products of D with A.
//
// Parallel layout: workgroup g owns a contiguous block of rows of Wc (row-parallel, Sec.
// III-A). Lane t of the first col_lanes owns the columns c = t + col_lanes k of every row of the
// block and keeps the first NRS rows of its columns in registers for the whole launch (reloaded only
// when the penalty changes); further rows sit in LDS or stream from memory. After the row-local
// update each row owner publishes its entry of the next w as an 8-byte {value, tag} word; every
// lane polls the words of its own columns until the tags match. That single round trip is both
// the data exchange and the synchronisation: there is no grid barrier.
//
// What bounds it: the exchange (alone, polled at once, 1.83 us for 3200 words over 256 workgroups and 1.5 us
// for 1600 over 128; neither half the bytes per word nor wider polls shorten it, so it is latency), then the
// multiply-adds and the reduction over lanes. A whole iteration took 3.4 us at 3200 FP32 rows with
// the reduction row by row and no pause, and takes 1.77; a check took 21 us and takes 14.
//
// Every check_interval iterations (Sec. III-C) the owners publish [x; y], every workgroup
// forms its rows of [P, A'; A, 0][x; y] with FP64 accumulation, reduces seven inf-norms as
// ordered bit patterns (exact and order-independent, NaN-propagating), publishes them, and
// every workgroup reduces all partials itself. All workgroups therefore take bit-identical
// decisions (eqs. primal, dual and rho_update) without a broadcast.
#pragma once
#include "layer_kernel.h"

#include "device_common.h"

namespace rqp {
namespace {

constexpr int BS = kLayerBlock;
constexpr int NWAVE = BS / kWave;
constexpr unsigned kSpinLimit = 1u << 22;
// Pauses (in units of 64 clocks) before the first poll of an exchange and between polls. A poll of all
// words by all workgroups moves megabytes over the fabric, and one that comes before the words can be
// there delays the words themselves: with the first poll at once an iteration took 2.96 us at 3200 FP32
// rows, 2.68 at 2400, 1.76 at 800, and 5.96 us at 3000 FP64 rows; with the pause 1.77, 1.65, 1.36 and
// 3.03. Half the pause and one and a half times it cost about 15 % and 10 %; a pause that adapts to
// whether the first poll hits settles longer or shorter than the best and was 5-20 % slower.
// The best pause grows with the words and the workgroups (us per iteration at pauses of 12 / 18 / 24; the
// rule is within 2.7 % of the best of 8, 12, 18, 24 and 30 at 40 grids between 136 and 4000 rows):
//   FP64, workgroups x rows: 11 x 136 1.46 / 1.51 / 1.67, 23 x 280 1.62 / 1.59 / 1.65, 32 x 400 1.69 / 1.60 /
//     1.70, 88 x 1100 2.23 / 1.89 / 1.87, 128 x 1600 2.54 / 2.17 / 2.05, 160 x 2000 2.63 / 2.14 / 2.07,
//     240 x 3000 3.93 / 3.17 / 2.99
//   FP32: 16 x 200 1.28 / 1.33 / 1.49, 30 x 600 1.73 / 1.76 / 1.92, 32 x 400 1.35 / 1.31 / 1.45,
//     128 x 1600 1.67 / 1.59 / 1.74, 240 x 3000 1.84 / 1.73 / 1.81
// so below 32 workgroups 12 and 18 are level or 12 wins, from 32 on 18 does, and 24 where FP64 words reach
// the quarter million. The norm partials' exchange is polled once a check and always waits kPollWait.
constexpr int kPollWait = 18, kPollWaitFew = 12, kPollWaitMany = 24;
template <typename T>
__device__ __forceinline__ void poll_wait(int L) {
  if (gridDim.x < 32)
    __builtin_amdgcn_s_sleep(kPollWaitFew);
  else if (sizeof(T) == sizeof(double) && gridDim.x * L > 256 * 1024)
    __builtin_amdgcn_s_sleep(kPollWaitMany);
  else
    __builtin_amdgcn_s_sleep(kPollWait);
}
constexpr int kPollSleep = 1;

template <typename T>
constexpr int words() {
  return LLWords<T>::kWords;
}

enum { ST_RUNNING = 0, ST_SOLVED = 1, ST_MAX_ITER = 2, ST_NONFINITE = 3, ST_ABORTED = 4, ST_INTERNAL = 5 };
constexpr int kMaxRho = 64;  // the host accepts at most 64 penalty values

// penalty grid and the geometric midpoints between neighbours, copied to LDS once per launch
struct RhoTable {
  double grid[kMaxRho];
  double mid[kMaxRho];
};
enum { N_RP = 0, N_RD, N_AX, N_Z, N_PX, N_ATY, N_Q, N_FLAGS };

// The error word holds the tag of the solve that failed, so a failure never leaks into a later
// solve (each solve has its own tag range).
__device__ __forceinline__ bool err_set(const unsigned* err, uint32_t tag) {
  return __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == tag;
}
__device__ __forceinline__ void err_raise(unsigned* err, uint32_t tag) {
  __hip_atomic_store(err, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Poll the exchange words of this lane's columns tid + cs k until every tag equals `tag`; only the last
// of the NC columns can lie past L (last: this lane's does not). Agent-scope loads of one word (FP32) or
// of the two words of a value together (FP64; each word is valid by its own tag). A lane leaves the loop
// by itself: one exit for the whole wave, words awaited one after another, or two polls in flight all
// took longer (1.67 us for an exchange of 3200 words over 256 workgroups; 1.85, 2.5 and 2.2 us).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
template <typename T, int NC>
__device__ __forceinline__ bool gather(const uint64_t* buf, int L, int cs, bool last, uint32_t tag, T (&v)[NC],
                                       const unsigned* err, uint32_t etag) {
  bool ok = true;
  unsigned spins = 0;
  poll_wait<T>(L);
  if constexpr (sizeof(T) == sizeof(float)) {
    uint64_t w[NC];
    const uint64_t* const p = buf + threadIdx.x;
    while (true) {
#pragma unroll
      for (int k = 0; k < NC; ++k) w[k] = k < NC - 1 || last ? ll_load_word(p + cs * k) : (uint64_t)tag << 32;
      bool all = true;
#pragma unroll
      for (int k = 0; k < NC; ++k) all &= ll_tag(w[k]) == tag;
      if (all) break;
      if ((++spins & 255u) == 0u && (spins > kSpinLimit || err_set(err, etag))) {
        ok = false;
        break;
      }
      // a short pause thins the polling traffic of all workgroups while the producers' stores travel
      __builtin_amdgcn_s_sleep(kPollSleep);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) v[k] = ll_value_f(w[k]);
  } else {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)buf, 0, (unsigned)L * 16u, 0x00027000);
    u32x4 w[NC];
    while (true) {
#pragma unroll
      for (int k = 0; k < NC - 1; ++k)
        w[k] = __builtin_amdgcn_raw_buffer_load_b128(rs, threadIdx.x * 16u, k * cs * 16, kAgentScope);
      // the column that can lie past L (reads zero) by the lane's offset alone: the uniform offset is no
      // part of the bounds check's contract
      w[NC - 1] = __builtin_amdgcn_raw_buffer_load_b128(rs, (threadIdx.x + cs * (NC - 1)) * 16u, 0, kAgentScope);
      bool all = true;
#pragma unroll
      for (int k = 0; k < NC; ++k) all &= (w[k].y == tag && w[k].w == tag) || (k == NC - 1 && !last);
      asm volatile("" ::: "memory");  // every round reads again
      if (all) break;
      if ((++spins & 255u) == 0u && (spins > kSpinLimit || err_set(err, etag))) {
        ok = false;
        break;
      }
      __builtin_amdgcn_s_sleep(kPollSleep);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) v[k] = bits_to_double((uint64_t)w[k].x | ((uint64_t)w[k].z << 32));
  }
  return ok;
}

// Poll the 2-word FP64 norm partials of all workgroups (count of them, at most 8 * 256: one per
// workgroup and norm); mx: the largest of this lane's entries tid and tid + BS, which carry norm
// tid % 8.
__device__ __forceinline__ bool gather_norms(const uint64_t* buf, int count, uint32_t tag, uint64_t& mx,
                                             const unsigned* err, uint32_t etag) {
  const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)buf, 0, (unsigned)count * 16u, 0x00027000);
  const unsigned tid = threadIdx.x;
  const bool in0 = (int)tid < count, in1 = (int)tid + BS < count;
  u32x4 w0, w1;
  unsigned spins = 0;
  __builtin_amdgcn_s_sleep(kPollWait);
  while (true) {
    w0 = __builtin_amdgcn_raw_buffer_load_b128(rs, tid * 16u, 0, kAgentScope);
    w1 = __builtin_amdgcn_raw_buffer_load_b128(rs, (tid + BS) * 16u, 0, kAgentScope);
    const bool miss = (in0 && (w0.y != tag || w0.w != tag)) || (in1 && (w1.y != tag || w1.w != tag));
    asm volatile("" ::: "memory");
    if (__builtin_amdgcn_ballot_w64(miss) == 0) break;
    if ((++spins & 255u) == 0u && (spins > kSpinLimit || err_set(err, etag))) return false;
    __builtin_amdgcn_s_sleep(kPollSleep);
  }
  const uint64_t v0 = (uint64_t)w0.x | ((uint64_t)w0.z << 32), v1 = (uint64_t)w1.x | ((uint64_t)w1.z << 32);
  mx = v0 > v1 ? v0 : v1;  // entries out of range read as zero
  return true;
}

// Poll one FP64 value (two words) until both tags equal `tag`.
__device__ __forceinline__ bool wait_f64(const uint64_t* p, uint32_t tag, double& v, const unsigned* err,
                                         uint32_t etag) {
  uint64_t w0 = ll_load_word(p), w1 = ll_load_word(p + 1);
  unsigned spins = 0;
  bool ok = true;
  while (ll_tag(w0) != tag || ll_tag(w1) != tag) {
    w0 = ll_load_word(p);
    w1 = ll_load_word(p + 1);
    if ((++spins & 255u) == 0u && (spins > kSpinLimit || err_set(err, etag))) {
      ok = false;
      break;
    }
  }
  v = bits_to_double(ll_bits64(w0, w1));
  return ok;
}

// Closed loop: the plant state after solve sv - 1, x_sv = Ad x_{sv-1} + Bd u_{sv-1}. Each
// workgroup keeps its own copy of the state in xpl (parity sv & 1); u comes from the words the
// first nu constraint-row owners published at the end of solve sv - 1 (tag utag), staged in
// ucur. Each wave forms PR state entries per pass (their loads in flight together):
// per entry, lane-strided FP64 products then a butterfly sum, the same order in every
// workgroup, so every copy is the same. Returns false if the wait for u timed out.
template <int NWV, int PR>
__device__ __forceinline__ bool plant_step(const LayerArgs& a, int sv, uint32_t utag, double* ucur, int* flag) {
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const uint64_t* uw = a.xu + (long)((sv - 1) & 1) * a.nu * 2;
  if (tid < a.nu) {
    double v;
    if (!wait_f64(uw + 2L * tid, utag, v, a.err, utag)) *flag = 1;
    ucur[tid] = v;
  }
  __syncthreads();
  if (*flag) return false;
  const double* xc = a.xpl + ((long)((sv - 1) & 1) * gridDim.x + blockIdx.x) * kMaxPlant;
  double* xn = a.xpl + ((long)(sv & 1) * gridDim.x + blockIdx.x) * kMaxPlant;
  const int nx = a.nx, nu = a.nu;
  for (int rb = wave * PR; rb < nx; rb += NWV * PR) {
    double dv[PR];
    int rc[PR];  // a valid row index for every slot (entries past nx are not stored)
#pragma unroll
    for (int b = 0; b < PR; ++b) {
      dv[b] = 0.0;
      rc[b] = rb + b < nx ? rb + b : nx - 1;
    }
    for (int c = lane; c < nx; c += kWave) {
      const double xv = xc[c];
#pragma unroll
      for (int b = 0; b < PR; ++b) dv[b] = fma(a.Ad[(long)rc[b] * nx + c], xv, dv[b]);
    }
    for (int c = lane; c < nu; c += kWave) {
      const double uv = ucur[c];
#pragma unroll
      for (int b = 0; b < PR; ++b) dv[b] = fma(a.Bd[(long)rc[b] * nu + c], uv, dv[b]);
    }
#pragma unroll
    for (int b = 0; b < PR; ++b) {
#pragma unroll
      for (int off = kWave / 2; off > 0; off >>= 1) dv[b] += __shfl_xor(dv[b], off, kWave);
      if (lane == 0 && rb + b < nx) xn[rb + b] = dv[b];
    }
  }
  __syncthreads();
  return true;
}

// State of the rows a workgroup owns, in LDS (entry i: row r0 + i, read and written by thread i
// except where a barrier lies between). Kept there and not in the owners' registers because every
// lane of the workgroup pays for those: the registers hold weights.
template <typename T>
struct RowState {
  T s[kMaxRows];    // x of an x row, z of a constraint row
  T y[kMaxRows];    // y of a constraint row
  T q[kMaxRows];    // q of an x row, l of a constraint row
  T u[kMaxRows];    // u of a constraint row
  T rho[kMaxRows];  // penalty of a constraint row
  // the part of the next update that does not wait for the product: (1 - alpha) x, or
  // (1 - alpha) z + y / rho
  T pre[kMaxRows];
  double ax[kMaxRows];  // constraint rows: (A x)_i (closed loops and scaled problems carry it along)
};

// Four consecutive entries of a row of the check matrix (16-byte aligned: ldw is a multiple
// of 4) and of the staged check vector.
__device__ __forceinline__ void load_quad(const float* p, float (&v)[4]) {
  const float4 t = *reinterpret_cast<const float4*>(p);
  v[0] = t.x;
  v[1] = t.y;
  v[2] = t.z;
  v[3] = t.w;
}
__device__ __forceinline__ void load_quad(const double* p, double (&v)[4]) {
  const double2 t0 = *reinterpret_cast<const double2*>(p), t1 = *reinterpret_cast<const double2*>(p + 2);
  v[0] = t0.x;
  v[1] = t0.y;
  v[2] = t1.x;
  v[3] = t1.y;
}

// The residual check's rows of this workgroup: dual rows cb .. cb + nck - 1 (x rows of [P, A'],
// all L columns) and primal rows pb .. pb + np - 1 (constraint rows, [A, 0]: the first n columns).
// The first cd dual and the first cp primal rows are kept in LDS (cache: dual rows of ldw entries,
// then primal rows of ldn) for the whole launch; the others are read from memory at every check.
template <typename T>
struct CheckRows {
  int cb, nck, pb, np, cd, cp;
  T* cache;
};

// Slice s of the LDS copy: one 1 KB wave instruction per wave, straight from memory to LDS. The
// slices are issued one per iteration of the first solve, behind the iteration's exchange, so that
// the read of the check matrix costs the first check nothing.
template <typename T>
__device__ __forceinline__ int cache_quads(const LayerArgs& a, const CheckRows<T>& cr) {
  constexpr int E = 16 / sizeof(T);
  return cr.cd * (int)(a.ldw / E) + cr.cp * (((a.n + 3) & ~3) / E);
}
template <typename T>
__device__ __forceinline__ void cache_slice(const LayerArgs& a, const CheckRows<T>& cr, int s, int wave, int lane) {
  constexpr int E = 16 / sizeof(T);  // entries per 16 bytes
  const int qd = (int)(a.ldw / E), qp = ((a.n + 3) & ~3) / E;
  const int nd = cr.cd * qd, total = nd + cr.cp * qp;
  const int e0 = (s * NWAVE + wave) * kWave;
  if (e0 >= total) return;
  int e = e0 + lane < total ? e0 + lane : total - 1;
  long off = (long)cr.cb * qd + e;  // in 16-byte quads
  if (e >= nd) {
    e -= nd;
    off = (long)(cr.pb + e / qp) * qd + e % qp;
  }
  lds_copy16(static_cast<const unsigned char*>(a.C) + off * 16, reinterpret_cast<unsigned char*>(cr.cache) + e0 * 16);
}

// Partial sums of the check rows. The rows are cut into units of kUnit columns and every wave takes
// a contiguous, equal share of the units (a lane holds 4 columns of a unit), so a wave reduces over
// its lanes once per row it touches instead of every wave once per row. body[i]: the sums of the
// wave that holds row i's first unit; head[w]: those of wave w for row head_row[w], which it starts in
// the middle of (-1: none). Each entry: the product with the x part (P x, or A x), with the y part
// (A'y), and (FP32 only: the rounding bound) the sum of the absolute values of the products, all FP64
// sums of the exact FP64 products.
constexpr int kUnit = 4 * kWave;
struct CheckSums {
  double body[kMaxCheckRows + kMaxRows][3];
  double head[NWAVE][3];
  int head_row[NWAVE];
};
// The sums of row i (dual rows first), in all 16 lanes of an aligned group (lane w of it adds wave
// w's part, in one fixed tree: independent of timing).
template <typename T>
__device__ __forceinline__ void row_sums(const CheckSums& cs, int i, double& p, double& q, double& f) {
  const int w = threadIdx.x % 16;
  const bool mine = w == 0 || cs.head_row[w] == i;
  const double* const src = w == 0 ? cs.body[i] : cs.head[w];
  p = mine ? src[0] : 0.0;
  q = mine ? src[1] : 0.0;
  f = mine && sizeof(T) == sizeof(float) ? src[2] : 0.0;
  auto sum16 = [](double v) {
    v = dpp_add<0xb1, 0xf>(v);    // quad_perm [1,0,3,2]
    v = dpp_add<0x4e, 0xf>(v);    // quad_perm [2,3,0,1]
    v = dpp_add<0x141, 0xf>(v);   // row_half_mirror
    return dpp_add<0x140, 0xf>(v);  // row_mirror
  };
  p = sum16(p);
  q = sum16(q);
  if constexpr (sizeof(T) == sizeof(float)) f = sum16(f);
}

// Forms the partial sums of the products with [x; y], staged in LDS (zeros up to whole units). A
// barrier must lie before and after.
template <typename T>
__device__ __forceinline__ void check_products(const LayerArgs& a, const CheckRows<T>& cr, CheckSums& cs,
                                               const T* stage) {
  constexpr bool F32 = sizeof(T) == sizeof(float);
  const int lane = threadIdx.x % kWave, wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int n = a.n, L = a.L, ldw = (int)a.ldw, ldn = (n + 3) & ~3;
  const int ud = (L + kUnit - 1) / kUnit, up = (n + kUnit - 1) / kUnit;
  const int nd = cr.nck * ud, total = nd + cr.np * up;
  const int t0 = total * wave / NWAVE, t1 = total * (wave + 1) / NWAVE;
  if (t0 >= t1) {
    if (lane == 0) cs.head_row[wave] = -1;
    return;
  }
  const T* const Cm = static_cast<const T*>(a.C);
  int row = t0 < nd ? t0 / ud : cr.nck + (t0 - nd) / up;
  int un = t0 < nd ? t0 % ud : (t0 - nd) % up;
  if (lane == 0) cs.head_row[wave] = un != 0 ? row : -1;
  double* dst = un != 0 ? cs.head[wave] : cs.body[row];
  double p = 0.0, q = 0.0, f = 0.0;
  // this lane's four entries of unit u of row r
  auto load = [&](int r, int u, T(&w)[4]) __attribute__((always_inline)) {
    const bool dual = r < cr.nck;
    const int c = u * kUnit + 4 * lane;
    const int i = dual ? r : r - cr.nck;
    if (c >= (dual ? ldw : ldn)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = (T)0;
    } else if (i < (dual ? cr.cd : cr.cp)) {
      load_quad(cr.cache + (dual ? i * ldw : cr.cd * ldw + i * ldn) + c, w);
    } else {
      load_quad(Cm + (long)((dual ? cr.cb : cr.pb) + i) * ldw + c, w);
    }
  };
  T w[4], wn[4];
  load(row, un, w);
#pragma unroll 1
  for (int t = t0; t < t1; ++t) {
    const bool dual = row < cr.nck;
    const bool end = un + 1 == (dual ? ud : up);  // last unit of the row
    const int row2 = end ? row + 1 : row, un2 = end ? 0 : un + 1;
    if (t + 1 < t1) load(row2, un2, wn);
    const int c0 = un * kUnit, c = c0 + 4 * lane;
    T v[4];
    load_quad(stage + c, v);
    if (c0 + kUnit <= n) {
#pragma unroll
      for (int e = 0; e < 4; ++e) p = fma((double)w[e], (double)v[e], p);
    } else if (c0 >= n) {
#pragma unroll
      for (int e = 0; e < 4; ++e) q = fma((double)w[e], (double)v[e], q);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // a primal row ends at column n: a non-finite y must not reach it through the zero block
        const bool in = c + e < n;
        const double wd = (double)w[e], vx = in ? (double)v[e] : 0.0, vy = in || !dual ? 0.0 : (double)v[e];
        p = fma(wd, vx, p);
        q = fma(wd, vy, q);
        if (!in && !dual) v[e] = (T)0;
      }
    }
    if constexpr (F32) {
      double t = fabs((double)w[0]) * fabs((double)v[0]);
#pragma unroll
      for (int e = 1; e < 4; ++e) t = fma(fabs((double)w[e]), fabs((double)v[e]), t);
      f += t;
    }
    if (end || t + 1 == t1) {
      if constexpr (F32) {
        double pqf[4] = {p, q, f, 0.0};
        const double s = reduce_rows<4>(pqf);  // lanes 0, 16 and 32 hold p, q and f
        if (row_writer<4>() && lane < 48) dst[lane >> 4] = s;
      } else {
        double pq[2] = {p, q};
        const double s = reduce_rows<2>(pq);  // lanes 0 and 32 hold p and q
        if (row_writer<2>()) dst[lane >> 5] = s;
      }
      p = 0.0;
      q = 0.0;
      f = 0.0;
      dst = cs.body[row2];
    }
    row = row2;
    un = un2;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = wn[e];
  }
}

// Bound factor of the check in FP32: with the stored matrices and the returned x, z, y rounded
// to FP32 (unit roundoff u = 2^-24), the products exact in FP64 and FP64 accumulation over at
// most L terms here and in the CPU's evaluation, |computed - FP64 value| <= kappa0 * sum |a v|
// per row with kappa0 = 2u + 2 (L + 8) 2^-53. The sum of absolute values is an FP64 sum like the others,
// so the factor 1.02 is room to spare (the rounding of the bound and of its own sum is below 1e-12).
// FP64 handles compute the FP64 residual itself (0).
template <typename T>
__device__ __forceinline__ double check_kappa(int L) {
  if constexpr (sizeof(T) == sizeof(double)) {
    return 0.0;
  } else {
    return 1.02 * (2.0 * 0x1p-24 + 2.0 * (double)(L + 8) * 0x1p-53);
  }
}
template <typename T>
__device__ __forceinline__ double unit_roundoff() {
  return sizeof(T) == sizeof(double) ? 0.0 : 1.01 * 0x1p-24;
}

struct CheckOut {
  int status;  // ST_* (ST_RUNNING: continue)
  int jn;      // grid index for the next iterations
  bool ok;     // false: an exchange timed out
};

// Publish [x; y] of the owned rows under tag ctag and gather all of it into `stage` (zeros up to whole
// units of the check). A barrier must follow; a timeout raises *fail.
template <typename T, int NC>
__device__ __forceinline__ void stage_xy(const LayerArgs& a, const RowState<T>& rs, uint64_t* xc, int r0, int nrows,
                                         int cs, bool wave_on, bool last, uint32_t ctag, uint32_t tag, T* stage,
                                         int* fail) {
  constexpr int NW = LLWords<T>::kWords;
  const int tid = threadIdx.x, L = a.L;
  if (tid < nrows) ll_store(xc + (long)(r0 + tid) * NW, r0 + tid < a.n ? rs.s[tid] : rs.y[tid], ctag);
  const int pad = (L + kUnit - 1) / kUnit * kUnit;
  if (L + tid < pad) stage[L + tid] = (T)0;
  if (wave_on) {
    T cv[NC];
    if (!gather<T, NC>(xc, L, cs, last, ctag, cv, a.err, tag)) *fail = 1;
#pragma unroll
    for (int k = 0; k < NC; ++k)
      if (k < NC - 1 || last) stage[tid + cs * k] = cv[k];
  }
}

// Residual check (eqs. primal, dual), stopping test and penalty rule (eq. rho_update; nearest
// grid value, Sec. III-C) at iteration k, check number nchk. [x; y] goes to every workgroup; dual
// side: this workgroup's share of the x rows of [P, A'] [x; y]; primal side: A x for the constraint
// rows it owns, formed afresh from the check matrix (FP64 accumulation, left in rs.ax); the seven
// partial inf-norms are published and every workgroup reduces all of them, so every workgroup
// takes the same decision. With the iteration in FP32 the published r_p and r_d are upper bounds,
// and ||Ax||, ||z||, ||Px||, ||A'y||, ||q|| lower bounds, of the FP64 values a CPU evaluation of
// the returned x, z, y with the caller's FP64 P, q, A gives (check_kappa), so SOLVED implies that
// the FP64 test passes.
//
// Everything here is latency: four barriers, two exchanges, and code that the instruction cache
// refetches at every check, so it is kept small (unrolled over the units of the products and over
// the waves' parts, with one thread summing a row's parts, seven LDS atomics per row and one thread
// deciding, a check took 19.7 us at 3200 FP32 rows on 256 workgroups).
template <typename T, int NC, bool XT>
__device__ __forceinline__ CheckOut check(const LayerArgs& a, RowState<T>& rs, const CheckRows<T>& cr, int r0,
                                          int nrows, int cs, bool wave_on, bool last, const T* cq, int k, int nchk,
                                          int j, uint32_t tag, const RhoTable& rt, CheckSums& sums, T* stage,
                                          int* fail, long hoff) {
  __shared__ unsigned long long nmax[8];        // the workgroup's partial norms (ordered bit patterns)
  __shared__ uint64_t nred[2][NWAVE][8];        // the waves' maxima over all workgroups, two parities of checks
  constexpr int NW = LLWords<T>::kWords;
  const int G = gridDim.x, g = blockIdx.x, tid = threadIdx.x;
  const int lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int L = a.L, par = nchk & 1;
  const uint32_t ctag = tag + (uint32_t)k;
  CheckOut out{ST_RUNNING, j, false};
  if (tid < 8) nmax[tid] = 0ull;
  stage_xy<T, NC>(a, rs, a.xc + (long)par * L * NW, r0, nrows, cs, wave_on, last, ctag, tag, stage, fail);
  __syncthreads();
  if (*fail) return out;
  check_products<T>(a, cr, sums, stage);
  __syncthreads();

  // norms: 16 lanes per row, lane i of them taking norm i
  const double kappa = check_kappa<T>(L), ut = unit_roundoff<T>();
  const int nr = cr.nck + cr.np;
  uint64_t nb = 0;
#pragma unroll 1
  for (int i = tid / 16; i < nr; i += BS / 16) {
    double p, q, d;
    row_sums<T>(sums, i, p, q, d);
    d *= kappa;
    const int which = lane % 16;
    double v = 0.0, f = 1.0;
    if (i < cr.nck) {
      const double qv = (double)cq[i], dq = ut * fabs(qv);
      if (XT && a.sc_dual) f = a.sc_dual[cr.cb + i];  // original units
      if (which == N_RD) v = fabs(p + qv + q) + d + dq;
      if (which == N_PX) v = lower_bound(fabs(p), d);
      if (which == N_ATY) v = lower_bound(fabs(q), d);
      if (which == N_Q) v = lower_bound(fabs(qv), dq);
    } else {
      const int lr = cr.pb - r0 + i - cr.nck;
      const double zv = (double)rs.s[lr], dz = ut * fabs(zv);
      if (XT && a.sc_prim) f = a.sc_prim[cr.pb + i - cr.nck - a.n];
      if (which == N_RP) v = fabs(p - zv) + d + dz;
      if (which == N_AX) v = lower_bound(fabs(p), d);
      if (which == N_Z) v = lower_bound(fabs(zv), dz);
      if (which == 0) rs.ax[lr] = p;
    }
    const uint64_t b = abs_bits(f * v);
    nb = b > nb ? b : nb;
  }
  if (wave * 4 < nr) {
    nb = max_swap<32>(max_swap<16>(nb));
    if (lane < 7) atomicMax(&nmax[lane], (unsigned long long)nb);
  }
  __syncthreads();
  uint64_t* const xn = a.xn + (long)par * G * 8 * 2;
  if (tid < 8) {
    uint64_t v = nmax[tid];
    if (tid == N_FLAGS) {
      // the host-mapped flag costs a PCIe round trip (~13 us measured), so it is read at
      // every kAbortEvery-th check only
      const bool ab = (nchk % kAbortEvery) == kAbortEvery - 1 && a.abort_flag &&
                      __hip_atomic_load(a.abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
      v = err_set(a.err, tag) ? 2u : (ab ? 1u : 0u);
    }
    ll_store_bits64(xn + (g * 8 + tid) * 2, v, ctag);
  }

  // all workgroups' partials; every wave reduces and decides for itself
  uint64_t mx = 0;
  if (!gather_norms(xn, G * 8, ctag, mx, a.err, tag)) *fail = 1;
  mx = max_over_groups(mx);
  if (lane < 8) nred[par][wave][lane] = mx;
  __syncthreads();
  if (*fail) return out;
  out.ok = true;
  static_assert(NWAVE == 16, "two waves' maxima per lane");
  const uint64_t m0 = nred[par][lane / 8][lane % 8], m1 = nred[par][8 + lane / 8][lane % 8];
  mx = max_over_groups(m0 > m1 ? m0 : m1);
  uint64_t nf[8];
  bool nonfinite = false;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)mx, i);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(mx >> 32), i);
    nf[i] = (uint64_t)lo | ((uint64_t)hi << 32);
    if (i < 7) nonfinite |= nf[i] >= kInfBits;
  }
  const double rp = bits_to_double(nf[N_RP]), rd = bits_to_double(nf[N_RD]);
  const double nax = bits_to_double(nf[N_AX]), nz = bits_to_double(nf[N_Z]);
  const double npx = bits_to_double(nf[N_PX]), naty = bits_to_double(nf[N_ATY]);
  const double nq = bits_to_double(nf[N_Q]);
  int st = ST_RUNNING;
  if (nonfinite) {
    st = ST_NONFINITE;
  } else if (a.terminate) {
    const double eps_p = a.eps_abs + a.eps_rel * fmax(nax, nz);
    const double eps_d = a.eps_abs + a.eps_rel * fmax(fmax(npx, naty), nq);
    if (rp <= eps_p && rd <= eps_d) st = ST_SOLVED;
  }
  if (st == ST_RUNNING && k == a.max_iter) st = ST_MAX_ITER;
  if (st == ST_RUNNING && nf[N_FLAGS] >= 2) st = ST_INTERNAL;
  if (st == ST_RUNNING && nf[N_FLAGS] == 1) st = ST_ABORTED;
  int jn = j;
  if (st == ST_RUNNING && a.n_rho > 1 && rp > 0.0 && rd > 0.0) {
    const double num = rp * fmax(fmax(npx, naty), fmax(nq, 1e-4));
    const double den = rd * fmax(fmax(nax, nz), 1e-4);
    const double rh = rt.grid[j] * sqrt(num / den);
    // lane i compares with midpoint i; the midpoints rise, so the count of those below is the index
    jn = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < a.n_rho - 1 && rh > rt.mid[lane]));
  }
  out.status = __builtin_amdgcn_readfirstlane(st);
  out.jn = jn;
  if (g == 0 && tid == 0) {
    if (a.rho_hist) a.rho_hist[hoff + nchk] = jn;
    if (a.prim_res) a.prim_res[hoff + nchk] = rp;
    if (a.dual_res) a.dual_res[hoff + nchk] = rd;
  }
  return out;
}

template <typename T, bool XT>
__device__ __forceinline__ void finish(const LayerArgs& a, const RowState<T>& rs, int r0, int nrows, int sv, int k,
                                       int st, int j, uint32_t tag, const double* exs) {
  const int tid = threadIdx.x, R = r0 + tid;
  if (tid < nrows) {
    // the handle keeps the (scaled) iterates; the outputs are in original units
    const T s = rs.s[tid];
    if (R < a.n) {
      static_cast<T*>(a.xs)[R] = s;
      static_cast<T*>(a.xo)[(long)sv * a.n + R] = XT && a.un_x ? (T)(a.un_x[R] * (double)s) : s;
    } else {
      const int i = R - a.n;
      const T y = rs.y[tid];
      static_cast<T*>(a.zs)[i] = s;
      static_cast<T*>(a.ys)[i] = y;
      a.axs[i] = rs.ax[tid];
      static_cast<T*>(a.zo)[(long)sv * a.m + i] = XT && a.sc_prim ? (T)(a.sc_prim[i] * (double)s) : s;
      static_cast<T*>(a.yo)[(long)sv * a.m + i] = XT && a.un_y ? (T)(a.un_y[i] * (double)y) : y;
      if (XT && a.Ad && i < a.nu) {
        // the first stage's applied control (the clamped constraint row plus its E x_s part)
        const double uv = ((double)s + exs[tid]) * (a.sc_prim ? a.sc_prim[i] : 1.0);
        a.traj_u[(long)sv * a.nu + i] = uv;
        ll_store(a.xu + ((long)(sv & 1) * a.nu + i) * 2, uv, tag);
      }
    }
  }
  if (blockIdx.x == 0 && tid == 0) {
    a.iterations[sv] = k;
    a.status[sv] = st;
    a.rho_index[sv] = j;
    *a.js = j;
  }
}

// This lane's columns of the first NRS rows of the block (zero past the block or past L).
template <typename T, int NC, int NRS>
__device__ __forceinline__ void load_stationary(const LayerArgs& a, int j, int r0, int nrows, int cs,
                                                T (&wst)[NRS][NC]) {
  const T* Wj = static_cast<const T*>(a.W) + (long)j * a.w_stride;
  const int tid = threadIdx.x;
#pragma unroll
  for (int rr = 0; rr < NRS; ++rr)
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int c = tid + cs * k;
      wst[rr][k] = (rr < nrows && tid < cs && c < a.L) ? Wj[(long)(r0 + rr) * a.ldw + c] : (T)0;
    }
}

// Rows NRS .. NRS + nl - 1 of the block live in LDS, row after row (ldw entries each); every lane
// writes and reads only its own columns, so no barrier is needed.
template <typename T, int NC>
__device__ __forceinline__ void load_lds_rows(const LayerArgs& a, int j, int first, int nl, int cs, T* wl) {
  const T* Wj = static_cast<const T*>(a.W) + (long)j * a.w_stride + (long)first * a.ldw;
  if ((int)threadIdx.x >= cs) return;
#pragma unroll 1
  for (int rr = 0; rr < nl; ++rr) {
    T v[NC];
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int c = threadIdx.x + cs * k;
      v[k] = Wj[c < a.L ? (long)rr * a.ldw + c : 0];
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int c = threadIdx.x + cs * k;
      if (c < a.L) wl[rr * (int)a.ldw + c] = v[k];
    }
  }
}

// Sum of the waves' partials of one row (contiguous in LDS), pairwise.
__device__ __forceinline__ float sum_waves(const float* p) {
  float s[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float4 t = *reinterpret_cast<const float4*>(p + 4 * i);
    s[i] = (t.x + t.y) + (t.z + t.w);
  }
  return (s[0] + s[1]) + (s[2] + s[3]);
}
__device__ __forceinline__ double sum_waves(const double* p) {
  double s[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const double2 t = *reinterpret_cast<const double2*>(p + 2 * i);
    s[i] = t.x + t.y;
  }
  return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
}

// The kernel reads its arguments through the kernarg segment pointer made opaque at the start of
// each phase (fresh), so a phase loads the fields it uses instead of every field of the whole
// persistent loop staying in scalar registers (which spills them into vector registers).
typedef const __attribute__((address_space(4))) LayerArgs* cargs_t;
__device__ __forceinline__ const LayerArgs& fresh(cargs_t p) {
  asm volatile("" : "+s"(p));
  return *(const LayerArgs*)p;
}

template <typename T, int NC, int NRS, bool XT>
__global__ void __launch_bounds__(BS) layer_kernel(LayerArgs a_in) {
  (void)a_in;
  const cargs_t kp = (cargs_t)__builtin_amdgcn_kernarg_segment_ptr();
  const LayerArgs& a = fresh(kp);
  constexpr int NW = LLWords<T>::kWords;
  // partial row sums of the waves, two parities of the iteration: a wave that is already past the next
  // exchange must not overwrite sums that an owner of a late workgroup still reads
  __shared__ __align__(16) T red[2][kMaxRows][NWAVE];
  __shared__ int fail_flag;
  __shared__ RhoTable rt;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  T* const cstage = reinterpret_cast<T*>(dyn_lds);  // the check vector (check_cols entries)
  T* const wl = cstage + a.check_cols;               // LDS rows of the layer (lds_rows of ldw entries)
  T* const ccache = wl + (long)a.lds_rows * a.ldw;   // rows of the check matrix (cache_bytes)

  const int G = gridDim.x, g = blockIdx.x, tid = threadIdx.x;
  const int lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int n = a.n, L = a.L;
  const int rbase = L / G, rextra = L % G;
  const int nrows = rbase + (g < rextra ? 1 : 0);
  const int r0 = g * rbase + (g < rextra ? g : rextra);
  const int nlds = nrows - NRS < a.lds_rows ? nrows - NRS : a.lds_rows;  // rows in LDS (none if <= 0)
  constexpr int RP = NRS > 8 && NC * words<T>() <= 5 ? 16 : 8;             // register rows reduced together
  constexpr int EB = layer_pass_rows<T>(NC);                               // further rows at a time
  const int cs = a.col_lanes;                                     // columns are spread over lanes 0 .. cs - 1
  const bool wave_on = wave * kWave < cs;                         // this wave holds columns
  const bool last = tid < cs && tid + cs * (NC - 1) < L;          // this lane's last column exists
  const bool wave_last = wave_on && wave * kWave + cs * (NC - 1) < L;  // some lane's of the wave does
  const int my_row = rows_held<RP>(), my_row_e = rows_held<EB>();
  const bool writer = row_writer<RP>();
  // Rows that the plant step and a loop's update of q, l, u take together, between solves, while the
  // weights stay in registers: one where those hold more than 26 of them, else rows of weights go to scratch
  // memory and back in every step (a step of two iterations of 400 / 800 FP64 rows took 9.9 / 10.7 us
  // with 4 and 2 and takes 8.4 / 9.3, of 3200 / 4000 FP32 rows 18.7 / 27.4 and 17.1 / 23.7).
  constexpr bool FULL = NRS * NC * words<T>() > 26;
  constexpr int PR = FULL ? 1 : 4, UB = XT && FULL ? 1 : 2;
  if (tid == 0) fail_flag = 0;
  for (int i = tid; i < 2 * kMaxRows * NWAVE; i += BS) (&red[0][0][0])[i] = (T)0;  // waves without columns
  if (tid < a.n_rho) rt.grid[tid] = a.grid[tid];
  if (tid < a.n_rho - 1) rt.mid[tid] = a.mid[tid];
  __syncthreads();

  // Solves s = 0 .. count-1 run one after another in this launch; the weights of the active
  // penalty stay on chip between them. Solve s uses tags tag0 + s * span, takes its data from
  // x0 + s * nx (when given) and writes its results at index s of the outputs.
  const uint32_t span = solve_span(a.max_iter);
  const int ci = a.check_interval, max_iter = a.max_iter;
  __shared__ RowState<T> rs;
  const bool own = tid < nrows, xrow = r0 + tid < n;
  const int R = r0 + tid;
  const bool seq = own && !xrow && a.eq[R - n] != 0;
  if (own) rs.ax[tid] = 0.0;
  int j = a.warm ? *a.js : a.j0;
  int lds_j = -1;  // penalty index of the rows now in LDS
  int wst_j = -1;  // penalty index of the rows now in registers
  T wst[NRS][NC];
  // this workgroup's share of the x rows for the dual side of the check, and their q
  // (split_term, split_row: a running maximum over h <= g, here a prefix maximum over wave 0,
  // lane l holding h = 4 l + 1 .. 4 l + 4; the grid has at most 256 workgroups)
  __shared__ int split[2];
  if (wave == 0) {
    double run = 0.0, mh[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = 4 * lane + i + 1;
      const double f = h <= G ? split_term(h, G, n, a.m, L) : 0.0;
      run = f > run ? f : run;
      mh[i] = run;
    }
    double inc = run;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const double o = __shfl_up(inc, off, kWave);
      if (lane >= off) inc = o > inc ? o : inc;
    }
    double exc = __shfl_up(inc, 1, kWave);
    if (lane == 0) exc = 0.0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int h = 4 * lane + i + 1;
      const double best = exc > mh[i] ? exc : mh[i];
      if (h == g) split[0] = split_row(best, n, L);
      if (h == g + 1) split[1] = split_row(best, n, L);
    }
    if (g == 0 && lane == 0) split[0] = 0;
  }
  __syncthreads();
  const int cb = split[0], nck = split[1] - split[0];
  __shared__ T cq[kMaxCheckRows];
  __shared__ CheckSums csum;
  CheckRows<T> cr;
  cr.cb = cb;
  cr.nck = nck;
  cr.pb = r0 > n ? r0 : n;
  cr.np = r0 + nrows > cr.pb ? r0 + nrows - cr.pb : 0;
  cr.cache = ccache;
  {
    const int db = (int)a.ldw * (int)sizeof(T), pb = ((n + 3) & ~3) * (int)sizeof(T);
    cr.cd = a.cache_bytes / db < nck ? a.cache_bytes / db : nck;
    cr.cp = (a.cache_bytes - cr.cd * db) / pb < cr.np ? (a.cache_bytes - cr.cd * db) / pb : cr.np;
  }
  // slices of the LDS copy of the check rows; a closed loop whose steps never check needs none
  if (XT && !a.final_check && a.max_iter < a.check_interval) cr.cd = cr.cp = 0;
  const int nslice = (cache_quads(a, cr) + BS - 1) / BS;
  int slice = 0;
  // closed loop: (E x_s)_i of the owned constraint rows; the applied control
  __shared__ double exs[kMaxRows];
  __shared__ double ucur[kMaxPlant];
  // XT instantiations also run closed loops and scaled problems; the others carry none of
  // that code (its registers would cost the plain solves)
  const bool closed = XT && a.Ad != nullptr;

  for (int sv = 0; sv < a.count; ++sv) {
    const LayerArgs& a = fresh(kp);
    const uint32_t tag = a.tag + (uint32_t)sv * span;
    const bool warm = sv == 0 ? a.warm != 0 : a.chain != 0;

    // update from an initial state (Sec. IV): q = F x0 for x rows, l = lo - E x0 and
    // u = hi - E x0 for constraint rows, FP64 products, one wave per row of the block; the
    // values reach the owners through LDS and are written back for later solves
    __syncthreads();  // the previous solve is done with rs and cq
    double* xpl = closed ? a.xpl + ((long)(sv & 1) * G + g) * kMaxPlant : nullptr;
    if (closed) {
      if (sv == 0) {
        for (int c = tid; c < a.nx; c += BS) xpl[c] = a.x0[c];
        __syncthreads();
      } else if (!plant_step<NWAVE, PR>(a, sv, tag - span, ucur, &fail_flag)) {
        if (tid == 0) err_raise(a.err, tag);
        finish<T, XT>(a, rs, r0, nrows, sv, 0, ST_INTERNAL, j, tag, exs);
        return;
      }
      if (g == 0)
        for (int c = tid; c < a.nx; c += BS) a.traj_x[(long)sv * a.nx + c] = xpl[c];
    }
    if (a.x0) {
      const double* x0 = closed ? xpl : a.x0 + (long)sv * a.nx;
      // rows 0 .. nrows-1: owned layer rows; rows nrows .. nrows+nck-1: the check's x rows
      // (UB rows of a wave at a time, their loads and lane sums interleaved)
      for (int rb = wave * UB; rb < nrows + nck; rb += NWAVE * UB) {
        double du[UB];
        const double* ar[UB];
#pragma unroll
        for (int u = 0; u < UB; ++u) {
          const int rr = rb + u < nrows + nck ? rb + u : rb;
          const int Rr = rr < nrows ? r0 + rr : cb + (rr - nrows);
          ar[u] = Rr < n ? a.F + (long)Rr * a.nx : a.E + (long)(Rr - n) * a.nx;
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
          if (rr >= nrows + nck) break;
          const int Rr = rr < nrows ? r0 + rr : cb + (rr - nrows);
          const double dv = du[u];
          if (lane == 0) {
            if (rr >= nrows) {
              cq[rr - nrows] = (T)dv;
            } else if (Rr < n) {
              rs.q[rr] = (T)dv;
              static_cast<T*>(const_cast<void*>(a.q))[Rr] = (T)dv;
            } else {
              const int i = Rr - n;
              if constexpr (XT) exs[rr] = dv;
              const T lo = (T)(a.plo[i] - dv), up = (T)(a.phi[i] - dv);
              rs.q[rr] = lo;
              rs.u[rr] = up;
              static_cast<T*>(const_cast<void*>(a.l))[i] = lo;
              static_cast<T*>(const_cast<void*>(a.u))[i] = up;
            }
          }
        }
      }
    } else if (tid < nck) {
      cq[tid] = static_cast<const T*>(a.q)[cb + tid];
    }
    __syncthreads();

    // row-owner state: cold (zero, start penalty), warm from the handle (first solve) or from
    // the previous solve of this launch. In the XT instantiation (closed loops, scaled
    // problems) a warm start that continues a solve takes z = A x from the product the
    // constraint-row owners carried along it (in registers within the launch, from the
    // handle's copy across launches); otherwise, and for a caller-given x, z = A x is formed
    // through the check product (keeping the carried value live costs the plain loop).
    const bool carried = XT && warm && (sv > 0 || a.warm_ax != 0);
    if (own) {
      if (xrow) {
        if (!a.x0) rs.q[tid] = static_cast<const T*>(a.q)[R];
        if (!warm) rs.s[tid] = (T)0;
        else if (sv == 0) rs.s[tid] = static_cast<const T*>(a.xs)[R];
      } else {
        const int i = R - n;
        if (!a.x0) {
          rs.q[tid] = static_cast<const T*>(a.l)[i];
          rs.u[tid] = static_cast<const T*>(a.u)[i];
        }
        if (!warm) rs.y[tid] = (T)0;
        else if (sv == 0) rs.y[tid] = static_cast<const T*>(a.ys)[i];
        if (!carried) rs.ax[tid] = 0.0;
        else if (sv == 0) rs.ax[tid] = a.axs[i];
        rs.s[tid] = carried ? (T)rs.ax[tid] : (T)0;
      }
    }
    if (!warm) j = a.j0;
    if (j != lds_j) {
      load_lds_rows<T, NC>(a, j, r0 + NRS, nlds, cs, wl);
      lds_j = j;
    }
    int nchk = 0;

    // warm start from a caller-given x: z = A x (Sec. II-B, warm starting)
    if (warm && !carried) {
      stage_xy<T, NC>(a, rs, a.xc, r0, nrows, cs, wave_on, last, tag, tag, cstage, &fail_flag);
      __syncthreads();
      if (fail_flag) {
        if (tid == 0) err_raise(a.err, tag);
        finish<T, XT>(a, rs, r0, nrows, sv, 0, ST_INTERNAL, j, tag, exs);
        return;
      }
      // the constraint rows of the block: [A, 0] [x; y] (the LDS copy once it is complete)
      CheckRows<T> pr = cr;
      pr.nck = 0;
      pr.cd = 0;
      pr.cache = cr.cache + (long)cr.cd * a.ldw;
      if (slice < nslice || sv == 0) pr.cp = 0;
      check_products<T>(a, pr, csum, cstage);
      __syncthreads();
      for (int i = tid / 16; i < pr.np; i += BS / 16) {
        double p, unused, unused2;
        row_sums<T>(csum, i, p, unused, unused2);
        if (lane % 16 == 0) {
          rs.ax[pr.pb - r0 + i] = p;
          rs.s[pr.pb - r0 + i] = (T)p;
        }
      }
      __syncthreads();
    }

    // first layer input w_1, and the penalty and next update's constant part of every owned row
    auto start_segment = [&](const LayerArgs& a, int k0) __attribute__((always_inline)) {
      if (own) {
        const T s = rs.s[tid], oma = (T)(1.0 - a.alpha);
        T w, pre;
        if (xrow) {
          w = (T)a.sigma * s - rs.q[tid];
          pre = oma * s;
        } else {
          const T rho = (T)(rt.grid[j] * (seq ? a.rho_eq_scale : 1.0)), y = rs.y[tid];
          rs.rho[tid] = rho;
          w = rho * s - y;
          pre = fma(oma, s, y / rho);
        }
        ll_store(a.xw + ((long)word_half(tag, k0 + 1) * L + R) * NW, w, tag + (uint32_t)(k0 + 1));
        rs.pre[tid] = pre;
      }
    };
    start_segment(a, 0);

    // the register rows of the active penalty, unless the previous solve left them in place
    if (wst_j != j) {
      load_stationary<T, NC, NRS>(a, j, r0, nrows, cs, wst);
      wst_j = j;
    }
    int k = 0;
    while (true) {
      const int kend = (k / ci + 1) * ci < max_iter ? (k / ci + 1) * ci : max_iter;
      {
        const LayerArgs& a = fresh(kp);
        const T alpha = (T)a.alpha, oma = (T)(1.0 - a.alpha), sigma = (T)a.sigma;
        [[maybe_unused]] const double alpha_d = a.alpha, oma_d = 1.0 - a.alpha;
        uint64_t* xw = a.xw;
        while (k < kend) {
          ++k;
          // layer matvec: rows of Wc_j times w_k
          T(*const rk)[NWAVE] = red[k & 1];
          if (wave_on) {
            T wv[NC];
            if (!gather<T, NC>(xw + (long)word_half(tag, k) * L * NW, L, cs, last, tag + (uint32_t)k, wv, a.err, tag))
              fail_flag = 1;
            // register rows, RP at a time: products, then one multi-row wave reduction
#pragma unroll
            for (int rb = 0; rb < NRS; rb += RP) {
              T acc[RP];
#pragma unroll
              for (int b = 0; b < RP; ++b) {
                acc[b] = (T)0;
                if (rb + b < NRS) {
#pragma unroll
                  for (int k2 = 0; k2 < NC - 1; ++k2) acc[b] = fma(wst[rb + b < NRS ? rb + b : 0][k2], wv[k2], acc[b]);
                }
              }
              if (wave_last) {
#pragma unroll
                for (int b = 0; b < RP; ++b)
                  if (rb + b < NRS) acc[b] = fma(wst[rb + b < NRS ? rb + b : 0][NC - 1], wv[NC - 1], acc[b]);
              }
              const T rsum = reduce_rows<RP>(acc);
              if (writer && rb + my_row < NRS) rk[rb + my_row][wave] = rsum;
            }
            // further rows, EB at a time, from LDS or memory
            for (int rb = NRS; rb < nrows; rb += EB) {
              const T* const Wj = static_cast<const T*>(a.W) + (long)j * a.w_stride + (long)r0 * a.ldw;
              T acc[EB], we[EB][NC];
#pragma unroll
              for (int b = 0; b < EB; ++b) {
                const int rr = rb + b < nrows ? rb + b : nrows - 1;
                if (rr - NRS < nlds) {
                  const T* const p = wl + (rr - NRS) * (int)a.ldw + tid;
#pragma unroll
                  for (int k2 = 0; k2 < NC - 1; ++k2) we[b][k2] = p[cs * k2];
                  we[b][NC - 1] = last ? p[cs * (NC - 1)] : (T)0;
                } else {
                  const T* const p = Wj + (long)rr * a.ldw + tid;
#pragma unroll
                  for (int k2 = 0; k2 < NC - 1; ++k2) we[b][k2] = p[cs * k2];
                  we[b][NC - 1] = last ? p[cs * (NC - 1)] : (T)0;
                }
              }
#pragma unroll
              for (int b = 0; b < EB; ++b) {
                acc[b] = (T)0;
#pragma unroll
                for (int k2 = 0; k2 < NC; ++k2) acc[b] = fma(we[b][k2], wv[k2], acc[b]);
              }
              const T rsum = reduce_rows<EB>(acc);
              if (row_writer<EB>() && rb + my_row_e < nrows) rk[rb + my_row_e][wave] = rsum;
            }
          }
          __syncthreads();
          if (fail_flag) {
            if (tid == 0) err_raise(a.err, tag);
            finish<T, XT>(a, rs, r0, nrows, sv, k, ST_INTERNAL, j, tag, exs);
            return;
          }

          // row-local update: relaxation, clamp (eq. clamp), dual update
          // No barrier after this: red has two parities, and a wave that writes one again has passed
          // the next iteration's barrier, which the owners reach after reading it.
          if (own) {
            const T pre = rs.pre[tid], q = rs.q[tid];
            const T v = sum_waves(rk[tid]);
            uint64_t* const xo = xw + ((long)word_half(tag, k + 1) * L + R) * NW;
            const T t = fma(alpha, v, pre);
            if (xrow) {
              if (k < kend) ll_store(xo, sigma * t - q, tag + (uint32_t)(k + 1));
              rs.s[tid] = t;
              rs.pre[tid] = oma * t;
            } else {
              const T rho = rs.rho[tid], zn = box_clamp(t, q, rs.u[tid]), y = rho * (t - zn);
              if (k < kend) ll_store(xo, rho * zn - y, tag + (uint32_t)(k + 1));
              rs.s[tid] = zn;
              rs.y[tid] = y;
              rs.pre[tid] = fma(oma, zn, y / rho);
              // closed loops, scaled problems: A x_{k+1} = alpha A x~ + (1 - alpha) A x_k, with
              // A x~ the layer output v (the z = A x of a warm start that continues this solve)
              if constexpr (XT) rs.ax[tid] = fma(alpha_d, (double)v, oma_d * rs.ax[tid]);
            }
          }
          if (slice < nslice) cache_slice(a, cr, slice++, wave, lane);
        }
      }

      const LayerArgs& ac = fresh(kp);
      // a fixed budget that is not a multiple of the check interval ends without a check
      // (closed loops; they run the XT instantiation)
      if constexpr (XT) {
        if (!ac.final_check && k == max_iter && k % ci != 0) {
          finish<T, XT>(ac, rs, r0, nrows, sv, k, ST_MAX_ITER, j, tag, exs);
          break;  // next solve of the sequence
        }
      }

      // check at iteration k (every check_interval iterations and at max_iter)
      __syncthreads();
      while (slice < nslice) cache_slice(ac, cr, slice++, wave, lane);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the LDS copy (the check has the barrier)
      const CheckOut co = check<T, NC, XT>(ac, rs, cr, r0, nrows, cs, wave_on, last, cq, k, nchk, j, tag, rt, csum,
                                           cstage, &fail_flag, (long)sv * ac.max_checks);
      ++nchk;
      if (!co.ok) {
        if (tid == 0) err_raise(ac.err, tag);
        finish<T, XT>(ac, rs, r0, nrows, sv, k, ST_INTERNAL, j, tag, exs);
        return;
      }
      if (co.status != ST_RUNNING) {
        finish<T, XT>(ac, rs, r0, nrows, sv, k, co.status, j, tag, exs);
        break;  // next solve of the sequence
      }
      if (co.jn != j) {
        j = co.jn;
        load_lds_rows<T, NC>(ac, j, r0 + NRS, nlds, cs, wl);
        lds_j = j;
        start_segment(ac, k);
        load_stationary<T, NC, NRS>(ac, j, r0, nrows, cs, wst);
        wst_j = j;
      } else {
        start_segment(ac, k);
      }
    }
  }

  // closed loop: the state after the last control, written by workgroup 0
  if (closed && g == 0) {
    const uint32_t last = a.tag + (uint32_t)(a.count - 1) * span;
    __syncthreads();
    if (!plant_step<NWAVE, PR>(a, a.count, last, ucur, &fail_flag)) {
      if (tid == 0) err_raise(a.err, last);
      return;
    }
    const double* xf = a.xpl + ((long)(a.count & 1) * G + g) * kMaxPlant;
    for (int c = tid; c < a.nx; c += BS) a.traj_x[(long)a.count * a.nx + c] = xf[c];
  }
}

// The kernel for nc columns per lane, with layer_reg_rows or (more) layer_more_rows rows in registers.
template <typename T, int NC, bool XT>
const void* fn_at(bool more) {
  constexpr int A = layer_reg_rows<T>(NC), B = layer_more_rows<T>(NC, XT);
  return more ? reinterpret_cast<const void*>(&layer_kernel<T, NC, B, XT>)
              : reinterpret_cast<const void*>(&layer_kernel<T, NC, A, XT>);
}
template <typename T, bool XT>
const void* fn_for(int nc, bool more) {
  switch (nc) {
    case 1: return fn_at<T, 1, XT>(more);
    case 2: return fn_at<T, 2, XT>(more);
    case 3: return fn_at<T, 3, XT>(more);
    case 4: return fn_at<T, 4, XT>(more);
    case 5: return fn_at<T, 5, XT>(more);
    case 6: return fn_at<T, 6, XT>(more);
    case 7: return fn_at<T, 7, XT>(more);
    case 8: return fn_at<T, 8, XT>(more);
    default: return nullptr;
  }
}

}  // namespace
}  // namespace rqp
