// Online-stage kernel of the ReLU-QP solver: the whole loop of Algorithm 1 in one launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rqp {

// Arguments of one persistent solve. Vectors are in the iterate precision T unless noted.
struct LayerArgs {
  int n, m, L;          // L = n + m rows of the compact layer
  long ldw;             // leading dimension of the layer and check matrices (elements)
  const void* W;        // n_rho layer matrices [D, DA'; AD, ADA'] (L x ldw each, T)
  long w_stride;        // elements between consecutive penalty matrices
  const void* C;        // check matrix [P, A'; A, 0] (L x ldw, T)
  const void* q;        // n
  const void* l;        // m
  const void* u;        // m
  const unsigned char* eq;  // m flags: l_i == u_i
  const double* grid;   // n_rho penalty values
  const double* mid;    // n_rho - 1 geometric midpoints between neighbouring grid values
  int n_rho;
  double sigma, alpha, eps_abs, eps_rel, rho_eq_scale;
  int max_iter, check_interval, terminate, warm, j0;
  void* xs;             // handle state x (n), z (m), y (m): read on a warm start, written at exit
  void* zs;
  void* ys;
  int* js;              // handle state penalty index
  double* axs;          // handle state A x (m, FP64): the constraint-row owners' carried product
  int warm_ax;          // a warm first solve takes z = A x from axs (the state came from a solve)
  int count;            // solves run one after another in this launch (>= 1)
  int chain;            // solves after the first start warm from the previous one
  int max_checks;       // per-solve stride of rho_hist, prim_res, dual_res
  void* xo;             // caller outputs (device), count solves: x count*n, z, y count*m
  void* zo;
  void* yo;
  int* iterations;      // count entries each
  int* status;
  int* rho_index;
  int* rho_hist;        // per check, may be null
  double* prim_res;     // per check, may be null
  double* dual_res;     // per check, may be null
  uint64_t* xw;         // exchange words: layer input, 2 parities x L x words
  uint64_t* xc;         // exchange words: check vector [x; y], 2 x L x words
  uint64_t* xn;         // exchange words: norm partials, 2 x G x 8 x 2
  uint32_t tag;         // first tag of the launch; solve s uses tag + s (max_iter + 2) onwards
  const int* abort_flag;  // host-mapped int, polled at checks
  unsigned* err;        // device word: holds the tag of a solve whose exchange timed out
  int lds_rows;         // rows per block kept in LDS (set by launch_layer from the plan)
  int check_cols;       // entries of LDS for the check vector (set likewise)
  int cache_bytes;      // bytes of LDS for rows of the check matrix (set likewise)
  int col_lanes;        // lanes of a workgroup that hold columns (set likewise)
  // optional in-kernel update from initial states (x0 != null, count x nx): q = F x0,
  // l = lo - E x0, u = hi - E x0, written to q, l, u before each solve starts
  const double* x0;
  const double* F;      // n x nx
  const double* E;      // m x nx
  const double* plo;    // m
  const double* phi;    // m
  int nx;
  // optional closed loop (Ad != null, needs x0): solve s starts from the plant state x_s, with
  // x_0 = x0 and x_{s+1} = Ad x_s + Bd u_s, where u_s = z_s[0:nu] + (E x_s)[0:nu] is the first
  // stage's applied control. The owners of constraint rows 0..nu-1 publish u_s in xu
  // (2 parities x nu x 2 words) and every workgroup steps the plant itself, in FP64, in one
  // fixed order (so every copy of x_{s+1} is the same). Trajectories go to traj_x
  // ((count + 1) x nx) and traj_u (count x nu), FP64.
  const double* Ad;     // nx x nx
  const double* Bd;     // nx x nu
  int nu;
  uint64_t* xu;
  double* xpl;          // each workgroup's copy of the plant state: 2 parities x grid x kMaxPlant
  double* traj_x;
  double* traj_u;
  int final_check;      // 0: a max_iter that is not a multiple of check_interval ends unchecked
  // Ruiz scaling (null: none). The kernel iterates on the scaled problem; the check weights
  // each row's terms so that residuals and norms are the original problem's, and the outputs
  // are written unscaled. sc_dual = 1 / (c D) (n), sc_prim = 1 / E (m), un_x = D (n),
  // un_y = E / c (m).
  const double* sc_dual;
  const double* sc_prim;
  const double* un_x;
  const double* un_y;
};

// nx and nu of a closed loop are at most kMaxPlant; grids are at most kMaxGrid workgroups.
constexpr int kMaxPlant = 256;
constexpr int kMaxGrid = 256;

// Rows per workgroup are at most kMaxRows; the host picks the grid accordingly.
constexpr int kLayerBlock = 1024;
constexpr int kMaxLayerRows = 8 * kLayerBlock;
constexpr int kMaxRows = 64;

// The two halves of the layer-input words. Word k (k = 1, 2, ...) of a solve whose tags start at `tag`
// carries tag + k and lies in half word_half(tag, k). Two consecutive words of a launch must lie in
// different halves: a workgroup overwrites word i by word i + 2 only after it gathered all of word i + 1,
// which every workgroup publishes only after it gathered all of word i, so nobody still polls for the word
// that is lost. Consecutive over the end of a solve too: a closed loop's step can end without a check, and
// the next one's first word is then held back by the owners of the applied control alone. With the half
// taken from the tag, word k = max_iter is followed by tag + solve_span(max_iter) + 1 = (tag + k) + 3. (A
// step that ends earlier ends at a check, whose exchanges wait for every workgroup.)
__host__ __device__ inline uint32_t solve_span(int max_iter) { return (uint32_t)max_iter + 2u; }  // tags of a solve
__host__ __device__ inline int word_half(uint32_t tag, int k) { return (int)((tag + (uint32_t)k) & 1u); }

// Split of the residual check over the workgroups. The check reads n L entries of [P, A'] for
// the x rows (dual side) and n m of [A, 0] for the constraint rows (primal side); each
// workgroup forms the constraint rows it owns in the layer (rows split evenly, L / G each), and
// the x rows are split so that every workgroup reads about (n L + n m) / G entries in all.
// split_term(h) is the x-row work (in entries) before workgroup h under that rule; the first x
// row of workgroup g is floor(max_{h <= g} split_term(h) / L), at most n (a running maximum
// keeps the split monotone; g = G gives n). The quotients are formed in double: exact for
// these magnitudes (every product is an integer below 2^53, and a non-integer quotient lies at
// least 1/L from an integer), so host and device agree.
__host__ __device__ inline double split_term(int h, int G, int n, int m, int L) {
  const double total = (double)n * (double)L + (double)n * (double)m;
  const double f = floor((double)h * total / (double)G);
  const int rbase = L / G, rextra = L % G;
  const double r0h = (double)h * rbase + (h < rextra ? h : rextra);
  const double v = f - (double)n * (r0h > n ? r0h - n : 0.0);
  return v > 0.0 ? v : 0.0;
}
__host__ __device__ inline int split_row(double best, int n, int L) {
  const double cb = floor(best / (double)L);
  return cb < (double)n ? (int)cb : n;
}
inline int check_split(int g, int G, int n, int m, int L) {
  double best = 0.0;
  for (int h = 1; h <= g; ++h) {
    const double f = split_term(h, G, n, m, L);
    best = f > best ? f : best;
  }
  return split_row(best, n, L);
}
// The largest share of x rows the split gives a workgroup: at most ceil(L / G) + 1.
constexpr int kMaxCheckRows = kMaxRows + 2;

// Rows of a block that stay in registers when a lane owns nc columns: at most 13, what
// ceil(L / 12.5) workgroups leave a block, and at most about 64 of the 128 registers a lane of a
// 1024-thread workgroup has.
template <typename T>
constexpr int layer_reg_rows(int nc) {
  return sizeof(T) == sizeof(double) ? (nc <= 2 ? 13 : 32 / nc) : (nc <= 5 ? 13 : 64 / nc);
}
// Further rows are multiplied this many at a time, each pass with a read of LDS (or memory) and a reduction
// over the lanes of its own.
template <typename T>
constexpr int layer_pass_rows(int nc) {
  const int regs = nc * (int)sizeof(T) / 4;
  return regs <= 4 ? 8 : (regs <= 8 ? 4 : 2);
}
// An instantiation for blocks of more rows (a smaller grid, or more than 3328 rows in all) keeps as many in
// registers as fit the same 64, at most 32, in whole groups of the 16 that are reduced together. It is
// taken where it saves a pass: 200 iterations of 1600 FP32 rows at 20 / 24 / 32 rows a block took 524 / 687 /
// 842 us with 13 rows in registers and take 453 / 452 / 454 with 32; at 3200 rows and 24 a block 876 and 673
// with 16, but at 20 a block, one pass either way, 615 and 672: its rows cost registers and products too.
// FP64 closed loops and scaled solves (xt) stop at 16, what else they hold leaves no room: 50 steps of 16
// iterations of 144 rows at 16 a block took 1849 us with 32 and take 1607, at 32 a block 1796 and 2469.
template <typename T>
constexpr int layer_more_rows(int nc, bool xt) {
  const int most = 64 * 4 / (int)sizeof(T) / nc / 16 * 16, cap = xt && sizeof(T) == sizeof(double) ? 16 : 32;
  return most > cap ? cap : (most > layer_reg_rows<T>(nc) ? most : layer_reg_rows<T>(nc));
}
template <typename T>
constexpr bool layer_takes_more(int nc, int rows, bool xt) {
  const int pass = layer_pass_rows<T>(nc), a = rows - layer_reg_rows<T>(nc), b = rows - layer_more_rows<T>(nc, xt);
  return (b > 0 ? (b + pass - 1) / pass : 0) < (a > 0 ? (a + pass - 1) / pass : 0);
}

// Lanes (a multiple of the wave size) that hold the columns of the rows. A wave pays for the reduction
// of its 13 rows over its lanes however few columns a lane has, so fewer, fuller waves run fewer
// instructions; but every column is one more polled word per lane. In units of instructions of the
// busiest SIMD: waves per SIMD times (13 per column plus the reduction's, about 64 in FP32 and 140 in
// FP64), plus 90 per polled word: within 2.5 % of the best of the measured lane counts at each size (us per
// iteration at the rule's / 1024 / 640 / 512 / 256 lanes: 3200 FP32 rows 1.77 / 1.73 / 1.84 / - / -, 2400 rows
// 1.65 / 1.68 / 1.63 / 1.65 / -, 800 rows 1.36 / 1.49 / 1.41 / 1.37 / 1.45; 800 FP64 rows 1.76 / 1.99 / 1.92 /
// 1.76 / -, 156 rows 1.55 / 1.91 / 1.72 / 1.59 / 1.52; -: too few lanes for these columns).
template <typename T>
inline int layer_col_lanes(int L) {
  const int most = sizeof(T) == sizeof(double) ? 2 : 5, red = sizeof(T) == sizeof(double) ? 140 : 64;
  int best = kLayerBlock, cost = 1 << 30;
  for (int cs = 64; cs <= kLayerBlock; cs += 64) {
    const int nc = (L + cs - 1) / cs;
    if (nc > most) continue;
    const int c = (cs + 255) / 256 * (13 * nc + red) + 90 * nc;
    if (c < cost) {
      best = cs;
      cost = c;
    }
  }
  return best;
}

// Kernel choice and resources for a problem on `grid` workgroups: the first layer_reg_rows rows of
// each block (layer_more_rows where that saves a pass) stay in registers and the next lds_rows in LDS for the
// whole launch; further rows stream from memory every iteration.
struct LaunchPlan {
  const void* fn;
  int lds_rows;
  int on_chip;     // rows a block can keep in registers and LDS
  int check_cols;  // entries of LDS for the check vector
  int cache_bytes; // LDS for rows of the check matrix
  int col_lanes;   // lanes of a workgroup that hold columns
  size_t dyn_bytes;
  int max_grid;    // largest cooperative grid with these resources
};
// xt: the instantiation that also runs closed loops and Ruiz-scaled problems.
template <typename T>
LaunchPlan plan_layer(int n, int m, int grid, bool xt);

// Launch the persistent solve as a cooperative grid of `grid` workgroups of kLayerBlock threads.
template <typename T>
hipError_t launch_layer(const LayerArgs& a, const LaunchPlan& p, int grid, hipStream_t st);

}  // namespace rqp
