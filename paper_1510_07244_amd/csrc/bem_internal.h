// Internal declarations of the MI355X BEM assembly library (not installed).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <map>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "../../include/bem.h"

namespace bem {

// --------------------------------------------------------------- quadrature
// q-point Gauss-Legendre rule on [0,1], nodes increasing.
void gauss_legendre01(int q, double *x, double *w);

// Points of a rule on one flat triangle in the coordinates of the affine map
// Phi(s,t) = v0 + s (v1 - v0) + t (v2 - v1), such that
//   int_tau f ~ sqrt(g) * sum_k w[k] f(Phi(s[k], t[k])).
struct TriRule {
  std::vector<double> s, t, w;
};
TriRule triangle_rule(int rule, int q);
// Constants of the Duffy rule of order q in the block kernels' layout (DuffyAt).
std::vector<double> duffy_table(int q);
// Constants of any other rule, with s' = s - 2/3 and t' = t - 1/3 from the
// centroid: s, t, w, e = t - s / 2, s', t', s'^2, s' e, e^2 [9][points].
std::vector<double> general_table(const TriRule &r);
// The same in FP32, with weights whose sum is that of the exact ones to a
// rounding of the last.
std::vector<float> duffy_table32(int q);
std::vector<float> general_table32(const TriRule &r);

// Sauter-Schwab rule of one singular class, factored as (x^, y^) = xi g(eta):
// per region and (eta1, eta2, eta3) Gauss triple the map g at xi = 1
// (xs, xt, ys, yt) and the weight w_b w_c w_d J(eta) / xi^3; the xi nodes and
// weights w_a xi_a^3 are in XiRule.
struct SSRule {
  std::vector<double> xs, xt, ys, yt, w;
};
struct XiRule {
  std::vector<double> x, w3;
};
enum { CLS_DISJOINT = 0, CLS_VERTEX = 1, CLS_EDGE = 2, CLS_IDENTICAL = 3 };
SSRule ss_rule(int cls, int q);
XiRule xi_rule(int q);

// Sauter-Schwab rule of one class for piecewise-constant entries, factored
// into directions d = g1 E1_i + g2 E2_i - g3 E1_j - g4 E2_j with weight w and
// radial nodes p (x - y = p d) with weights ws (single layer) and wd (double
// layer); series: see singular_rule.
constexpr int kSeries = 12;  // coefficients per power series
struct SingularRule {
  std::vector<double> g[4], w;
  std::vector<double> p, ws, wd;
  double series[4][kSeries];  // single layer even, odd; double layer even, odd
};
SingularRule singular_rule(int cls, int q);

// --------------------------------------------------------------- geometry
// Per-triangle geometry, structure of arrays: geo[f * ldg + i].
enum GeoField {
  G_V0X, G_V0Y, G_V0Z,  // first vertex
  G_E1X, G_E1Y, G_E1Z,  // v1 - v0
  G_E2X, G_E2Y, G_E2Z,  // v2 - v1
  G_SG,                 // sqrt of the Gram determinant = 2 * area
  G_NX, G_NY, G_NZ,     // outward unit normal
  G_LOX, G_LOY, G_LOZ,  // bounding box
  G_HIX, G_HIY, G_HIZ,
  G_R2,                 // largest squared distance of a point from the centroid
  GEO_NF
};

// sticky device flags
// FLAG_LIST: a sub-tile listed more pairs for the FP64 pass than its list
// holds (mirrored edge-adjacent pairs of edges shared by many triangles)
enum : unsigned { FLAG_EINVAL = 1u, FLAG_NONFINITE = 2u, FLAG_LIST = 4u };

// Device copies of the quadrature tables of one (rule, q_regular, q_singular),
// in one allocation.
struct DevRules {
  double *mem = nullptr;
  int nq = 0;                   // points per triangle (regular rule)
  const double *tri = nullptr;  // [3][nq]: s, t, w (general_table: the first rows of sums)
  // constants of the block kernels' regular sums, in double and in float:
  // duffy_table for the Duffy orders 2 .. 6, else general_table
  const double *sums = nullptr, *sums32 = nullptr;
  // Sauter-Schwab eta tables per class 1..3 (piecewise-linear bases)
  int np[4] = {0, 0, 0, 0};
  const double *ss[4] = {nullptr, nullptr, nullptr, nullptr};  // [5][np]: xs, xt, ys, yt, w
  int nxi = 0;                  // Sauter-Schwab order q
  const double *xi = nullptr;   // [2][q]: xi, w xi^2
  // factored singular rules per class 1..3 (piecewise-constant entries):
  // series [4][kSeries], then directions [5][nd]: g1 .. g4, w, then radial
  // nodes [3][nr]: p, ws, wd
  int nd[4] = {0, 0, 0, 0}, nr[4] = {0, 0, 0, 0};
  const double *sing[4] = {nullptr, nullptr, nullptr, nullptr};
};

// Device Sauter-Schwab tables as seen by the kernels of piecewise-constant
// entries (DevRules::sing).
struct SSArgs {
  const double *tab[4];
  int32_t nd[4], nr[4];
};

// Tables of the piecewise-linear kernels (DevRules::ss, xi).
struct P1Rules {
  const double *eta[4];  // per class [5][np]
  int32_t np[4];
  const double *xi;      // [2][q]
  int32_t q;
};
SSArgs ss_args(const DevRules &r);

// Arguments of the block kernels (passed by value).
struct BlockArgs {
  const double *v;
  const int32_t *tri;
  int32_t nv, nt;
  const double *geo;
  int64_t ldg;
  int32_t nblocks;
  const int32_t *row_ptr, *row_idx, *col_ptr, *col_idx;
  int64_t row_len, col_len;
  const int64_t *out_off;
  const int64_t *mirror_off;  // coupling of a single layer: transposed copies (or null)
  void *out;
  void *out2;          // both layers in one pass: the double layer's output
  int64_t out_len;
  const double *rule;  // [3][nq]
  const double *sums;  // DevRules::sums, mixed form sums32 (float)
  int32_t nq, nq_pad;
  int32_t tr, tc;      // sub-tile rows / columns
  int32_t wide, slots; // columns of a full sub-tile, which may list tr * wide
                       // pairs; list slots of this one (at least tr * tc)
  int32_t split;       // workgroups per block (per-block kernels)
  int32_t *brief;      // per block: whether its Helmholtz phases are short
                       // (launch_begin), null: every work item finds out
  SSArgs ss;
  double kappa;
  double near_ratio;   // mixed form: near-singular box-distance ratio
  unsigned *flags;
};

struct EntryArgs {
  const double *v;
  const int32_t *tri;
  int32_t nv, nt;
  const double *geo;
  int64_t ldg;
  int64_t n;
  const int32_t *rows, *cols;
  void *out;
  const double *rule;
  int32_t nq;
  SSArgs ss;
  double kappa;
  unsigned *flags;
};

struct GreenArgs {
  const double *geo;
  int64_t ldg;
  int32_t nt;
  int32_t ncl;
  const int32_t *row_ptr, *row_idx;
  int64_t row_len;
  int32_t m;
  const double *z, *zn, *zw, *delta;
  const int64_t *out_off;
  void *out;
  int64_t out_len;
  const double *rule;
  int32_t nq;
  double kappa;
  unsigned *flags;
};

struct ContractArgs {
  int32_t nmat;
  const int32_t *nrows, *rank, *piv_cols;
  int32_t max_rank;
  const double *pinv;
  const void *A;
  const int64_t *a_off;
  int32_t acols;
  int64_t a_len;
  void *V;
  const int64_t *v_off;
  int64_t v_len;
  unsigned *flags;
};

struct PivInvArgs {
  int32_t nmat;
  const int32_t *nrows, *rank, *piv_rows, *piv_cols;
  int32_t max_rank;
  const void *A;
  const int64_t *a_off;
  int32_t acols;
  int64_t a_len;
  double *pinv;
  unsigned *flags;
};

// Arguments of the persistent batched block kernel: one BlockArgs per batch
// entry (all with the same rule and sub-tile shape) and a queue of sub-tiles.
struct PersistentArgs {
  const BlockArgs *batches;  // device [nbatch]
  const int32_t *mode;       // device [nbatch]: bit 0 coupling block list,
                             // bits 1-2 layer (BEM_SLP, BEM_DLP, kBoth = 2)
  const int4 *tiles;         // device [ntiles]: batch, block, first row, first column
  int32_t ntiles, nbatch;
  int32_t *counter;          // device queue head, 0 at launch
  int32_t grid;              // workgroups
};

// Grouped gathered matrix-vector products of the H^2 matrix (bem_h2mv.hip).
struct GemvArgs {
  int32_t ngroups, nblocks;
  const int32_t *grp_ptr;            // [ngroups + 1] blocks of each group
  const int32_t *out_ptr, *out_idx;  // [ngroups + 1], output indices into y
  int64_t out_len;                   // length of out_idx
  const int32_t *in_ptr, *in_idx;    // [nblocks + 1], input indices into x
  int64_t in_len;                    // length of in_idx
  const int64_t *a_off;              // [nblocks] matrix offsets (entries)
  const void *A;
  int64_t a_len;
  const void *x;
  int64_t x_len;
  void *y;
  int64_t y_len;
  unsigned *flags;
};
hipError_t launch_gemv(bool cplx, bool trans, const GemvArgs &a, hipStream_t s);
size_t dot_scratch_doubles();
hipError_t launch_dot(bool cplx, bool conj, int64_t n, const double *x, const double *y,
                      double *part, double *out, hipStream_t s);
hipError_t launch_axpby(bool cplx, int64_t n, double ar, double ai, const double *x, double br,
                        double bi, double *y, hipStream_t s);
// one conjugate-gradient update with the scalars in state (bem_cg_step)
hipError_t launch_cg_step(int64_t n, double *state, double *x, double *r, double *p,
                          const double *q, double *dot_part, hipStream_t s);
hipError_t launch_mass(bool cplx, int32_t nt, const double *geo, int64_t ldg, double cr, double ci,
                       const double *x, double *y, hipStream_t s);

// Piecewise-linear bases (bem_p1.hip).
struct P1Args {
  const double *v;
  const int32_t *tri;
  int32_t nv, nt;
  const double *geo;
  int64_t ldg;
  int64_t n;
  const int32_t *rows, *cols;
  void *out;  // [n][9] entries
  const double *rule;
  int32_t nq;
  P1Rules ss;
  double kappa;
  unsigned *flags;
};
struct P1GatherArgs {
  int32_t nrv, ncv, ntr, ntc;
  const int32_t *rs_ptr, *rs_tri, *rs_loc;
  const int32_t *cs_ptr, *cs_tri, *cs_loc;
  int64_t rs_len, cs_len;
  const void *local;
  void *out;
  unsigned *flags;
};
hipError_t launch_p1_pairs(int kernel, int layer, const P1Args &a, hipStream_t s);
hipError_t launch_p1_gather(bool cplx, const P1GatherArgs &a, hipStream_t s);

// ----------------------------------------------------------- learned form
constexpr int kSelQ = 6;  // selector outputs: predicted log10 error at orders 1 .. 6

// Training samples of the order selector (inputs and targets of pairs).
struct SampleArgs {
  const int32_t *tri;
  int32_t nt;
  const double *geo;
  int64_t ldg;
  int64_t n;
  const int32_t *rows, *cols;
  float *x, *t;                   // [n][8], [n][kSelQ]
  const double *rule[kSelQ + 1];  // Duffy rules of orders 1 .. kSelQ, then the reference order
  int32_t nq[kSelQ + 1];
  double kappa;
  unsigned *flags;
};

// Order selection over the entries of near-field blocks.
struct SelectArgs {
  const int32_t *tri;
  int32_t nt;
  const double *geo;
  int64_t ldg;
  int32_t nblocks;
  const int32_t *row_ptr, *row_idx, *col_ptr, *col_idx;
  int64_t row_len, col_len;
  const int64_t *out_off;
  int8_t *orders;
  int64_t out_len;
  const void *net;                 // packed network (launch_pack_net)
  const double *tin_c, *tin_n;     // per-triangle inputs [3][ldt] (launch_tri_inputs)
  const float *tin_f;              // d, area, aspect [3][ldt]
  int64_t ldt;
  const float *range;              // device [16]: training minima, maxima of the inputs (or null)
  int32_t layer, q_plain, q_min;
  int32_t group;                   // rows of a column that share one decision (1 .. 8)
  float margin, log_tol;
  double kappa;
  unsigned *flags;
};

// Per-entry orders of the learned near-field kernel: Duffy rules of orders
// 2 .. q_max (index = order) and the order map (one byte per output entry).
struct OrderRules {
  const double *rule[BEM_MAX_ORDER + 1];
  const double *duffy[BEM_MAX_ORDER + 1];
  const int8_t *orders;
  int32_t q_max;
};

int mlp_params(int n_out);
size_t mlp_grad_scratch_floats(int n_out, int64_t n);
hipError_t launch_mlp_grad(int n_out, const float *P, int64_t n, const float *x, const float *t,
                           float *part, float *lpart, float *grad, float *loss, hipStream_t s);
hipError_t launch_mlp_adam(int64_t np, float *p, const float *g, float *m, float *v, float lr,
                           float b1, float b2, float eps, float c1, float c2, hipStream_t s);
// packed FP16 network for the matrix-core kernels (mlp_packed_bytes bytes)
size_t mlp_packed_bytes();
hipError_t launch_pack_net(int n_out, const float *P, void *packed, hipStream_t s);
hipError_t launch_tri_inputs(const double *geo, int64_t ldg, int nt, double *tc, double *tn,
                             float *tf, int64_t ldt, hipStream_t s);
hipError_t launch_mlp_forward(bool f16, int n_out, const float *P, const void *packed, int64_t n,
                              const float *x, float *y, hipStream_t s);
hipError_t launch_selector_samples(int kernel, int layer, const SampleArgs &a, hipStream_t s);
hipError_t launch_select_orders(const SelectArgs &a, int grid, hipStream_t s);
hipError_t launch_blocks_learned(int kernel, int layer, const BlockArgs &a, const OrderRules &o,
                                 size_t lds_bytes, hipStream_t s);

// rule: rule_variant of the plan's rule; the layer of each entry is in
// PersistentArgs::mode, its sub-tile shape in its BlockArgs
hipError_t launch_persistent(int kernel, bool mixed, int rule, const PersistentArgs &p,
                             size_t lds_bytes, hipStream_t s);
// before launch_persistent: the queue's head to 0, and the phase kinds of the
// blocks of every batch entry that keeps them (BlockArgs::brief; max_blocks: the
// most of one entry, 0 if none keeps any)
hipError_t launch_begin(int32_t *counter, const BlockArgs *batches, int32_t nbatch, int32_t max_blocks,
                        hipStream_t s);

hipError_t launch_green(int kernel, int side, const GreenArgs &a, int grid_y, hipStream_t s);
hipError_t launch_contract(bool cplx, const ContractArgs &a, int grid_y, hipStream_t s);
hipError_t launch_pivot_inverse(bool cplx, const PivInvArgs &a, hipStream_t s);

// launchers (bem_kernels.hip); return a hipError_t
// device address of the fixed geometry scratch of the allocation-free entry
// point on `device` (which must be current)
hipError_t noalloc_scratch(int device, double **ptr);
hipError_t launch_geometry(const bem_mesh &m, double *geo, int64_t ldg, unsigned *flags,
                           hipStream_t s);
// layer: BEM_SLP, BEM_DLP or 2, the near field of both layers in one pass
// (a.out: single layer, a.out2: double layer); rule: rule_variant
hipError_t launch_blocks(int kernel, int layer, int rule, bool coupling, bool mixed,
                         const BlockArgs &a, size_t lds_bytes, hipStream_t s);
hipError_t launch_entries(int kernel, int layer, bool mixed, const EntryArgs &a, hipStream_t s);
// sub-tile shape (rows, columns) and LDS bytes of the block kernel for a
// padded rule size within an LDS budget; false if nothing fits
bool block_tile_shape(int nq_pad, bool mixed, size_t lds_budget, int *tr, int *tc,
                      size_t *lds_bytes, bool coupling = false, bool both = false);
size_t block_lds_bytes(int nq_pad, int tr, int tc, bool mixed, bool lists = true,
                       bool both = false, int slots = 0);
// bytes that a requested sub-tile shape is limited by (bem_tune)
size_t requested_lds_bytes(int nq, int x_chunk, int tr, int tc, bool mixed, bool both);
// smaller sub-tiles (a->tc, slots) and workgroups per block (a->split) for a
// launch of few blocks
void split_blocks(BlockArgs *a, bool coupling, bool mixed, bool lists, bool both, size_t *lds_bytes);
int rule_chunk(int nq, int kernel);
// kernel variant of a rule (regular_rule, order, points) and the room of its
// column points in LDS
int rule_variant(int regular_rule, int q, int nq);
bool rule_is_duffy(int variant);
int rule_pad(int variant, int nq);

}  // namespace bem

struct bem_ctx;

namespace bem {

struct DeviceGuard {  // make the context's device current, restore on exit
  int prev = -1;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) (void)hipSetDevice(dev);
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

// shared argument checks and context helpers (bem_capi.cpp); they set the
// context's error text and return a BEM_ code
int fail(bem_ctx *ctx, int code, const std::string &msg);
int hip_fail(bem_ctx *ctx, hipError_t e, const char *where);
// hipMalloc of the library's buffers; fails when BEM_FAULT_INJECT=alloc
hipError_t dev_malloc(void **p, size_t bytes);
int check_op(bem_ctx *ctx, const bem_op *op);
int check_mesh(bem_ctx *ctx, const bem_mesh *m);
int check_blocks(bem_ctx *ctx, const bem_blocks *b, const void *out, int64_t out_len);
int get_rules(bem_ctx *ctx, const bem_op *op, const DevRules **out);
// geometry scratch of the context for nt triangles; leading dimension out
int ensure_geo(bem_ctx *ctx, int32_t nt, int64_t *ldg);
// release the device resources of the context's live plans and detach them
// (bem_plan.cpp; called by bem_destroy)
void detach_plans(bem_ctx *ctx);

}  // namespace bem

struct bem_ctx {
  int device = 0;
  size_t lds_budget = 64 * 1024;  // LDS bytes one workgroup may use
  std::string err;
  unsigned *flags = nullptr;      // device, 1 word
  double *geo = nullptr;          // device scratch
  double *noalloc_geo = nullptr;  // fixed geometry array of the allocation-free entry point
  double *dot_part = nullptr;     // device: partial sums of bem_vec_dot
  size_t geo_cap = 0;             // doubles
  float *mlp_scratch = nullptr;   // device: per-workgroup gradient partial sums
  size_t mlp_cap = 0;             // floats
  void *sel_scratch = nullptr;    // device: packed network + per-triangle selector inputs
  size_t sel_cap = 0;             // bytes
  std::map<std::tuple<int, int, int>, bem::DevRules> rules;
  std::set<bem_plan *> plans;     // live batched plans (released with the context)
};
