// Internal declarations shared by the HIP translation units of libbirk.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <string>
#include <vector>

#include "birk.h"
#include "birk_df32.h"

namespace birk {

constexpr int kCus = 256;   // compute units

// Longest transform a single workgroup performs in LDS (complex elements).
constexpr int kLdsMaxLog = 12;
constexpr int kLdsMax = 1 << kLdsMaxLog;
constexpr int kFftThreads = 256;

template <typename T> struct C2;
template <> struct C2<double> { using type = double2; };
template <> struct C2<float> { using type = float2; };
template <> struct C2<df32> { using type = df32c; };
template <typename T> using cplx = typename C2<T>::type;

// Index of a storage type in the per-precision table arrays: 0 double, 1 float,
// 2 double-float.
template <typename T>
constexpr int prec_index() {
  return std::is_same<T, double>::value ? 0 : std::is_same<T, float>::value ? 1 : 2;
}
constexpr int kNumPrec = 3;

// Dynamic LDS a kernel may be launched with.  The limit belongs to the kernel, not to a plan: it is
// always set to the most that any plan launches it with, so that plans on other threads cannot
// find it lowered between their own setting and launch.
template <typename F>
inline void lds_limit(F f, int most) {
  (void)hipFuncSetAttribute((const void*)f, hipFuncAttributeMaxDynamicSharedMemorySize, most);
}

// Per-instance data of the preconditioner and the solve.
struct Instance {
  int64_t Nn = 0, N = 0;
  int nx = 0;
  int64_t off = 0;      // vector offset (elements)
  int64_t joff = 0;     // per-node Jacobian offset (elements)
  int64_t jcoff = 0;    // constant Jacobian offset (elements)
  int64_t scan_off = 0; // offset into the preconditioner scan scratch (doubles)
  int64_t htab_off = 0;  // offset into htab
  double* w = nullptr;  // CC weights on the device [Nn]
};

// One component of one instance, for the per-component corrections of the b-form
// products and the endpoint row (birk_bform.hip).
struct CompDesc {
  int64_t off;       // vector offset of the component
  int64_t Nn;        // its node count
  const double* w;   // CC weights of its instance
  int64_t part;      // offset of its reduction partials
};
constexpr int kCompTiles = 256;  // most reduction tiles per component

// One instance, for the node-wise model kernels of the Newton solve (birk_newton.hip).
struct InstDesc {
  int64_t off;       // vector offset
  int64_t Nn;        // node count
  int64_t joff;      // per-node Jacobian offset
  int64_t nx;        // state count
  int64_t jcoff;     // constant Jacobian offset
  int64_t scan_off;  // offset into the preconditioner scan scratch
  const double* w;   // CC weights
};

// Four-step twiddles W_M^t = hi[t >> shift] * lo[t & (2^shift - 1)], one array pair per
// precision, shared by every transform of length M in the plan.
struct TwiddleSet {
  const void* hi[kNumPrec] = {nullptr, nullptr, nullptr};
  const void* lo[kNumPrec] = {nullptr, nullptr, nullptr};
  int shift = 0;
};

// Three-pass power-of-two product (birk_fast.hip): a run of consecutive instances with
// the same N, whose nc components are then contiguous with stride N_n.
// Tile schedule of the three-pass kernels (environment defaults, or the autotuner's
// choice per group of same-length components).
struct FastKnobs {
  int lds_kb[2] = {128, 64};  // LDS budget per workgroup of the runtime-length kernels [8-byte, 4-byte reals]
  int split = 0;              // 0: rows of the first DCT are the longer side (L2 >= L1); 1: L1 >= L2
  int tb = 0;                 // rows per pass-B tile (0: from the LDS budget; 2 or 4 in the register kernel)
  int b_threads = 512;        // workgroup size cap of the runtime-length pass B
  int xcd = 1;                // XCD-aware tile order
  int b2 = 1;                 // compile-time-length kernels where they apply
  int streams = 1;            // 2 or 3: the components run in that many parts on as many
                              // streams, so that one part's next pass fills another's tail
  int narrow = 0;             // 1: passes A and C in narrower tiles (4 columns for 8 at L1 = 2^9, 2^10; 8
                              // for the 16 of large float groups); plans of 8-byte reals start with 1
  int b3 = 1;                 // two-row pass B with the row transforms register-resident at both ends
};

struct FastGroup {
  int64_t Nn = 0, N = 0;
  int nc = 0;
  int64_t off = 0;       // vector offset of the first component
  int64_t work_off = 0;  // complex elements into work[0], work[1]
  int64_t part_off = 0;  // doubles into partials
  TwiddleSet tw;         // M = 2N
  FastKnobs kn;          // tile schedule of this group
};

// General product path (birk_dct.hip): one pair of components (2p, 2p + 1) of one
// instance.  Plain old data, copied to the device; kernels index it by pair.
struct PairDesc {
  int64_t src = 0;       // vector offset of component 2p
  int64_t Nn = 0, N = 0, L = 0, M = 0;
  int64_t work = 0;      // complex offset of this pair's slot in work[0..2]
  int64_t part = 0;      // offset of the pair's c^_0 partials (2 per block)
  int64_t slot = 0;      // complex elements of its slot: the power of two >= 3N, or M = L
  int R = 1;             // chirp convolutions: M = R 2^logM, M1 = R 2^logM1 (R = 1, 3, 5)
  int cls = 0;           // log2 of the power of two >= 3N (or of L): the tuner's class
  int logM = 0, logM1 = 0, logM2 = 0, tw_shift = 0;
  int has2 = 0;          // component 2p + 1 exists
  int nblk = 0;          // 256-wide blocks over [0, N_n)
  const void* chirp[kNumPrec] = {nullptr, nullptr, nullptr};  // Bluestein chirp, or null (L = M)
  const void* filt[kNumPrec] = {nullptr, nullptr, nullptr};   // Bluestein filter spectrum / M
  const void* thi[kNumPrec] = {nullptr, nullptr, nullptr};    // four-step twiddles (M > kLdsMax)
  const void* tlo[kNumPrec] = {nullptr, nullptr, nullptr};
};

// Work lists of the general path.  Each launch of a phase covers every pair of every
// size: its grid is a list of tiles (pair, block) read from the device.
struct PairSet {
  std::vector<PairDesc> host;
  PairDesc* dev = nullptr;
  int2* tiles_m = nullptr;    // (pair, block of 256 over [0, M))
  int2* tiles_n = nullptr;    // (pair, block of 256 over [0, N_n))
  int2* tiles_lds = nullptr;  // (first pair, count): whole transforms of M <= kLdsMax
  int2* tiles_c4 = nullptr;   // (pair, column block) of the two-step FFTs' column passes
  int2* tiles_r4 = nullptr;   // (pair, row block) of their row pass
  int thr_c = 0, thr_r = 0;   // chirp convolutions: threads and LDS reals of a workgroup
  int lds_c = 0, lds_r = 0;
  int n_m = 0, n_n = 0, n_lds = 0, n_c4 = 0, n_r4 = 0;
  int64_t work = 0;           // complex elements needed per work buffer
  int64_t parts = 0;          // doubles of partials needed
};

// Components whose whole product runs in one workgroup's LDS (birk_lds.hip): one launch over the
// tiles (first pair, count) of pairs of one length, or over single components.
struct LdsSet {
  std::vector<PairDesc> host;
  PairDesc* dev = nullptr;
  int2* tiles = nullptr;
  int ntiles = 0;
  int nlong = 0;      // of them, at the end, those of the longest length
  int threads = 0;    // workgroup size: an eighth of the longest length, at least one wave
  int lds_reals = 0;  // dynamic LDS of a workgroup
};

// Scans of P^{-1} and P^{-T} (birk_scan.hip to n_x = kScanNx, birk_wide.hip to kWideNx): one
// instance of one n_x class.
constexpr int kScanNx = 8, kWideNx = 12;
constexpr int kWideNodes = 16, kWideGroup = 32;   // above kScanNx: nodes per round, tiles per group
struct ScanDesc {
  int64_t Nn, off, joff, jcoff;
  int64_t hoff;              // H_k kept in float (mixed solves), elements into htab
  int64_t cmap, tmap, gmap;  // chunk, tile and group maps in the scan scratch (doubles)
  const double* w;           // CC weights
  int rounds;                // nodes per tile / 64 (16 above kScanNx)
  int ntile;
};
struct ScanTiles {           // another tiling of a class: descriptors, tiles and groups as below
  ScanDesc* dev = nullptr;
  int2 *tiles = nullptr, *groups = nullptr;
  int n_tile = 0, n_group = 0;
};
struct ScanClass {
  ScanTiles four;            // one J per instance: four nodes a lane (or empty)
  int nx = 0;
  ScanDesc* dev = nullptr;
  int2* tiles = nullptr;     // (instance, tile)
  int2* groups = nullptr;    // (instance, group of 64 (32 above kScanNx) tiles)
  int2* nodes = nullptr;     // (instance, block of 256 nodes)
  int* small = nullptr;      // instances worked by one workgroup
  int n_tile = 0, n_group = 0, n_nodes = 0, n_small = 0;
  int small_waves = 0;       // waves of those workgroups
};

// Krylov vector segmentation: tiles of kSegChunk elements, each inside one instance.
constexpr int kSegChunk = 2048;
struct SegSet {
  int2* tiles = nullptr;    // (instance, chunk)
  int ntiles = 0;
  int2* ranges = nullptr;   // per instance [first tile, end tile)
  int64_t* ioff = nullptr;  // per instance vector offset
  int64_t* ilen = nullptr;  // per instance length n_x N_n
  int64_t* icol = nullptr;  // per instance first component (of the plan's)
};

}  // namespace birk

struct birk_plan {
  int device = 0;
  hipStream_t stream = nullptr;
  birk_precision prec = BIRK_F64;
  std::vector<birk::Instance> inst;
  std::vector<birk::FastGroup> fgroups;
  birk::PairSet gen[2];           // general-path pairs: [0] 2N a power of two, [1] Bluestein
  birk::LdsSet lds[2];            // pairs that fit one workgroup: [0] 2N a power of two, [1] Bluestein
  birk::LdsSet lds_even;          // single components, N = 512, 1024, 2048 (logM = log2 N)
  int noalloc_nbuf = 3;           // work buffers that birk_apply_noalloc accounts for
  std::vector<birk::ScanClass> sclass;  // its instances by n_x, up to kWideNx
  birk::SegSet seg;               // Krylov segmentation of the batch
  std::vector<void*> allocs;      // device tables owned by the plan
  int64_t total_len = 0;
  int64_t total_jnode = 0;
  int64_t total_jconst = 0;
  int64_t total_work = 0;     // complex elements per work buffer
  int64_t total_part = 0;
  int64_t total_scan = 0;
  void* work[3] = {nullptr, nullptr, nullptr};   // complex work buffers sized for double
  double* partials = nullptr;
  double* scan = nullptr;     // preconditioner scan scratch
  float* htab = nullptr;      // H_k in float (per-node J, n_x <= kScanNx; mixed plans)
  const void* lds_tw[birk::kNumPrec] = {nullptr, nullptr, nullptr};  // exp(-2 pi i t / kLdsMax)
  void* tmp_vec[4] = {nullptr, nullptr, nullptr, nullptr};  // vectors of total_len doubles
  // Krylov workspace, allocated by the first solve that needs it.
  int krylov_m = 0;
  void* krylov_Q = nullptr;   // (2m + 1) vectors of the Krylov precision (Q and Z)
  void* krylov_vec = nullptr; // 4 vectors of the Krylov precision
  double* krylov_dots = nullptr;  // [batch][2][kKryMaxDots + 1]
  double* krylov_part = nullptr;  // reduction partials [kKryMaxDots + 1][tiles]
  double* krylov_coef = nullptr;  // per instance: scale factors / combination coefficients,
                                  // followed by the counts krylov_cnt (one upload for both)
  int* krylov_cnt = nullptr;      // per instance: number of combined basis vectors
  double* krylov_gm = nullptr;    // device-side GMRES state, kGmStride doubles per instance
  double* krylov_prm = nullptr;   // per instance (active, tolerance, ||r||), then 3 flags
  void* krylov_stage = nullptr;   // pinned host staging: dots, singular flag, coefficients + counts
  int* flag = nullptr;            // device flag: singular pivot seen
  birk::CompDesc* comps = nullptr;  // component table (device), one entry per component
  int64_t ncomp = 0;
  int64_t max_nn = 0;               // longest component
  birk::InstDesc* idesc = nullptr;  // instance table (device)
  int2* pfwd_tiles = nullptr;       // P y tiles: (instance, component * tiles + tile)
  int pfwd_ntiles = 0;
  int2* pfwd_pairs = nullptr;       // P y scans: (instance, component)
  int pfwd_npairs = 0;
  int2* pfwd_btiles = nullptr;      // P y, all components at once: (instance, tile)
  int pfwd_nbtiles = 0;
  int pfwd_maxnx = 0;               // largest n_x of the plan
  int pfwd_unx = 0;                 // the n_x every instance shares, else 0
  void* newton_buf = nullptr;       // Newton workspace, allocated by the first Newton solve
  void* kkt_buf = nullptr;          // KKT / MINRES workspace, allocated by the first KKT solve
  double* comp_val = nullptr;       // one double per component (last node, or a total)
  double* comp_part = nullptr;      // per-component reduction partials (CompDesc::part)
  int use_fast = 1;               // power-of-two N takes the three-pass path
  birk::FastKnobs fast_kn;        // default tile schedule of the three-pass groups
  int blu_split = 0;              // nominal log2 M1 of the chirp convolutions (0: by length)
  // HIP graphs of the products (birk_plan_set_graphs), per (direction, input, output)
  struct GraphSlot {
    int transpose;
    const void* v;
    void* out;
    hipGraphExec_t exec;  // null until the second use of the triple
    uint64_t used;
  };
  int use_graphs = 0;
  std::vector<GraphSlot> graphs;
  // HIP graphs of GMRES chunks (graph mode): Arnoldi steps [j0, j0 + k) for one precision,
  // restart length, Jacobian pointer and kind, preconditioner setting and J z storage
  struct KryGraph {
    int prec, j0, k, m;
    const double* J;
    int jk, use_precond, keep_jz, cached;
    hipGraphExec_t exec;
  };
  std::vector<KryGraph> kgraphs;
  uint64_t graph_clock = 0;
  // extra streams and their fork / join events of the multi-stream three-pass schedule
  static constexpr int kExtraStreams = 2;
  hipStream_t xstream[kExtraStreams] = {nullptr, nullptr};
  hipEvent_t ev_fork = nullptr;
  hipEvent_t ev_join[kExtraStreams] = {nullptr, nullptr};
};

namespace birk {

// ---- products (birk_dct.hip) ----
template <typename T>
hipError_t apply_product(birk_plan* p, const T* v, T* out, int transpose, hipStream_t s);

// Lay out the general-path pairs and the fast groups of a plan, with their table needs;
// called once at plan creation, before any allocation of work buffers.
void plan_products(birk_plan* p);
// Allocate and fill every transform table and work list (after the work buffers exist).
hipError_t build_tables(birk_plan* p);

// A device array of the plan (in p->allocs) holding a copy of `bytes` host bytes.
hipError_t upload_raw(birk_plan* p, const void* h, size_t bytes, void** d);

// ---- chirp convolutions beyond one workgroup (birk_blu.hip) ----
// R and logM of the pair's convolution length; its two-step split from the nominal log2 M1
// x (and back); whether the kernels cover x; the split a pair starts with.
void blu_length(PairDesc& d, birk_precision prec);
void blu_set_split(PairDesc& d, int x);
int blu_split(const PairDesc& d);
bool blu_split_ok(const PairDesc& d, int x);
int blu_default_split(const PairDesc& d);
// Tile lists, launch sizes and descriptors of a set on the device, and their release.
hipError_t blu_lists(birk_plan* p, PairSet& ps);
void blu_free_lists(birk_plan* p, PairSet& ps);
hipError_t blu_filters(birk_plan* p, const PairSet& ps, hipStream_t s);
template <typename T>
hipError_t product_blu(birk_plan* p, const PairSet& ps, const T* v, T* out, int transpose, hipStream_t s);

// ---- whole products in LDS (birk_lds.hip) ----
// Sort the set's pairs by length and upload its descriptors and tile list.
hipError_t finalize_lds(birk_plan* p, LdsSet& ls);
hipError_t finalize_lds_even(birk_plan* p, LdsSet& ls);
template <typename T>
hipError_t product_lds(birk_plan* p, const T* v, T* out, int transpose, hipStream_t s);

// ---- power-of-two three-pass path (birk_fast.hip) ----
bool fast_eligible(int64_t N);
template <typename T>
hipError_t fast_product(birk_plan* p, const FastGroup& g, const T* v, T* out, int transpose, hipStream_t s);
void fast_sizes(const birk_plan* p, int64_t N, int nc, int64_t* work, int64_t* part);
// Autotuner of the three-pass groups (birk_plan_tune); appends a summary to *report.
hipError_t tune_fast(birk_plan* p, hipStream_t s, std::string* report);
// Autotuner of the general path: the two-step split of each Bluestein size (birk_dct.hip).
hipError_t tune_general(birk_plan* p, hipStream_t s, std::string* report);

// ---- b-form corrections and the endpoint row (birk_bform.hip) ----
// Build the component table and its partial-sum scratch (after the weights exist).
hipError_t plan_bform(birk_plan* p);
// out[c][k] -= out[c][N] for every component c (B^a v -> B^b v).
template <typename T>
hipError_t bform_correct(birk_plan* p, T* out, hipStream_t s);
// Partial sums of every component of g, kept for bform_correct_T.
template <typename T>
hipError_t bform_sums(birk_plan* p, const T* g, hipStream_t s);
// out[c][k] -= w_k (1^T g_c) from the sums of bform_sums (B^aT g -> B^bT g).
template <typename T>
hipError_t bform_correct_T(birk_plan* p, T* out, hipStream_t s);
// xb[c] = xa[c] + w^T v_c.
template <typename T>
hipError_t endpoint(birk_plan* p, const double* xa, const T* v, double* xb, hipStream_t s);

// ---- Newton solve of the nonlinear IVP (birk_newton.hip) ----
hipError_t plan_instances(birk_plan* p);
// Two-body right-hand side F and per-node Jacobian J (either may be null), n_x = 6.
hipError_t two_body(birk_plan* p, double mu, double scale, const double* X, double* F, double* J, hipStream_t s);

// ---- preconditioner and Jacobian products (birk_solve.hip) ----
template <typename T>
hipError_t jac_times(birk_plan* p, int jac_kind, const double* J, const T* x, T* y,
                     hipStream_t s);
// J x, or J^T x, of the instances with n_x > kWideNx (part of jac_times and jac_t_times).
template <typename T, bool TRANS>
hipError_t jac_many(birk_plan* p, int jac_kind, const double* J, const T* x, T* y, hipStream_t s);
template <typename T>
hipError_t precond_forward(birk_plan* p, int jac_kind, const double* J, const T* y, T* out,
                           hipStream_t s);
// Build the P y work lists and the Krylov segmentation (after scan_off and the weights
// exist); allocations are recorded in p->allocs.
hipError_t plan_solve(birk_plan* p);
// ---- P^{-1} and P^{-T}, n_x <= kWideNx (birk_scan.hip, birk_wide.hip) ----
// Instances with more states get no class and are left untouched.
hipError_t plan_scan(birk_plan* p);
int64_t scan_scratch(int64_t Nn, int nx);                         // doubles
int64_t scan_htab(int64_t Nn, int nx, birk_precision prec);       // elements of the float H_k
// Float plans, per-node J, n_x <= kScanNx: H_k of this J to the plan's table (pivots checked
// into the plan's flag).
hipError_t scan_prepare(birk_plan* p, const double* J, hipStream_t s);
// out = P^{-1} y, jout (or null) = J out; cached = 1: from the H_k of scan_prepare where it
// kept them, otherwise K_k is formed from J and factored in the kernels.  flag (or null)
// receives 1 where a node's pivot is singular.
template <typename T>
hipError_t scan_inverse(birk_plan* p, int jac_kind, const double* J, const T* y, T* out, T* jout, int cached,
                        hipStream_t s, int* flag);
// out = P^{-T} y
hipError_t scan_inverse_t(birk_plan* p, int jac_kind, const double* J, const double* y, double* out, hipStream_t s);
// the n_x > kScanNx classes of the two
int wide_rounds(int64_t Nn);
template <typename T>
hipError_t wide_inverse(birk_plan* p, const ScanClass& sc, int per_node, const double* J, const T* y, T* out, T* jout,
                        int* flag, hipStream_t s);
hipError_t wide_inverse_t(birk_plan* p, const ScanClass& sc, int per_node, const double* J, const double* y,
                          double* out, hipStream_t s);

// ---- Krylov passes (birk_krylov.hip) ----
// Reductions accumulate in double.
constexpr int kKryMaxDots = 32;
// Device-side GMRES state per instance (doubles): rotated Hessenberg columns R
// (column-major, kGmLd rows per column), g, cos, sin, then the scalars of GM_*.
constexpr int kGmLd = kKryMaxDots + 1;
constexpr int kGmR = 0;
constexpr int kGmG = kGmLd * kKryMaxDots;
constexpr int kGmCs = kGmG + kGmLd;
constexpr int kGmSn = kGmCs + kKryMaxDots;
constexpr int kGmMisc = kGmSn + kKryMaxDots;
enum { GM_RUN, GM_ACTIVE, GM_JEND, GM_INNER, GM_STATUS, GM_TOL, GM_RNORM, kGmMiscLen };
constexpr int kGmStride = kGmMisc + kGmMiscLen + 1;
namespace kry {
template <typename T>
void sub(const T* a, const T* b, T* z, int64_t n, hipStream_t s);
// Segmented forms over every instance of the batch at once (basis vectors Q_k a plan length
// apart; per instance i results at out + i * ostride).
// norm slot of out: ||v||^2
void snorms(const birk_plan* p, const double* v, double* out, int64_t ostride, hipStream_t s);
// r = beta - x + t, norm slot of out: ||r||^2
void residual(const birk_plan* p, const double* beta, const double* x, const double* t, double* r, double* out,
              int64_t ostride, hipStream_t s);
// G = X - xa - G per component (G holds B^a F on entry); norm slot of out: ||G||^2, slot 0: ||X||^2
void ivp_residual(const birk_plan* p, const double* xa, const double* X, double* G, double* out, int64_t ostride,
                  hipStream_t s);
// Step j of GMRES from u = a - b: two Gram-Schmidt passes against q_0 .. q_j (coefficients and
// ||u||^2 in dots: two blocks of kGmLd per instance), the Hessenberg column into st, and
// whether the instance runs on into flags.  q_{j+1} = u / ||u|| follows from next_vector,
// which a next step starts with.
template <typename T>
void gram_schmidt(const birk_plan* p, T* Q, int j, const T* a, const T* b, T* u, double* dots, int64_t dstride,
                  double* st, double* flags, hipStream_t s);
template <typename T>
void next_vector(const birk_plan* p, const T* u, const double* dots, int64_t dstride, T* q, hipStream_t s);
// y = alpha[i] x
void sscale(const birk_plan* p, const double* x, double* y, const double* alpha, hipStream_t s);
// x = x0 + sum_{k < cnt[i]} c[i][k] Q0_k, and with Q1 y = y0 + the same of Q1 (x, y double, the
// sums in double; x0, y0 null: zero; x0 may be x, y0 y)
template <typename T>
void scombine(const birk_plan* p, const double* c, int64_t cstride, const int* cnt, const T* Q0, const double* x0,
              double* x, const T* Q1, const double* y0, double* y, hipStream_t s);
// Start of a GMRES cycle: q = r / ||r|| and the states, prm = (active, tolerance, ||r||) per
// instance; its end: the coefficients and their count, and what the host reads.
template <typename T>
void gm_start(const birk_plan* p, const double* r, T* q, const double* prm, double* st, hipStream_t s);
void gm_solve(const birk_plan* p, double* st, double* coef, int64_t cstride, int* cnt, double* flags, hipStream_t s);
}  // namespace kry

// ---- the KKT form and MINRES (birk_kkt.hip) ----
// y_k = J_k^T x_k per node, double.
hipError_t jac_t_times(birk_plan* p, int jac_kind, const double* J, const double* x, double* y, hipStream_t s);
// MINRES on [[H, A^T], [A, 0]] [chi; lambda] = [f; g] (h or f null: identity, zero).
birk_status kkt_solve(birk_plan* p, int jac_kind, const double* J, const double* h, const double* f,
                      const double* g, double* chi, double* lam, const birk_solve_opts* o, birk_solve_info* info);

}  // namespace birk
