// Internal declarations shared by the host driver and the kernel translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <vector>

#include "msc.h"

namespace msc {

constexpr int kMaxShifts = 64;
constexpr int kBlock = 256;          // threads per workgroup for every solver kernel
constexpr int kMaxGrid = 2048;       // 256 CUs x 8 resident workgroups
constexpr int kXcds = 8;             // MI355X: 8 accelerator complex dies, one L2 each
// A "last workgroup" ticket site: eight group counters 128 bytes apart and a final one.
constexpr int kTicketStride = 32;
constexpr int kTicketSite = 9 * kTicketStride;

// Reliable updates of the complex64 phase: the host launches the update kernels every
// kRuCheck iterations; they run when the period (msc_params::reliable_every) is due, or
// when the recursive |r|^2 has dropped below kRuDelta2 times its value at the last update
// (a residual that falls fast would otherwise run far below what the complex64 operator
// can certify before the next replacement).
constexpr int kRuCheck = 10;
constexpr double kRuDelta2 = 1e-2;

// The deviation of P from its short form beyond which an iteration without the direction takes
// it up (multishift.hip).  Ordinary lattices and grids (condition up to 1e6) stay below 1e-13 in
// FP64 and 3e-4 in complex64.  Steps of a 60 x 60 grid with a penalty of 1e8 / 1e10 / 1e12 / 1e14 on
// an edge, FP64: 473 / 476 / 478 / 479, as with the direction from the start (without it at
// all 516 / 567 / 687 / none); 1e4 / 1e6 / 1e8 in complex64: 468 / 482 / 570 (none without it).
constexpr double kDevLimit64 = 1e-9, kDevLimit32 = 1e-2;
// Largest deviation of the FP64 phase of a mixed solve for which the complex64 phase, whose
// rounding is 5e8 times as large, starts without the direction.
constexpr double kDevSwitch = 2e-12;
// Head launches whose update mode is recorded for the byte model of sampled timings.
constexpr int kMaxSamples = 256;

// Steps of the all-shift update one pass over x_j and p_j may fold together.
constexpr int kMaxSteps = 8;
constexpr int kRing = kMaxSteps + 1;  // residuals kept: launch l's in slot l % kRing

// Scalar state of one multishift solve, resident in device memory.  Shift index j runs over
// the shifts sorted ascending; j = 0 is the driving shift sigma0.  No kernel waits for its
// own reduction: each workgroup stores a partial sum and the workgroups of the next kernel
// add the partials up themselves, in one fixed order, so they all obtain the same value.
//
// RotState: the state at the start of the iteration n that a launch of parity par runs,
// rot[par]; one workgroup of its last kernel writes rot[par ^ 1] while the others read.
struct RotState {
  double g, a, P;              // |r_{n-1}|^2, a_{n-1} and p_{n-1}^H (A + sigma0) p_{n-1}
  int iter;                    // n, the steps taken
  int launch;                  // the launch that takes step n (r_n lies in its ring slot)
  int halt;                    // 1: the kernels of this iteration do no work
  int m;                       // steps composed since x_j and p_j were last written
  int fresh;                   // 1: x_j and p_j were never written
  double zeta[kMaxShifts];     // zeta_j^(n)
  double zeta_prev[kMaxShifts];
  // p_j now is cp[0] p_j + sum_{k<m} cp[k+1] r_{n-m+k}; x_j gained the like with cx
  double cx[kMaxSteps + 1][kMaxShifts];
  double cp[kMaxSteps + 1][kMaxShifts];
  int active[kMaxShifts];      // shift j still updated
  int took[kMaxShifts];        // shift j took part in a composed step
};

struct SolveState {
  double sigma0;
  double tol2, sw2;  // (mixed_margin tol)^2; switch_tol^2 (0: no switch): times |b|^2
  double bnorm2;
  int max_iter, ns, freeze;
  int n_reliable;
  // replaced residual of the iteration at hand (reliable update, direction taken up): whether
  // it was, and the recursive residual's g_n; g right after the last one (or the precision
  // switch)
  int ru_flag, pad_;
  double ru_g, R_ru;
  double dev;                   // largest deviation of P from its short form (step_plan)
  double g_n, c_n;              // summed by K1 for K2 (multishift.hip)
  double s[kMaxShifts];         // sigma_j - sigma0
  int freeze_iter[kMaxShifts];
  int orig[kMaxShifts];         // caller's index of sorted shift j
  // the halted sequence: its state's index in rot, steps taken, |r|^2, tol2 |b|^2, 1 on a
  // breakdown
  int fin, iter, status, pad2_;
  double R, eps2;
  double c;                     // Re(r_n^H s_{n-1}) there
  RotState rot[2];
  // per sampled iteration (MsArgs::sample) that applied its steps: shifts listed and
  // residuals read; per phase (0: FP64, 1: complex64) the sums over all applications
  int smp_nact[kMaxSamples];
  int smp_m[kMaxSamples];
  int n_upd[2];
  int n_kept[2];
};

// Per-kernel partial-sum scratch, sized for kMaxGrid workgroups x kMaxShifts values.
struct Scratch {
  double* partial = nullptr;    // kMaxGrid * kMaxShifts doubles
  unsigned* tickets = nullptr;  // 16 counters, zero between launches
  double* res2 = nullptr;       // kMaxShifts doubles (verification output)
};

// CSR in device memory with int32 row pointers.
template <class V> struct Csr {
  const int32_t* rowptr = nullptr;
  const int32_t* col = nullptr;
  const V* val = nullptr;
};

// Sliced ELLPACK copy of a CSR matrix for the iteration SpMVs: slices of kSlice rows
// (one wavefront, one row per lane), the diagonal held apart in `diag`, the off-diagonal
// entries of a slice stored by pairs.  Entry k of lane l of slice s sits at
//   (cptr[s] + k / 2) * 2 kSlice + 2 l + (k % 2),
// so a lane reads two entries with one load and a wavefront reads whole cache lines;
// cptr[s + 1] - cptr[s] is the slice's width in pairs.  Padding entries hold 0 and a
// valid column.
constexpr int kSlice = 64;
template <class V> struct Sell {
  const int32_t* cptr = nullptr;  // nslices + 1
  const int32_t* col = nullptr;
  const V* val = nullptr;
  const V* diag = nullptr;        // n
  int32_t wp = 0;                 // > 0: every slice is wp pairs wide (cptr[s] = s wp)
  // Narrow columns (both set, or both null: then col is read).  Entry position e of pair
  // column c (e = 0, 1; c counts pair columns over all slices) has base cbase[2c + e];
  // the pair of lane l holds the two 16-bit offsets from those bases, entry 0 in the low
  // half, at col16[c kSlice + l].
  const uint32_t* col16 = nullptr;
  const int32_t* cbase = nullptr;
};

// Matrix-free staggered operator M = m + D on a periodic 4-D lattice (every extent >= 3):
// w holds W_mu(x) = eta_mu(x)/2 U_mu(x) value-major as [4][K][V] (direction, entry of the
// row-major 3x3 matrix, site with x0 fastest; K = 9, or 6 with rows = 2), so that
//   (D v)(x) = sum_mu [ W_mu(x) v(x + mu) - W_mu(x - mu)^H v(x - mu) ]
// (eta_mu does not depend on x_mu).  Row 3 s + c of M is colour c of site s.
template <class V> struct Stencil {
  const V* w = nullptr;
  int32_t rows = 3;  // rows of each link stored: 3, or 2 (SU(3): the third is rebuilt)
  int32_t L[4] = {0, 0, 0, 0};
  int64_t stride[4] = {0, 0, 0, 0};  // 1, L0, L0 L1, L0 L1 L2
  int64_t vol = 0;
  double mass = 0.0;
};

// Order in which the waves of the iteration kernels (K1 and K2 on the sliced path) visit
// the slices of 64 rows, for operators with a lattice structure: rows s1 slices apart are
// neighbours in one direction (a plane), rows s2 slices apart in the slowest one (a slab),
// and a plane is cut into tiles of cs slices.  on = 0: every workgroup sweeps one
// contiguous range of slices.
struct SweepOrder {
  int32_t s1, s2, cs, on;
};

// Device buffers of one sliced ELLPACK matrix (both value precisions share the columns).
struct SellStore {
  int64_t nslices = 0;
  int64_t pairs = 0;              // total pairs of all slices
  int32_t wp = 0;                 // common width in pairs when all slices agree, else 0
  int32_t* cptr = nullptr;
  int32_t* col = nullptr;
  double2* val64 = nullptr;
  float2* val32 = nullptr;
  double2* diag64 = nullptr;
  float2* diag32 = nullptr;
  uint32_t* col16 = nullptr;      // narrow columns, when every slice column's entries span
  int32_t* cbase = nullptr;       // less than 2^16 (else both null)
};

struct Workspace {
  size_t n = 0;
  int ns = 0;
  int prec = -1;
  // complex128: the residual ring (kRing n), u (A = M^H M: n; A given: its w, two n), s (A =
  // M^H M: n, A given: two n) and the ns directions
  void* ring = nullptr;
  void* u = nullptr;
  void* s = nullptr;
  void* pk = nullptr;
  void* ring32 = nullptr;  // complex64 copies for the second phase of a mixed solve
  void* u32 = nullptr;
  void* s32 = nullptr;
  void* pk32 = nullptr;
  double2* t64 = nullptr;   // n complex128 (reliable updates, products)
  double2* u64 = nullptr;   // 8 * n complex128 (verification SpMM chunk)
  SolveState* st = nullptr;
  int* h_halt = nullptr;    // host-coherent word: halt | switch request << 1
  int* d_halt = nullptr;    // its device address
  hipEvent_t ev[2] = {nullptr, nullptr};
};

// A host-coherent word that kernels set and the host reads after an event.
struct HaltWord {
  int* host = nullptr;
  int* dev = nullptr;       // its device address
  hipEvent_t ev[2] = {nullptr, nullptr};
};

struct BssState;

// Buffers of the batched single-shift CG (mp vectors of n each).
struct BssWorkspace {
  size_t n = 0;
  int mp = 0;
  int prec = -1;
  void* p = nullptr;
  void* t = nullptr;
  void* r = nullptr;
  void* e = nullptr;
  BssState* st = nullptr;
  int* h_halt = nullptr;    // host-coherent copy of st->halt, written by the last IK2
  int* d_halt = nullptr;    // its device address
  hipEvent_t ev[2] = {nullptr, nullptr};
};

}  // namespace msc

struct msc_op_s {
  int kind = 0;
  int64_t n = 0, nnz = 0, nnz_h = 0;
  int device = 0;
  int32_t* rowptr = nullptr;     // M (or A): int32[n+1]
  int32_t* col = nullptr;
  double2* val64 = nullptr;
  float2* val32 = nullptr;
  int32_t* rowptr_h = nullptr;   // M^H (kind MHM only)
  int32_t* col_h = nullptr;
  int32_t* perm_h = nullptr;     // entry of M^H -> entry of M
  double2* val64_h = nullptr;
  float2* val32_h = nullptr;
  std::vector<double> sigma;
  msc::Workspace ws;
  msc::BssWorkspace bws;
  msc::Scratch scratch;
  void* bcg = nullptr;           // BiCGStab-M buffers (one allocation)
  size_t bcg_bytes = 0;
  void* osb = nullptr;           // per-shift right-hand sides: guesses and tables
  size_t osb_bytes = 0;
  // real copies of the sliced matrix (built on the first real solve of a real operator)
  double* rval64 = nullptr;
  float* rval32 = nullptr;
  double* rdiag64 = nullptr;
  float* rdiag32 = nullptr;
  int real_state = 0;            // 0 not checked, 1 real (copies built), -1 not real
  void* rws = nullptr;           // real solve buffers
  size_t rws_bytes = 0;
  msc::HaltWord halt;            // of the real and the BiCGStab solve
  double2* yadj = nullptr;       // adjoint solutions, ns * n complex128
  size_t yadj_count = 0;
  double* adj_small = nullptr;   // 256 doubles: Gram sums and shift factors
  msc::SweepOrder order{0, 0, 0, 0};  // lattice structure of the rows (zeros: none found)
  msc::SweepOrder order_sites{0, 0, 0, 0};    // the same in blocks of 64 sites (links'
  msc::SweepOrder order_sites64{0, 0, 0, 0};  // kernels; complex64 and FP64 tile spans)
  int64_t rowhist[8] = {0, 0, 0, 0, 0, 0, 0, 0};  // rows by length: 0, 1, 2-3, ..., >= 64
  bool stencil = false;          // matrix-free staggered operator (links kept below)
  msc::Stencil<double2> w64;     // W_mu(x) = eta_mu(x)/2 U_mu(x), complex128 and
  msc::Stencil<float2> w32;      // complex64 copies (device memory owned by the op)
  double su3_dev = 1.0;          // largest deviation of a link from SU(3)
  bool two_rows = false;         // every link is in SU(3): the iteration reads wc64 / wc32,
  msc::Stencil<double2> wc64;    // the first two rows of each W_mu(x) (6 values), and
  msc::Stencil<float2> wc32;     // rebuilds the third from them
  bool sell = false;             // sliced ELLPACK copies built (M, and M^H for kind MHM)
  msc::SellStore sell_m, sell_mh;
};

namespace msc {

// ---- launchers implemented in the kernel translation units -------------------------
// All launchers enqueue on `s` and return hipGetLastError() of the launch.

// setup.hip
hipError_t launch_validate_csr(const int64_t* rowptr, const int32_t* col, int64_t n, int64_t nnz,
                               int* d_err, hipStream_t s);
hipError_t launch_rowptr_to32(const int64_t* in, int32_t* out, int64_t n, hipStream_t s);
// Row-length histogram (8 power-of-two buckets: 0, 1, 2-3, ..., >= 64) into hist[8].
hipError_t launch_row_hist(const int32_t* rowptr, int64_t n, unsigned long long* hist, hipStream_t s);
hipError_t launch_cast_vals(const double2* in, float2* out, int64_t nnz, hipStream_t s);
hipError_t build_adjoint(const int32_t* rowptr, const int32_t* col, int64_t n, int64_t nnz,
                         int32_t* rowptr_h, int32_t* col_h, int32_t* perm_h, hipStream_t s);
hipError_t launch_adjoint_vals(const int32_t* perm_h, const double2* val64, double2* val64_h,
                               float2* val32_h, int64_t nnz, hipStream_t s);
// Build the sliced ELLPACK copy of a CSR matrix into `out` when its padding stays small
// (slots <= 1.5 nnz + 2 kSlice per slice); *built tells whether it was.  The narrow
// columns are added when every slice column's entries span less than 2^16.  Synchronises `s`.
hipError_t build_sell(const int32_t* rowptr, const int32_t* col, const double2* val64, int64_t n,
                      int64_t nnz, SellStore& out, bool* built, hipStream_t s);
// Rewrite the values (and diagonal) of a built copy from the CSR values.
hipError_t refill_sell(const int32_t* rowptr, const int32_t* col, const double2* val64, int64_t n,
                       const SellStore& out, hipStream_t s);
void free_sell(SellStore& out);
// Matrix-free staggered operator set-up: w64 = eta/2 U from the caller's complex128
// links [4][V][3][3], stored [4][9][V], w32 = complex64 copy; and the scalar CSR of M = m + D built from
// w64 (25 entries per row, columns sorted): rowptr int64[n+1], col int32[25n],
// vals complex128[25n].
hipError_t launch_stencil_links(const double2* links, const Stencil<double2>& geo,
                                double2* w64, float2* w32, hipStream_t s);
hipError_t launch_stencil_csr(const Stencil<double2>& op, int64_t* rowptr, int32_t* col,
                              double2* vals, hipStream_t s);
// Largest deviation of the caller's links [4][V][3][3] from SU(3) over all links,
// max(|U U^H - I|, |det U - 1|) entrywise, into *dev (as the bits of a double; the
// caller zeroes it first).
hipError_t launch_su3_deviation(const double2* links, int64_t nlinks, unsigned long long* dev,
                                hipStream_t s);
// The first two rows of every W_mu(x) of the full copy w64 [4][9][V] into wc64 / wc32
// [4][6][V].
hipError_t launch_two_rows(const double2* w64, int64_t nlinks, double2* wc64, float2* wc32,
                           hipStream_t s);

// multishift.hip
struct MsArgs {
  int kind;
  int64_t n;
  int lanes;
  int grid;
  Csr<double2> m64, mh64;
  Csr<float2> m32, mh32;
  int launch, par;       // the launch, and its parity: its iteration's state is st->rot[par]
  int gd, gg;            // workgroups that leave partials of d_n (K1) and of g_n, c_n (K2)
  int sell;              // K1/K2 read the sliced ELLPACK copies below
  int64_t nslices;
  Sell<double2> s64, sh64;
  Sell<float2> s32, sh32;
  const double2* b;
  double2* x;            // caller's x, shift-major, caller order
  void* ring;            // kRing residuals of n
  void* u;               // u = M r (A = M^H M), A r (A given, CSR)
  void *w[2], *s[2];     // A given, sliced copy: w and s alternate; else s[0] alone
  void* pk;              // ns directions, sorted order
  int* hflag;            // host-coherent word: halt | switch request << 1 | direction request << 2
  int dir;               // 1: the iterations carry the direction p, in s[0], and x_0
  int resume;            // 1: the first iteration after launch_direction
  double dev_limit;      // without it: the deviation of P from which on it is taken up
  int flushed;           // 1: the composed steps were applied after the last iteration
  int ru_force;          // reliable update: 1 runs it whatever the residual
  int ru_check;          // 1: this iteration begins with a reliable update where one is due
  int stencil;           // K1 and K2 apply M and M^H from links (kind MHM, sell = 1):
                         // 0 no, 3 full links, 2 two rows per link (w64 / w32 in that form)
  SweepOrder ord;        // order of the slices, or of the links' blocks of 64 sites
  int march, m1, m2;     // links: t-slices per column of the march, and whether K1 / K2 march
  int split;             // links: a wave for each direction
  int small;             // links: the lattice fits one workgroup, which can take
  int span;              // this many iterations in one launch (0: the pair of kernels)
  Stencil<double2> w64;
  Stencil<float2> w32;
  int sample;            // slot of SolveState::smp_* for this iteration, -1: not sampled
  double2* t64;
  SolveState* st;
  Scratch sc;
};
// The grids and the march of a phase's iterations (a.gd, a.gg, a.march, a.m1, a.m2).
void prepare_iteration(int prec, MsArgs& a);
hipError_t launch_init(const MsArgs& a, hipStream_t s);
// One iteration of parity a.par, with a.ru_check after the FP64 reliable update where it is
// due; with `flush` it ends with the application of the composed steps.  ev (optional, 6
// events): start/stop pairs attached to K1, K2 and the application.
hipError_t launch_iteration(int prec, const MsArgs& a, hipStream_t s, hipEvent_t* ev, bool flush);
// The composed steps of a halted sequence.
hipError_t launch_final_flush(int prec, const MsArgs& a, hipStream_t s);
// The halted sequence goes on at a.par and a.launch (after launch_final_flush) carrying its
// direction (`load`: taken up now, from those of the shifts) and with r_n = b - ax, `ax` being
// (A + sigma0) x_0.
hipError_t launch_direction(int prec, const MsArgs& a, bool load, const double2* ax, hipStream_t s);
// Second phase of a mixed solve: copy r, s, p_j of a64 (complex128) into a32's complex64
// buffers and re-arm the state at a32.par (after launch_final_flush).
hipError_t launch_switch_to_mixed(const MsArgs& a64, const MsArgs& a32, int ns, hipStream_t s);
// FP64 true residual norms^2 of shifts [k0, k0+kc) (kc <= 8) of x into sc.res2[k0..].
hipError_t launch_verify(const MsArgs& a, const double* sigma_by_caller_index, int k0, int kc,
                         double2* u64, hipStream_t s);
// One product out = (A + shift) in (in and out may be the same buffer).
struct ApplyArgs {
  int kind, prec, lanes;
  int64_t n;
  Csr<double2> m64, mh64;
  Csr<float2> m32, mh32;
  int sell;                // FP64 may read the sliced copies below
  int64_t nslices;
  Sell<double2> s64, sh64;
  int links;               // FP64 may read the links w64 (all nine values)
  Stencil<double2> w64;
  SweepOrder ord;          // of the links' blocks of 64 sites
  const double2* in;
  double2* out;
  double shift;
  void* tmp;               // n values of the working precision
};
hipError_t launch_apply(const ApplyArgs& a, hipStream_t s);

// No-allocation apply: its temporary in a file-scope device array of this many bytes per GPU.
// It is held to n <= 2^21 rows (FP64, A = M^H M) or 2^22 (FP64 with A given; complex64), half of
// what the one temporary would allow except for A given in FP64.
constexpr size_t kNoAllocScratchBytes = size_t(64) << 20;
// Bytes of that array that one apply of n rows counts for.
size_t apply_scratch_bytes(int kind, int prec, int64_t n);
// The array's address on `device`, which must be the current device; looked up with
// hipGetSymbolAddress on the first call per device and kept.
hipError_t noalloc_scratch(int device, void** ptr);
// launch_apply with its temporary at `base` (the address noalloc_scratch
// returned); hipErrorInvalidValue when n exceeds the array.
hipError_t launch_apply_noalloc(ApplyArgs a, void* base, hipStream_t s);

// bicgstab.hip -- multishift BiCGStab for a general A (complex FP64 scalars)
constexpr int kBcgGrid = 1024;               // most workgroups of its kernels
constexpr int kBcgSteps = 4;                 // most steps of the shifts folded into one application
constexpr int kBcgRing = kBcgSteps + 1;      // r_n in slot n % kBcgRing, s_n in n % kBcgSteps
constexpr int kBcgTerms = 2 * kBcgSteps + 2; // p(s), r_0 .. r_D, s_0 .. s_{D-1}
// State at the start of iteration n (indexed by n's parity; BA writes the other one, which
// BB reads).  Shifts sorted ascending, j = 0 driving.
struct BcgRot {
  double2 rho, al, be;     // rho_n-1, al_{n-2}, be_{n-1} (in the one BB reads: of n)
  int iter, halt;          // n; 1: nothing left to do
  int m, fresh;            // steps composed so far; 1: x(s) and p(s) never written
  int check, pad_;         // 1: the BA before only summed r_n, whose step this one ends
  double2 z[kMaxShifts], zo[kMaxShifts], tau[kMaxShifts];
  // p(s) now is sum_e cp[e] term_e and x(s) gained sum_e cx[e] term_e
  double2 cx[kBcgTerms][kMaxShifts], cp[kBcgTerms][kMaxShifts];
  int active[kMaxShifts], took[kMaxShifts];  // took: part of a composed step
};
struct BcgState {
  double sigma0, tol2, bnorm2;
  double2 alpha;                     // BB -> the next BA
  int iter, max_iter, status, ns, bad, pad_;  // bad: BB found w^H v = 0 or not finite
  double s[kMaxShifts];              // sigma_j - sigma0
  double2 zn[kMaxShifts], als[kMaxShifts];    // z_{n+1}, al(s): BB -> the next BA
  int freeze_iter[kMaxShifts], orig[kMaxShifts];
  int at_end[kMaxShifts];            // still advanced when the sequence halted
  BcgRot rot[2];
};
struct BcgArgs {
  int64_t n;
  int lanes, par;
  int steps;               // steps of the shifts folded into one application, <= kBcgSteps
  Csr<double2> m;
  int sell;                // read the sliced copy
  int64_t nslices;
  Sell<double2> sm;
  const double2* b;       // right-hand side, also the shadow vector
  double2* x;             // caller's x, shift-major, caller order
  double2* r;             // kBcgRing residuals
  double2* s;             // kBcgSteps half-step residuals
  double2 *p[2], *v[2], *t;
  double2* pk;            // ns directions, sorted order
  BcgState* st;
  double* partial;        // >= 13 kBcgGrid doubles
  int* hflag;             // host-coherent word: 1 once halted
};
hipError_t launch_bcg_start(const BcgArgs& a, hipStream_t s);
hipError_t launch_bcg_iteration(const BcgArgs& a, hipStream_t s);

// real_ms.hip -- multishift CG for a real symmetric positive-definite A
template <class T> struct SellReal {
  const int32_t* cptr = nullptr;
  const int32_t* col = nullptr;
  const uint32_t* col16 = nullptr;  // narrow columns (with cbase), or null: col is read
  const int32_t* cbase = nullptr;
  int32_t wp = 0;
  const T* val = nullptr;           // real parts of the sliced copy's values
  const T* diag = nullptr;
};
constexpr int kRealGrid = 1024;          // most workgroups of its kernels
constexpr int kRealRing = kMaxSteps + 1;  // residuals kept: r_n in slot n % kRealRing
constexpr int kRealCheck = 4;            // systems verified by one launch
struct RealSigma {
  double v[kRealCheck];
};
// State at the start of iteration n's kernel (indexed by n's parity; the kernel's
// workgroup 0 writes the other one).  Shifts sorted ascending, j = 0 driving.
struct RealRot {
  double g, a, P;          // |r_{n-1}|^2, a_{n-1} and p_{n-1}.(A + sigma0) p_{n-1}
  int iter, halt;          // n; 1: nothing left to do
  int m, fresh;            // steps composed so far; 1: x and p never written
  double zeta[kMaxShifts], zeta_prev[kMaxShifts];
  // p_j now is cp[0] p_j + sum_{i<m} cp[i+1] r_i and x_j gained the like with cx, r_i the
  // residuals of the composed steps
  double cx[kMaxSteps + 1][kMaxShifts], cp[kMaxSteps + 1][kMaxShifts];
  int active[kMaxShifts], took[kMaxShifts];  // took: part of a composed step
};
struct RealState {
  double sigma0, tol2, bnorm2, R, eps2;
  double ru_g;             // |r_n|^2 of the recursive residual that RealArgs::resume replaced
  int fin;                 // the halted sequence's state in rot
  int iter, max_iter, ns, status, freeze;
  int n_upd, n_kept;       // x_j/p_j updates and residuals read by applications
  double s[kMaxShifts];
  int freeze_iter[kMaxShifts], orig[kMaxShifts];
  RealRot rot[2];
};
struct RealArgs {
  int64_t n, nslices;
  int par, steps;          // parity of the iteration; steps folded into one application
  int dir;                 // 1: the iteration carries the direction p (in s) and x_0
  int resume;              // 1: the first one after launch_real_direction
  SellReal<double> m64;
  SellReal<float> m32;
  const double* b;
  double* x;               // caller's x, shift-major, caller order (FP64 always)
  void* r;                 // kRealRing residuals; double or float by precision, as pk
  double *w[2], *s[2];
  void* pk;                // ns directions, sorted order
  RealState* st;
  double* partial;
  unsigned* tickets;       // one ticket site
  int* hflag;              // host-coherent word: 1 once halted | 4 the direction is to be taken up
};
hipError_t launch_real_extract(const double2* v64, double* r64, float* r32, int64_t count,
                               unsigned long long* imax, hipStream_t s);
hipError_t launch_real_start(int prec, const RealArgs& a, hipStream_t s);
hipError_t launch_real_iteration(int prec, const RealArgs& a, hipStream_t s);
// The halted sequence goes on at a.par with r_n = b - (A + sigma0) x_0 and its direction (`load`:
// taken up now, from the shifts').
hipError_t launch_real_direction(int prec, const RealArgs& a, bool load, hipStream_t s);
hipError_t launch_real_verify(const RealArgs& a, const double* x, const RealSigma& sg, int cnt,
                              double* out, hipStream_t s);

// osborn.hip -- a right-hand side per shift through common-residual initial guesses
constexpr int kOsbSlices = 256;  // workgroups per vector of the norm reduction
hipError_t launch_osb_divdiff(const double2* B, const int* orig, const double* inv, double2* W,
                              int m, int64_t n, hipStream_t s);
hipError_t launch_osb_sub(double2* y, const double2* t, int64_t n, hipStream_t s);
hipError_t launch_osb_combine(const double2* W, const double* w, const int* orig, double2* x,
                              int m, int64_t n, hipStream_t s);
hipError_t launch_osb_add(double2* x, const double2* d, int64_t count, hipStream_t s);
hipError_t launch_osb_norms(const double2* v, int count, int64_t n, double* partial,
                            unsigned* tickets, double* out, hipStream_t s);

// batched_cg.hip -- m <= kBssMax single-shift systems sharing one operator
constexpr int kBssMax = 16;
constexpr int kResChunk = 8;

struct BssState {
  double R[kBssMax];        // |r_j|^2 (recursive, inner)
  double a[kBssMax];        // step of system j this iteration
  double b[kBssMax];        // direction coefficient of system j
  double target2[kBssMax];  // inner stop: R_j <= target2_j
  double sigma[kBssMax];
  int active[kBssMax];
  int upd[kBssMax];         // system j was updated this iteration (e_j += a_j p_j)
  int iters[kBssMax];
  int bad[kBssMax];         // breakdown of system j
  int list[2][kBssMax];     // systems of an iteration of parity 0 / 1
  int nlist[2];
  int m, iter, max_iter, halt, k3_enable, pad_;
};

struct BssArgs {
  int kind;
  int m;                                // systems
  int lanes;                            // CSR: lanes per row
  int par;                              // parity of the iteration: it takes st->list[par]
  int64_t n;
  Csr<double2> m64, mh64;
  Csr<float2> m32, mh32;
  int sell;                             // 1: the SpMVs read the sliced ELLPACK copies
  int64_t nslices;
  Sell<double2> s64, sh64;
  Sell<float2> s32, sh32;
  int links;                            // rows per link read instead (2 or 3), 0: none
  Stencil<double2> w64;
  Stencil<float2> w32;
  void* p; void* t; void* r; void* e;   // m vectors of n, working precision, one after the other
  BssState* st;
  double* partial;                      // kMaxGrid * kBssMax
  unsigned* tickets;
  int* hflag;                           // host-coherent copy of st->halt
};

struct XPtrs {
  double2* x[kBssMax];
};

// FP64 residual r_q = f_q - (A + sig_q) x_q for q < kc (<= kResChunk) systems; writes
// |r_q|^2 to out[q] and, when r != nullptr, r (cast) into vector j0 + q of r and p and
// zero into that of e.
struct ResArgs {
  Csr<double2> m1;          // M (MHM) -- first half
  Csr<double2> m2;          // M^H (MHM) or A (HERM)
  int sell;                 // 1: read the sliced ELLPACK copies s1, s2 instead
  int64_t nslices;
  Sell<double2> s1, s2;
  int mhm;
  int64_t n;
  int64_t vol;              // > 0: r, p and e colour by colour (sites per colour), else in row order
  int kc;
  int j0;
  const double2* x[kResChunk];
  const double2* f[kResChunk];
  double sig[kResChunk];
  double2* u;               // kResChunk * n scratch (MHM)
  void* r; void* p; void* e;
  double* partial;
  unsigned* ticket;
  double* out;
};

// batched_ms.hip -- many independent multishift solves per launch
constexpr int kBatchMaxRhs = 4;
constexpr int kBatchMaxShifts = 16;
constexpr int kBatchChunkRows = 256;
constexpr int kBatchPartial = 8 * kBatchMaxRhs;  // partial sums of a chunk: two sets per wave

struct BatchState {
  // per right-hand side q: |r_n|^2, the tolerances, and of the step before a, b, P and |r|^2
  double R[kBatchMaxRhs], bnorm2[kBatchMaxRhs], eps2[kBatchMaxRhs], sw_eps2[kBatchMaxRhs];
  double a[kBatchMaxRhs], b[kBatchMaxRhs];             // this step's
  double a1[kBatchMaxRhs], P1[kBatchMaxRhs], g1[kBatchMaxRhs];
  double ru_g[kBatchMaxRhs];   // a reliable update's old |r|^2
  double c[kBatchMaxRhs];      // Re r_n^H s_{n-1}
  double dev[kBatchMaxRhs];    // largest deviation of P from its short form
  int iter[kBatchMaxRhs], halt[kBatchMaxRhs], status[kBatchMaxRhs];
  int step[kBatchMaxRhs];      // this iteration takes a step
  int ru[kBatchMaxRhs];        // r was replaced since the last step
  int m[kBatchMaxRhs];         // steps composed since x_k and p_k were last written
  int last[kBatchMaxRhs];      // ring step of the newest of them
  int n_upd[kBatchMaxRhs][2], n_kept[kBatchMaxRhs][2];  // per phase: updates, residuals read
  // per (q, sorted shift k), index q * 16 + k (k = 0: the driving system, zeta = 1)
  double zeta[kBatchMaxRhs * kBatchMaxShifts], zeta_prev[kBatchMaxRhs * kBatchMaxShifts];
  double cx[kMaxSteps + 1][kBatchMaxRhs * kBatchMaxShifts];  // the composed steps (RotState)
  double cp[kMaxSteps + 1][kBatchMaxRhs * kBatchMaxShifts];
  int active[kBatchMaxRhs * kBatchMaxShifts], freeze_iter[kBatchMaxRhs * kBatchMaxShifts];
  int took[kBatchMaxRhs * kBatchMaxShifts];
  // per system
  double s[kBatchMaxShifts];
  int orig[kBatchMaxShifts];
  double sigma0;
  int ns, nrhs, phase32, done;
  int wait;                    // until the next BF: 1 switch to complex64, 2 take the direction up
  int dir;                     // 1: the system carries its directions (in s) and its x_0
  int fresh;                   // 1: x_k and p_k were never written
  int slot;                    // steps since the phase began: r lies in ring slot slot % ring
  int max_iter, n_reliable, iters_fp64;
};

struct BatchSys {
  int kind;
  int nchunks;            // chunks of this system (kBatchPartial partial sums each)
  int64_t n;
  Csr<double2> m64, mh64;
  Csr<float2> m32, mh32;
  int sell;               // the SpMVs read the system's sliced ELLPACK copies below
  Sell<double2> s64, sh64;
  Sell<float2> s32, sh32;
  int links, links32;     // link rows read in place of a stored copy, FP64 and complex64 (2 or 3), or 0
  Stencil<double2> w64;
  Stencil<double2> v64;   // all nine values: the FP64 products of updates and verification
  Stencil<float2> w32;
  const double2* b;       // nrhs * n (rhs-major)
  double2* x;             // nrhs * ns * n (rhs-major, shift-major, caller order)
  // n x RR each: rhs-interleaved, on links rhs by rhs and colour by colour within; pk:
  // [shift][rhs][row].  The complex64 vectors but pk32 lie where the FP64 phase's lay.
  int ring;               // residual slots
  double2 *ring64, *u64, *s64v, *pk64, *ru64;
  float2 *slot32, *ring32, *u32, *s32v, *pk32;   // slot32: slot 0, ring32: the others
  BatchState* st;
  double* partial;
  unsigned* tickets;      // 4 sites
  const double* sig;      // shifts, caller's order
  double* res2;           // kMaxShifts per right-hand side
};

struct BatchArgs {
  const BatchSys* sys;
  const int4* chunks;     // (system, row0, row1, chunk index within the system)
  int nchunks;
  int nsys;
  int grid;
  int lanes;
  int rr;                 // right-hand sides per system, padded (1, 2 or 4)
  int* active_systems;    // unfinished systems in FP64 [0], in complex64 [1], with directions [2]
  int phases;             // what an iteration steps: 1 FP64, 2 complex64, 4 systems with directions
};

hipError_t launch_batch_init(const BatchArgs& a, hipStream_t s);
hipError_t launch_batch_iteration(const BatchArgs& a, bool flush, hipStream_t s);
hipError_t launch_batch_reliable(const BatchArgs& a, hipStream_t s);
// |b - (A + sigma_k) x_k|^2 of every system, right-hand side and shift into res2
hipError_t launch_batch_verify(const BatchArgs& a, int nrhs, int ns, hipStream_t s);

// grad.hip
// out[3q..3q+2] = Re<gref, g_q>, Im<gref, g_q>, |g_q|^2 for q < kc (<= 16); g shift-major.
hipError_t launch_gram(const double2* gref, const double2* g, int64_t n, int kc, double* partial,
                       unsigned* ticket, double* out, hipStream_t s);
hipError_t launch_scale_shifts(double2* y, const double* d_c, int ns, int64_t n, hipStream_t s);
// out[q] = |g_q - c_q gref|^2 for q < kc (<= 16)
hipError_t launch_diffnorm(const double2* gref, const double2* g, const double* d_c, int64_t n,
                           int kc, double* partial, unsigned* ticket, double* out, hipStream_t s);
hipError_t launch_sum_shifts(const double2* y, int ns, int64_t n, double2* out, hipStream_t s);
// grad (nnz complex128, creation order) of sum_k Re(g_k^H x_k) given x and y (shift-major);
// u, w: scratch of 4 n complex128 each (A = M^H M only).
hipError_t launch_grad_vals(int kind, int lanes, const Csr<double2>& m, const double2* x,
                            const double2* y, int64_t n, int ns, double2* u, double2* w,
                            double2* grad, hipStream_t s);

hipError_t launch_bss_iteration(int prec, const BssArgs& a, hipStream_t s);
hipError_t launch_residual(int prec, int lanes, const ResArgs& v, hipStream_t s);
hipError_t launch_accum(int prec, const BssArgs& a, const XPtrs& xp, hipStream_t s);

}  // namespace msc
