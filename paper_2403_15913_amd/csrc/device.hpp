// Device-side descriptors shared by the host orchestration (api.cpp) and the
// HIP kernels (kernels.hip). Plain structs of device pointers: one PatDev per
// uploaded symbolic analysis, one InstDev per numeric instance (a factor, or
// one member of a batch). Kernels receive an array of InstDev and a work list
// of (instance, supernode) or (instance, row block) pairs, so the single
// instance, the batched and the served forms run the same kernels.
#pragma once
#include <cstdint>

#include "lds_layout.hpp"

namespace kkt {

// A pointer into device memory held in a descriptor, in the global address
// space on the device. A plain pointer loaded from memory could point
// anywhere, so its accesses would compile to flat instructions, which also
// count on the LDS counter: every LDS read behind a flat store then waits for
// the store's round trip to HBM.
#if defined(__HIP_DEVICE_COMPILE__)
#define KKT_GLOBAL __attribute__((address_space(1)))
#else
#define KKT_GLOBAL
#endif
template <class T>
struct dptr {
    KKT_GLOBAL T* p;
    dptr() = default;
    KKT_HD dptr(T* q) : p((KKT_GLOBAL T*)q) {}
    KKT_HD operator T*() const { return (T*)p; }
    KKT_HD T* operator->() const { return (T*)p; }
};

// Entries of K with more than this many products of J entries are assembled
// by a 16-lane group each instead of one thread (the symbolic analysis lists
// them once per pattern).
constexpr int kHeavyPairs = 8;
// Columns of J with more than this many entries are summed by a 16-lane group
// each in the J^T v kernels (listed once per pattern).
constexpr int kLongColumn = 8;

struct PatDev {
    int n, m, ns;
    int nlevels;
    dptr<const int> sn_col0;     // ns+1
    dptr<const int> sn_ncol;
    dptr<const int> sn_nrow;
    dptr<const int64_t> sn_rowofs;
    dptr<const int64_t> sn_lofs;
    dptr<const int64_t> sn_uofs;
    dptr<const int64_t> sn_vofs;
    dptr<const int> rows;
    dptr<const int> rel;
    dptr<const int> rel_np;
    dptr<const int> ch_ptr;
    dptr<const int> ch_list;
    dptr<const int64_t> pinv_ofs;  // per ch_list entry
    dptr<const int> pinv;          // parent update row -> child update row, or -1
    dptr<const int64_t> k_snptr;
    dptr<const int> k_loc;
    dptr<const int> k_w;
    dptr<const int> k_diag;
    dptr<const int64_t> k_pptr;
    dptr<const int> pair_a;
    dptr<const int> pair_b;
    dptr<const int> jrow;
    dptr<const int> perm;
    dptr<const int> iperm;
    dptr<const int64_t> sp_ptr;
    dptr<const int> k_csr;
    dptr<const int> sp_col;
    dptr<const int> j_ptr;
    dptr<const int> j_col;
    dptr<const int> jt_ptr;
    dptr<const int> jt_e;
    dptr<const int> jt_row;
    // J by columns in pivot order: the entries of column perm[k] are
    // jtp_ptr[k] .. jtp_ptr[k+1], with their rows and CSR entry indices
    dptr<const int> jtp_ptr;
    dptr<const int> jtp_row;
    dptr<const int> jtp_e;
    dptr<const int> jtp_long;    // pivot positions of the columns with more than kLongColumn entries
    int nlong;                   // ... and their number
    dptr<const int> j_colp;      // pivot position of the column of every CSR entry of J
};

struct RefineState {
    double omega, omega_prev, eta, eta_prev, relres, relres_prev;
    double tol;
    int maxit;
    int it;        // corrections applied so far
    int done;      // 1: stop refining this instance
    int revert;    // 1: the previous iterate is the better one
};

// what the host reads of one instance after a refinement check, written by
// the decision kernel into pinned host memory: the refinement record, the
// factor status pair and the queue schedule's error latch
struct RefineReport {
    RefineState rs;
    int status[2];
    int err;
};

// Conjugate-gradient record of one instance (eq. (schurcomp)), written by the
// instance's workgroup 0 of the kernel that takes each decision.
struct CgState {
    double rrs[2];           // r_k . r_k of iteration k in rrs[k & 1]
    double rr_new, pq, cnorm, tol;
    double eta_tol;          // > 0: also stop once the saddle system's eta bound is below it
    double norm_a;           // ||[[K0, J^T], [J, 0]]||_inf
    double norm_rhs;         // max(||f||_inf, ||g||_inf)
    double rmax, dymax;      // ||r||_inf and ||dy||_inf of the last eta test
    double eta;              // normwise backward error of (dx, dy) on the saddle system
    int it, maxit, done, status;
    int eta_stop;            // 1: stopped by the eta bound
};

// Full-system (augmented) refinement record of one instance: the backward
// errors of the current and previous iterates and the stop rule's state.
struct AugState {
    double eta, eta_prev, omega, omega_prev, tol;
    int it, maxit, done, revert;
};

// Interior-point loop record (one problem per factor)
struct IpmState {
    double mu, tau, gap, err, r1max, r4max, cn, un, ap, ad, delta, tol, sigma, tau_min;
    int it, done, status, maxit;
};

struct InstDev {
    PatDev P;
    // offsets of this instance inside the caller's concatenated arrays
    int64_t w_off, j_off, n_off, m_off;
    // numeric storage owned by the factor
    dptr<double> L;          // supernode panels, column-major, leading dimension = front rows
    dptr<double> U;          // update matrices, column-major u x u
    dptr<double> V;          // solve update vectors
    dptr<double> kval;       // assembled lower-triangle entries of K (grouped by supernode)
    dptr<double> kcsr;       // the same values in the symmetric row lists (both triangles, original rows)
    dptr<double> rpart;      // residual block maxima: 5 per residual block
    dptr<double> js;         // Lifted-KKT: J values scaled by their row's Sigma_s (HyKKT: copy of J)
    dptr<double> dinv;       // reciprocals of the pivots of L (pivot order)
    dptr<double> y;          // permuted work vector (n)
    dptr<double> r;          // residual (n)
    dptr<double> xprev;      // previous refinement iterate (n)
    dptr<double> tn;         // scratch (n)
    dptr<double> fg;         // HyKKT f_gamma in pivot order (n)
    dptr<double> cvec;       // HyKKT Schur right-hand side c (m)
    dptr<double> rvec;       // CG residual (m)
    dptr<double> pvec;       // CG direction (m)
    dptr<double> qvec;       // S_gamma p (m)
    dptr<double> pvec2;      // CG direction, second buffer (m): iterations alternate
    dptr<double> jtv;        // HyKKT: J values by columns in pivot order (jtp_ptr layout)
    dptr<double> k0csr;      // single factors: W + Sigma_x + delta I in the symmetric row lists (kcsr layout)
    dptr<double> jraw;       // Lifted-KKT, single factors: J values by rows (js holds them scaled)
    dptr<double> ssv;        // Lifted-KKT, single factors: Sigma_s (m)
    dptr<double> aug_b;      // augmented solve: condensed right-hand side (n, original numbering)
    dptr<double> aug_t;      // augmented solve: correction K^{-1} b (n)
    dptr<double> aug_e;      // augmented solve: residual (e1 n, e2 m, e4 m)
    dptr<double> aug_prev;   // augmented solve: previous iterate (dx n, ds m, dz m)
    dptr<AugState> aug;
    dptr<double> red;        // per-block partial sums (deterministic reductions)
    dptr<int> status;        // [0] latched status, [1] first failing pivot (permuted index)
    dptr<RefineState> rs;
    dptr<CgState> cg;
};

// One per front work item, in launch order: what a front's kernels read
// first, as absolute addresses, so its first data loads wait for this record
// alone instead of a chain of descriptor lookups. The first two children are
// inline; later children are read from the pattern arrays.
struct FrontDesc {
    dptr<const double> kv;       // original entries of K in the front
    dptr<const int> kl;          // their panel places (column << 16 | row)
    dptr<double> L;              // stored panel
    dptr<double> U;              // update matrix (u x u)
    dptr<double> V;              // update vector (u)
    dptr<double> y;              // work vector at the front's first column
    dptr<double> dinv;           // pivot reciprocals at the front's first column
    dptr<const int> rw;          // rows of the update part (instance numbering)
    dptr<const int> done;        // the instance's refinement stop flag
    dptr<const int> cgdone;      // the instance's CG stop flag
    dptr<const double> cU[2];    // first two children: update matrices,
    dptr<const double> cV[2];    //   update vectors,
    dptr<const int> crl[2];      //   relative rows of their update parts,
    dptr<const int> cinv[2];     //   inverse maps (this front's update row -> theirs, or -1),
    int cuc[2], cnb[2];     //   update sizes, and rows mapping into this front's columns
    int r, c, col0, nk;     // rows, columns, first column, entries of K
    int nch, ch0, inst, id; // children, first child in ch_list, instance, supernode
};

struct WorkItem {
    int inst;
    int id;   // supernode, or first row of a block
};

// one 16 x 16 tile (lower part) of a front's update matrix
struct StripItem {
    int inst;
    int id;     // supernode
    int tile;   // (row block << 16) | column block
    int item;   // the front's work item (index into the front descriptors)
};

}  // namespace kkt
