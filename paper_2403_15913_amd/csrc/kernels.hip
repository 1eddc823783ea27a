// HIP kernels for gfx950 (MI355X): the numeric phase of the Newton-step KKT
// solve (Pacaud & Shin, arXiv 2403.15913, sections "Condensed KKT system" and
// "Hybrid linear solver").
//
//   k_assemble   K = W + Sigma_x + J^T diag(d) J for every lower entry of K
//                (eq. (kkt:condensed); d = Sigma_s for Lifted-KKT, eq.
//                (liftedkkt); d = gamma for K_gamma, eq. (hykkt)).
//   k_factor     multifrontal supernodal Cholesky, one workgroup per front:
//                the front panel lives in LDS, children's update matrices are
//                extend-added in a fixed order (deterministic), then a dense
//                partial Cholesky (POTRF + TRSM) and the update-matrix SYRK.
//   k_fwd/k_bwd  supernodal triangular sweeps L y = P b and L^T z = y.
//   k_residual   r = b - K x with the normwise / componentwise backward-error
//                reductions that drive Richardson refinement.
//   CG kernels   J^T p, J t, dots and axpys of the Schur-complement CG.
//
// All arithmetic is FP64.
#include <hip/hip_runtime.h>

#include <climits>
#include <cstdint>
#include <utility>

#include "device.hpp"
#include "kernels.hpp"

namespace kkt {

#ifndef KKT_SMALL_WAVES_PER_EU
#define KKT_SMALL_WAVES_PER_EU 3
#endif
#define KKT_ST_NOT_SPD 4
#define KKT_ST_NONFINITE 5


// ---------------------------------------------------------------------------
// fills (used instead of hipMemsetAsync so the sequences stay graph-safe)
// ---------------------------------------------------------------------------
__global__ void k_fill_i32(int* __restrict__ p, int v, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// per-instance factor status pairs: (0 = ok, INT_MAX = no failing column yet)
__global__ void k_status_init(int* __restrict__ status, int ninst) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q < ninst) {
        status[2 * q] = 0;
        status[2 * q + 1] = INT_MAX;
    }
}

// segment copies: blocks (segment, part) stride over one segment each
constexpr int kCopyParts = 8;
__global__ __launch_bounds__(256) void k_copy_segments(const CopySeg* __restrict__ segs) {
    const CopySeg sg = segs[blockIdx.x / kCopyParts];
    const int part = blockIdx.x % kCopyParts;
    for (int64_t i = (int64_t)part * blockDim.x + threadIdx.x; i < sg.len; i += (int64_t)kCopyParts * blockDim.x)
        sg.dst[i] = sg.src[i];
}

// Workgroups go to the 8 XCDs in turn (workgroup b runs on XCD b mod 8) and
// every XCD has an L2 of its own. This renumbering hands each XCD one
// contiguous share of the launch's items, so neighbouring items, which read
// the same data (rows of J, a front's stored panel), meet in one L2 instead
// of being fetched into all eight.
constexpr int kNumXcd = 8;
__device__ __forceinline__ int xcd_block() {
    const int b = blockIdx.x, nb = gridDim.x;
    const int x = b % kNumXcd, q = nb / kNumXcd, rem = nb % kNumXcd;
    return x * q + min(x, rem) + b / kNumXcd;
}

// ---------------------------------------------------------------------------
// assembly: one thread per lower entry of K
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_assemble(const InstDev* __restrict__ insts, Calls C,
                                                  const WorkItem* __restrict__ items) {
    const WorkItem it = items[xcd_block()];
    const InstDev& I = insts[it.inst];
    const int64_t nnzk = I.P.k_snptr[I.P.ns];
    const int64_t e = (int64_t)it.id + threadIdx.x;
    if (e >= nnzk) return;
    const int64_t p0 = I.P.k_pptr[e], p1 = I.P.k_pptr[e + 1];
    if (p1 - p0 > kHeavyPairs) return;  // k_assemble_heavy's entry
    double v = 0.0;
    const int wi = I.P.k_w[e];
    if (wi >= 0) v += C.w[I.w_off + wi];
    const int di = I.P.k_diag[e];
    if (di >= 0) v += C.sx[I.n_off + di] + C.delta;
    const double* __restrict__ jv = C.jv + I.j_off;
    // single factors that need it keep W + Sigma_x + delta I (general HyKKT:
    // plus the inequality rows' J^T Sigma_s J, the condensed matrix K_k), for
    // the saddle-system and augmented-system residuals
    if (C.keep_k0) {
        double v0 = v;
        if (C.eqm) {
            // (J_a w) J_b with w = Sigma_s on inequality rows, 0 on equality rows
            const double* __restrict__ ss = C.ss + I.m_off;
            for (int64_t p = p0; p < p1; p++) {
                const int a = I.P.pair_a[p], r = I.P.jrow[a];
                const double w = C.eqm[r] ? 0.0 : ss[r];
                v0 += (jv[a] * w) * jv[I.P.pair_b[p]];
            }
        }
        const int c0 = I.P.k_csr[2 * e], c1 = I.P.k_csr[2 * e + 1];
        I.k0csr[c0] = v0;
        if (c1 >= 0) I.k0csr[c1] = v0;
    }
    if (C.ss) {
        // js[a] = J_a * Sigma_s[row of a] (k_jscale), so each product is
        // (J_a Sigma_s) J_b with two gathers
        const double* __restrict__ js = I.js;
        // four pairs per round: indices, then values, all loads issued before
        // the products are added in pair order
        for (int64_t p = p0; p < p1; p += 4) {
            int a[4], b[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                const int64_t pc = min(p + q, p1 - 1);
                a[q] = I.P.pair_a[pc];
                b[q] = I.P.pair_b[pc];
            }
            double x[4], y[4];
#pragma unroll
            for (int q = 0; q < 4; q++) {
                x[q] = js[a[q]];
                y[q] = jv[b[q]];
            }
#pragma unroll
            for (int q = 0; q < 4; q++)
                if (p + q < p1) v += x[q] * y[q];
        }
    } else {
        double acc = 0.0;
        for (int64_t p = p0; p < p1; p++) acc += jv[I.P.pair_a[p]] * jv[I.P.pair_b[p]];
        v += C.gamma * acc;
    }
    I.kval[e] = v;
    // row-ordered copy (both triangles) for the residual and K x
    const int c0 = I.P.k_csr[2 * e], c1 = I.P.k_csr[2 * e + 1];
    I.kcsr[c0] = v;
    if (c1 >= 0) I.kcsr[c1] = v;
    if (!isfinite(v)) atomicMax(&I.status[0], KKT_ST_NONFINITE);
}

// Entries of K with more than kHeavyPairs products: columns of J that many
// rows share (a stage's coupling variables) give a few entries long product
// lists, which would keep a whole wave of the one-thread-per-entry kernel
// looping for one lane. Here 16 lanes take one entry: lane l sums products
// l, l + 16, ... in order, then a fixed butterfly over the 16 lanes, so every
// run gives the same value.
__global__ __launch_bounds__(256) void k_assemble_heavy(const InstDev* __restrict__ insts, Calls C,
                                                        const WorkItem* __restrict__ items, int nitems) {
    const int h = blockIdx.x * 16 + (threadIdx.x >> 4), l = threadIdx.x & 15;
    if (h >= nitems) return;  // whole 16-lane groups leave together
    const WorkItem it = items[h];
    const InstDev& I = insts[it.inst];
    const int64_t e = it.id;
    const int64_t p0 = I.P.k_pptr[e], p1 = I.P.k_pptr[e + 1];
    const double* __restrict__ jv = C.jv + I.j_off;
    // Lifted-KKT: (J_a Sigma_s) J_b from k_jscale's scaled copy; K_gamma: J_a J_b
    const double* __restrict__ ja = C.ss ? I.js : jv;
    // HU products per lane and round: indices, then values, all loads issued
    // before the products are added in the lane's order
    constexpr int HU = 5;
    double acc = 0.0;
    for (int64_t p = p0 + l; p < p1; p += 16 * HU) {
        int a[HU], b[HU];
#pragma unroll
        for (int q = 0; q < HU; q++) {
            const int64_t pc = min(p + 16 * q, p1 - 1);
            a[q] = I.P.pair_a[pc];
            b[q] = I.P.pair_b[pc];
        }
        double x[HU], y[HU];
#pragma unroll
        for (int q = 0; q < HU; q++) {
            x[q] = ja[a[q]];
            y[q] = jv[b[q]];
        }
#pragma unroll
        for (int q = 0; q < HU; q++)
            if (p + 16 * q < p1) acc += x[q] * y[q];
    }
    // general HyKKT, single factors: the inequality rows' part alone, for K_k
    double accH = 0.0;
    if (C.eqm && C.keep_k0) {
        const double* __restrict__ ss = C.ss + I.m_off;
        for (int64_t p = p0 + l; p < p1; p += 16) {
            const int a = I.P.pair_a[p], r = I.P.jrow[a];
            const double w = C.eqm[r] ? 0.0 : ss[r];
            accH += (jv[a] * w) * jv[I.P.pair_b[p]];
        }
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        acc += __shfl_xor(acc, o, 16);
        accH += __shfl_xor(accH, o, 16);
    }
    if (l != 0) return;
    double v = 0.0;
    const int wi = I.P.k_w[e];
    if (wi >= 0) v += C.w[I.w_off + wi];
    const int di = I.P.k_diag[e];
    if (di >= 0) v += C.sx[I.n_off + di] + C.delta;
    const int c0 = I.P.k_csr[2 * e], c1 = I.P.k_csr[2 * e + 1];
    if (C.keep_k0) {
        I.k0csr[c0] = v + accH;
        if (c1 >= 0) I.k0csr[c1] = v + accH;
    }
    v += C.ss ? acc : C.gamma * acc;
    I.kval[e] = v;
    I.kcsr[c0] = v;
    if (c1 >= 0) I.kcsr[c1] = v;
    if (!isfinite(v)) atomicMax(&I.status[0], KKT_ST_NONFINITE);
}

// Lifted-KKT: J values scaled by their row's Sigma_s (general HyKKT: by gamma
// on the equality rows), one thread per entry
__global__ __launch_bounds__(256) void k_jscale(const InstDev* __restrict__ insts, Calls C,
                                                const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int p = it.id + threadIdx.x;
    if (p >= I.P.j_ptr[I.P.m]) return;
    const int row = I.P.jrow[p];
    const double d = (C.eqm && C.eqm[row]) ? C.gamma : C.ss[I.m_off + row];
    I.js[p] = C.jv[I.j_off + p] * d;
}

// Lifted-KKT, single factors: J's values by rows (jraw) and by columns in
// pivot order (jtv) over the entry blocks of J, or Sigma_s (rows = 1) over the
// row blocks, kept for the augmented-system solve
__global__ __launch_bounds__(256) void k_keep_lifted(const InstDev* __restrict__ insts, Calls C,
                                                     const WorkItem* __restrict__ items, int rows) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int p = it.id + threadIdx.x;
    if (rows) {
        if (p < I.P.m) I.ssv[p] = C.ss[I.m_off + p];
        return;
    }
    if (p >= I.P.j_ptr[I.P.m]) return;
    const double* __restrict__ jv = C.jv + I.j_off;
    I.jraw[p] = jv[p];
    I.jtv[p] = jv[I.P.jtp_e[p]];
}

// K_gamma: the factor keeps J's values, by rows (jraw) and by columns in pivot
// order (jtv), for the Schur-complement CG; one thread per entry
__global__ __launch_bounds__(256) void k_jcopy(const InstDev* __restrict__ insts, Calls C,
                                               const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int p = it.id + threadIdx.x;
    if (p >= I.P.j_ptr[I.P.m]) return;
    const double* __restrict__ jv = C.jv + I.j_off;
    I.jraw[p] = jv[p];
    I.jtv[p] = jv[I.P.jtp_e[p]];
}

// ---------------------------------------------------------------------------
// dense building blocks
// ---------------------------------------------------------------------------
typedef double d4 __attribute__((ext_vector_type(4)));

// v_mfma_f64_16x16x4f64 on gfx950: lane l supplies A[l%16][l/16] and
// B[l/16][l%16]; element e of the result in lane l is D[4e + l/16][l%16].
__device__ inline d4 mfma_f64_16x16x4(double a, double b, d4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

__device__ inline int rup16(int x) { return (x + 15) & ~15; }

// value of a wave-uniform lane (scalar broadcast)
__device__ inline double readlane_d(double v, int l) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, l);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// value of lane K of this lane's 16-lane row (DPP row broadcast: a
// cross-lane move inside the vector unit, no LDS round trip)
template <int K>
__device__ __forceinline__ double row_bcast(double v) {
    return __longlong_as_double(__builtin_amdgcn_mov_dpp(__double_as_longlong(v), 0x150 + K, 0xF, 0xF, false));
}

// value of the wave's first active lane, as a wave-uniform (scalar) value
__device__ inline double readfirstlane_d(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)b);
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Square root and its reciprocal of a Cholesky pivot d > 0 (finite): the
// hardware estimate of 1/sqrt(d) (relative error about 3e-8, subnormal d
// included) and one Newton step, which leaves a relative error of about
// 1.5e-15 over the whole positive range; no scaling or range test needed.
__device__ __forceinline__ void pivot_roots(const double d, double& inv, double& ljj) {
    const double t = __builtin_amdgcn_rsq(d);
    inv = fma(0.5 * t, fma(-d * t, t, 1.0), t);
    ljj = d * inv;
}

// f(integral_constant<int, I>) for I = 0 .. N-1, unrolled at compile time
template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// 16x16 tile of A B^T from a column-major panel P (leading dimension ld): A =
// rows i0..i0+15, B = rows j0..j0+15, both over columns k0..k0+15. Rows >= rlim are read clamped (their results
// are not used).
__device__ inline d4 tile_abt(const double* P, int ld, int i0, int j0, int k0, int rlim, int lane) {
    const int lr = lane & 15, lk = lane >> 4;
    const int iac = min(i0 + lr, rlim - 1), jbc = min(j0 + lr, rlim - 1);
    const double* const Lk = P + (int64_t)(k0 + lk) * ld;
    double a[4], b[4];
#pragma unroll
    for (int q = 0; q < 4; q++) {
        a[q] = Lk[4 * q * ld + iac];
        b[q] = Lk[4 * q * ld + jbc];
    }
    d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; q++) acc = mfma_f64_16x16x4(a[q], b[q], acc);
    return acc;
}

// LDS accumulation without a read-back (destinations distinct where order
// matters); cheaper than a read, an add and a write that wait for each other
__device__ __forceinline__ void lds_add(double* p, double v) {
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Empty asm that takes a value in a vector register: emits nothing, but
// keeps the optimizer from sinking a batch of loads into the predicated
// blocks that consume them (which would serialise the loads).
__device__ inline void pin(double& x) { asm volatile("" : "+v"(x)); }
__device__ inline void pin(double2& x) { asm volatile("" : "+v"(x.x), "+v"(x.y)); }
__device__ inline void pin(int& x) { asm volatile("" : "+v"(x)); }

// Copy n doubles (n even, both 16-byte aligned) with UNR independent 16-byte
// loads in flight per thread.
template <int UNR = 16>
__device__ inline void copy_vec(double* __restrict__ dst, const double* __restrict__ src, int n, int tid, int nt) {
    const double2* s2 = (const double2*)src;
    double2* d2 = (double2*)dst;
    const int n2 = n >> 1;
    // loads use a clamped (always valid) index so all UNR are issued
    // unconditionally and stay in registers; only the stores are predicated
    for (int base = tid; base < n2; base += nt * UNR) {
        double2 v[UNR];
#pragma unroll
        for (int k = 0; k < UNR; k++) v[k] = s2[min(base + k * nt, n2 - 1)];
#pragma unroll
        for (int k = 0; k < UNR; k++) pin(v[k]);
#pragma unroll
        for (int k = 0; k < UNR; k++) {
            const int q = base + k * nt;
            if (q < n2) d2[q] = v[k];
        }
    }
}

__device__ inline int even_up(int x) { return (x + 1) & ~1; }

// lower-triangular tile enumeration: t -> (ti, tj) with tj0 <= tj <= ti < nb
__device__ inline void tri_tile(int t, int tj0, int nb, int& ti, int& tj) {
    tj = tj0;
    int span = nb - tj;
    while (t >= span) { t -= span; tj++; span = nb - tj; }
    ti = tj + t;
}

// ---------------------------------------------------------------------------
// multifrontal factorisation of one front per workgroup
// ---------------------------------------------------------------------------
// The front panel (r rows x c columns) lives in LDS. It is assembled from the
// original entries of K and the children's update matrices and factored in
// 16-column blocks; the update matrix U = -L21 L21^T is formed on the matrix
// cores and the children's pass-through entries are added to it.
//
// Bound: neither flops nor bytes but the dependent steps of one front (one per
// compute unit on most levels) and the instructions each wave issues in them.
// Clocks of a 66 x 198 front (about 2.4 GHz): children added 20k, a column
// block 7k (its pivot chain 3.5k), the look-ahead update of the next column
// block 2.7k. Twelve waves rather than eight, since a wave issues at most
// every fourth cycle and the updates have that many independent tiles;
// sixteen spill (128 registers). Measured, factor launches of the paper-scale
// tree (2,001 fronts, 13 levels): eight waves with a column-major panel 702
// us, eight waves with the blocked panel 614 us, twelve 570 us, sixteen 671 us.
constexpr int kFactorThreads = 768;
constexpr int kFactorQueueThreads = 512;
// small fronts: four waves per workgroup, so several fronts share a compute
// unit. 168 registers let three do so where the LDS allows (measured on 256
// NMPC instances: factor launches 2.53 -> 2.22 ms with the blocked panel,
// 2.41 ms with two workgroups per compute unit)
constexpr int kFactorThreadsSmall = 256;
static_assert(kFactorThreads <= 1024 && kFactorThreadsSmall >= 128, "one panel wave and one update wave at least");

// A front's panel in LDS, in column blocks of 16: block kb holds the rows from
// its diagonal block down, row by row, 16 doubles each, so a lane reaches its
// row's entries, or its part of a matrix-core operand, with 16-byte accesses
// at offsets that depend on the lane alone (a wave issues one instruction
// every four cycles at best, so on a compute unit that holds one front the
// instruction count of each step is what its time goes by). Rows: the front's
// own, padded to cp, then the update rows, padded to 16; padding stays zero.
// Within a row, entry k sits at slot(k), which puts the four columns a lane
// supplies to four matrix instructions (4q + l / 16 to the q-th) side by
// side, and the row's eight 16-byte pieces are permuted by the row number, so
// that consecutive rows spread over the banks.
constexpr int kRow = kFrontRowStride;
__device__ __forceinline__ int block_base(const int kb, const int rt) { return kRow * (kb * rt - 8 * kb * (kb + 1)); }
__device__ __forceinline__ constexpr int slot(const int k) { return ((k & 3) << 2) | (k >> 2); }
__device__ __forceinline__ int in_row(const int row, const int k) { return slot(k) ^ ((row & 7) << 1); }

// Operand of one 16-row block and 16 columns: lane l holds row l % 16, columns
// 4q + l / 16 for instruction q. p: the lane's row; o: in_row of column l / 16.
struct Frag {
    double2 lo, hi;
    __device__ __forceinline__ double operator[](const int q) const {
        return q == 0 ? lo.x : q == 1 ? lo.y : q == 2 ? hi.x : hi.y;
    }
};
__device__ __forceinline__ Frag frag_load(const double* __restrict__ p, const int o) {
    Frag f;
    f.lo = *(const double2*)(p + o);
    f.hi = *(const double2*)(p + (o ^ 2));
    return f;
}

// Dense part of a front whose panel is column-major in LDS (leading dimension
// ld = r | 1): fronts taller than the panel waves can cover. The pivot chain
// by wave 0 beside the updates, then the rows below the diagonal block by all
// threads (the blocked path's arithmetic). With eight waves or more, those
// that share wave 0's SIMD (waves 4, 8) stay out of the updates beside the
// chain, so the pivot chain has its SIMD to itself.
template <class UnitF, class StoreF>
__device__ __forceinline__ void factor_tall(const InstDev& I, const FrontDesc& F, double* __restrict__ P, double* invd,
                                            const int nuu, UnitF u_unit, StoreF u_store) {
    const int c = F.c, r = F.r, ld = r | 1;
    const int cp = rup16(c), nbc = cp >> 4, nbr = rup16(r) >> 4;
    const int tid = threadIdx.x, nt = blockDim.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwave = nt >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    struct TFrag {
        double b[4], a0[4], a1[4];
    };
    // columns k0 .. k0 + 15, rows from rb (column operand) and ra (two row
    // blocks); rows past r are read clamped
    auto frag = [&](TFrag& G, const int k0, const int rb, const int ra) {
        const double* const Lk = P + (k0 + lk) * ld;
        const int ib = min(rb + lr, r - 1), i0 = min(ra + lr, r - 1), i1 = min(ra + 16 + lr, r - 1);
#pragma unroll
        for (int q = 0; q < 4; q++) {
            G.b[q] = Lk[4 * q * ld + ib];
            G.a0[q] = Lk[4 * q * ld + i0];
            G.a1[q] = Lk[4 * q * ld + i1];
        }
    };
    auto mult = [&](const TFrag& G, d4& s0, d4& s1) {
#pragma unroll
        for (int q = 0; q < 4; q++) {
            s0 = mfma_f64_16x16x4(G.b[q], G.a0[q], s0);
            s1 = mfma_f64_16x16x4(G.b[q], G.a1[q], s1);
        }
    };
    // block kb's update of the column blocks [tj0, tj1) in two-tile units t0,
    // t0 + ts, ...; columns past c are not written (they stay zero)
    auto update_units = [&](const int kb, const int tj0, const int tj1, const int t0, const int ts) {
        int tj = tj0, t = t0;
        while (tj < tj1) {
            const int nu = (nbr - tj + 1) >> 1;
            if (t >= nu) {
                t -= nu;
                tj++;
                continue;
            }
            const int ti = tj + 2 * t;
            const int row0 = (ti << 4) + lr, row1 = row0 + 16, cu0 = (tj << 4) + lk;
            const int ra0 = min(row0, r - 1), ra1 = min(row1, r - 1);
            TFrag G;
            frag(G, kb << 4, tj << 4, ti << 4);
            double p0[4], p1[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                p0[e] = P[(cu0 + 4 * e) * ld + ra0];
                p1[e] = P[(cu0 + 4 * e) * ld + ra1];
            }
            d4 s0 = {0.0, 0.0, 0.0, 0.0}, s1 = s0;
            mult(G, s0, s1);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                if (row0 < r && cu0 + 4 * e < c) P[(cu0 + 4 * e) * ld + row0] = p0[e] - s0[e];
                if (row1 < r && cu0 + 4 * e < c) P[(cu0 + 4 * e) * ld + row1] = p1[e] - s1[e];
            }
            t += ts;
        }
    };
    const bool many = nwave >= 8;
    const int upd_w = wave - 1 - (many ? wave >> 2 : 0), upd_n = many ? nwave - nwave / 4 : nwave - 1;
    for (int ph = 0;; ph++) {
        const bool la = ph & 1;
        const int kb = ph >> 1;
        const int j0 = kb << 4, w = min(16, c - j0);
        if (!la && wave == 0) {
            // Each 16-lane row of the wave holds the block, lane i of a row
            // holding row j0+i (entries right of the diagonal are never read
            // back; rows past r are zero).
            const bool live = j0 + lr < r;
            const int row = min(j0 + lr, r - 1);
            double a[16];
#pragma unroll
            for (int k = 0; k < 16; k++) a[k] = P[(j0 + k) * ld + row];
            if (!live) {
#pragma unroll
                for (int k = 0; k < 16; k++) a[k] = 0.0;
            }
            static_for<16>([&](auto J) {
                constexpr int j = J;
                if (j < w) {
                    double d = readfirstlane_d(row_bcast<j>(a[j]));
                    if (!(d > 0.0) || !isfinite(d)) {
                        if (lane == 0) {
                            int* const status = I.status;
                            atomicMin(&status[1], F.col0 + j0 + j);
                            atomicMax(&status[0], KKT_ST_NOT_SPD);
                        }
                        d = 1.0;
                    }
                    double inv, ljj;
                    pivot_roots(d, inv, ljj);
                    a[j] = lr == j ? ljj : a[j] * inv;
                    if (lane == 0) invd[j] = inv;
                    static_for<16>([&](auto K) {
                        constexpr int k = K;
                        if constexpr (k > j) a[k] = fma(-a[j], row_bcast<k>(a[j]), a[k]);
                    });
                }
            });
            if (lane < 16 && live) {
#pragma unroll
                for (int k = 0; k < 16; k++)
                    if (k < w && k <= lr) P[(j0 + k) * ld + j0 + lr] = a[k];
            }
        } else if (la || (kb > 0 && !(many && (wave & 3) == 0))) {
            update_units(la ? kb : kb - 1, kb + 1, la ? kb + 2 : nbc, la ? wave : upd_w, la ? nwave : upd_n);
        }
        __syncthreads();
        if (la) continue;
        if (tid < w) F.dinv[j0 + tid] = invd[tid];
        // rows below the diagonal block: x = p L_kk^{-T}; column j of L_kk is
        // fetched (contiguous, broadcast to all lanes) while step j-1 computes
        for (int i = j0 + 16 + tid; i < r; i += nt) {
            double x[16], lc[16], ln[16];
#pragma unroll
            for (int k = 0; k < 16; k++) x[k] = P[(j0 + k) * ld + i];
#pragma unroll
            for (int k = 0; k < 16; k++) lc[k] = P[j0 * ld + j0 + k];
#pragma unroll
            for (int j = 0; j < 16; j++) {
                if (j + 1 < 16) {
#pragma unroll
                    for (int k = 0; k < 16; k++) ln[k] = P[(j0 + j + 1) * ld + j0 + k];
                }
                if (j < w) {
                    x[j] *= invd[j];
#pragma unroll
                    for (int k = j + 1; k < 16; k++) x[k] = fma(-x[j], lc[k], x[k]);
                }
#pragma unroll
                for (int k = 0; k < 16; k++) lc[k] = ln[k];
            }
#pragma unroll
            for (int k = 0; k < 16; k++)
                if (k < w) P[(j0 + k) * ld + i] = x[k];
        }
        __syncthreads();
        if (kb + 1 == nbc) break;
    }
    // panel -> HBM: same layout, contiguous 16-byte stores
    copy_vec(F.L, P, even_up(ld * c), tid, nt);
    for (int t = wave; t < nuu; t += nwave) {
        int ti, tj;
        u_unit(t, ti, tj);
        d4 s0 = {0.0, 0.0, 0.0, 0.0}, s1 = s0;
        TFrag G;
        for (int k0 = 0; k0 < cp; k0 += 16) {
            frag(G, k0, c + (tj << 4), c + (ti << 4));
            mult(G, s0, s1);
        }
        u_store(ti, tj, s0, s1);
    }
}

// EK, EC: the first extend-add batch of a child holds EC columns per wave in
// each of EK chunks of 64 rows; US: units of the update matrix one wave
// accumulates in registers beside the panel (register budget of the caller)
template <int EK, int EC, int US>
__device__ __forceinline__ void factor_front(const InstDev& I, const FrontDesc& F, double* __restrict__ P,
                                             double* invd, const bool fused_update) {
    const int c = F.c, r = F.r;
    const int u = r - c, nch = F.nch;
    const int cp = rup16(c);
    const int ld = r | 1;  // of the stored panel
    double* __restrict__ const Lst = F.L;
    double* __restrict__ const dinv = F.dinv;
    const int tid = threadIdx.x, nt = blockDim.x;
    // the wave index as a scalar: everything derived from it is uniform
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwave = nt >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int nbc = cp >> 4, nbu = (u + 15) >> 4, nbr = nbc + nbu, rt = nbr << 4;
    // At most four waves factor a panel block (one per 64 rows below its
    // diagonal block), and at least one is left for the updates. Taller
    // fronts use a plain column-major panel (leading dimension ld).
    const int maxp = min(4, nwave - 1);
    const bool blocked = front_blocked(r, c, maxp);
    const int shift = blocked ? cp - c : 0;  // panel row of an update row: row + shift
    // place of (row, column) of the front in the LDS panel
    auto place = [&](const int row, const int col) {
        const int prow = row < c ? row : row + shift;
        return blocked ? block_base(col >> 4, rt) + prow * kRow + in_row(prow, col & 15) : col * ld + row;
    };

    // Assembly of the front: the original entries of K, then the children's
    // update matrices (entries (a, b), a >= b, whose column b maps into the
    // panel), child by child in a fixed order (two children can add into the
    // same entry). One wave takes columns wave, wave + nwave, ... of a child,
    // its lanes the rows in chunks of 64: the relative rows of a chunk are
    // loaded once and serve all of its columns (a column's own relative index
    // is a lane of the same registers), so an entry costs one load. The
    // panel is cleared and K's entries are placed while the first child's
    // loads are in flight, and a child's loads are issued before the previous
    // child is added; one copy of the code serves every child.
    struct Child {
        const double* Uc;
        const int* rl;
        int uc, nb;
    };
    // child k (0-based): the first two from the front descriptor
    auto child_at = [&](const int k) {
        Child C;
        if (k < 2) {
            C.uc = k ? F.cuc[1] : F.cuc[0];
            C.nb = k ? F.cnb[1] : F.cnb[0];
            C.Uc = k ? F.cU[1] : F.cU[0];
            C.rl = k ? F.crl[1] : F.crl[0];
        } else {
            const PatDev& T = I.P;
            const int ch = __builtin_amdgcn_readfirstlane(T.ch_list[F.ch0 + k]);
            const int cc = __builtin_amdgcn_readfirstlane(T.sn_ncol[ch]);
            C.uc = __builtin_amdgcn_readfirstlane(T.sn_nrow[ch]) - cc;
            C.nb = __builtin_amdgcn_readfirstlane(T.rel_np[ch]);
            C.Uc = I.U + T.sn_uofs[ch];
            C.rl = T.rel + T.sn_rowofs[ch] + cc;
        }
        return C;
    };
    struct ExtBatch {
        int ra[EK];        // relative rows of the first EK chunks
        double v[EK][EC];  // the wave's first EC columns there
    };
    // chunk q holds entries of column b: some row at or below the diagonal
    auto ext_has = [&](const Child& C, const int q, const int b) {
        return (q << 6) < C.uc && b < C.nb && b < (q << 6) + 64;
    };
    auto ext_load = [&](ExtBatch& B, const Child& C) {
        const double* Ub = C.Uc + (int64_t)wave * C.uc;
        const int64_t step = (int64_t)nwave * C.uc;
#pragma unroll
        for (int q = 0; q < EK; q++) B.ra[q] = C.rl[min((q << 6) + lane, C.uc - 1)];
#pragma unroll
        for (int j = 0; j < EC; j++, Ub += step) {
#pragma unroll
            for (int q = 0; q < EK; q++)
                if (ext_has(C, q, wave + j * nwave)) B.v[q][j] = Ub[min((q << 6) + lane, C.uc - 1)];
        }
    };
    // place of (relative row, relative column): a lane's row part and a
    // column part (bits 0-3 of both are combined by exclusive or)
    auto row_at = [&](const int ra) {
        const int prow = ra < c ? ra : ra + shift;
        return blocked ? prow * kRow | (prow & 7) << 1 : ra;
    };
    auto col_at = [&](const int rb) { return blocked ? block_base(rb >> 4, rt) | slot(rb & 15) : rb * ld; };
    auto place_at = [&](const int pa, const int pb) {
        return blocked ? (pa & ~15) + (pb & ~15) + ((pa ^ pb) & 15) : pa + pb;
    };
    // one entry per lane of column b, chunk q (the destinations of one child
    // are distinct, so the adds need no order among themselves)
    auto ext_one = [&](const Child& C, const int q, const int b, const int pa, const int pb, const double v) {
        const int a = (q << 6) + lane;
        if (a >= b && a < C.uc) lds_add(&P[place_at(pa, pb)], v);
    };
    auto ext_add = [&](const Child& C, const ExtBatch& B) {
        int pa[EK];
#pragma unroll
        for (int q = 0; q < EK; q++) pa[q] = row_at(B.ra[q]);
#pragma unroll
        for (int j = 0; j < EC; j++) {
            const int b = wave + j * nwave;
            // (columns of a child number at most 128)
            const int pb = col_at(__builtin_amdgcn_readlane(b < 64 ? B.ra[0] : B.ra[1], b & 63));
#pragma unroll
            for (int q = 0; q < EK; q++)
                if (ext_has(C, q, b)) ext_one(C, q, b, pa[q], pb, B.v[q][j]);
        }
        // the rest: columns past the batch, and chunks past it
        for (int q = 0; (q << 6) < C.uc; q++) {
            const int b0 = q < EK ? wave + EC * nwave : wave;
            if (!ext_has(C, q, b0)) continue;
            const int ac = min((q << 6) + lane, C.uc - 1);
            const int pq = row_at(C.rl[ac]);
            for (int b = b0; ext_has(C, q, b); b += 4 * nwave) {
                double v[4];
                int rb[4];
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    const int bj = min(b + j * nwave, C.nb - 1);
                    v[j] = C.Uc[(int64_t)bj * C.uc + ac];
                    rb[j] = C.rl[bj];
                }
#pragma unroll
                for (int j = 0; j < 4; j++)
                    if (ext_has(C, q, b + j * nwave)) ext_one(C, q, b + j * nwave, pq, col_at(rb[j]), v[j]);
            }
        }
    };
    // tall fronts: the waves take the chunks of a child instead (there are more
    // chunks than a batch holds), sixteen columns in flight
    auto ext_tall = [&](const Child& C) {
        for (int q = wave; (q << 6) < C.uc; q += nwave) {
            const int ac = min((q << 6) + lane, C.uc - 1);
            const int pq = row_at(C.rl[ac]);
            for (int b = 0; ext_has(C, q, b); b += 16) {
                double v[16];
                int rb[16];
#pragma unroll
                for (int j = 0; j < 16; j++) {
                    const int bj = min(b + j, C.nb - 1);
                    v[j] = C.Uc[(int64_t)bj * C.uc + ac];
                    rb[j] = C.rl[bj];
                }
#pragma unroll
                for (int j = 0; j < 16; j++)
                    if (ext_has(C, q, b + j)) ext_one(C, q, b + j, pq, col_at(rb[j]), v[j]);
            }
        }
    };
    {
        const int nk = F.nk;
        const int* __restrict__ kl = F.kl;
        const double* __restrict__ kv = F.kv;
        constexpr int KU = 8;
        double kvv[KU];
        int klv[KU];
#pragma unroll
        for (int k = 0; k < KU; k++) {
            const int q = max(min(tid + k * nt, nk - 1), 0);
            kvv[k] = kv[q];
            klv[k] = kl[q];
        }
        Child Cn = {}, Cc = {};
        ExtBatch Bn, Bc;
        for (int k = -1; k < nch; k++) {
            const bool next = k + 1 < nch;
            if (next) {
                Cn = child_at(k + 1);
                if (blocked && Cn.nb > 0) ext_load(Bn, Cn);
            }
            if (k < 0) {
                double2* const P2 = (double2*)P;
                const double2 z = {0.0, 0.0};
                const int n2 = (blocked ? block_base(nbc, rt) + nbc * 16 * kRow : ld * cp) >> 1;
                for (int q = tid; q < n2; q += nt) P2[q] = z;
                __syncthreads();
#pragma unroll
                for (int q = 0; q < KU; q++)
                    if (tid + q * nt < nk) P[place(klv[q] & 0xffff, klv[q] >> 16)] = kvv[q];
                for (int q = tid + KU * nt; q < nk; q += nt) {
                    const int loc = kl[q];
                    P[place(loc & 0xffff, loc >> 16)] = kv[q];
                }
            } else if (Cc.nb > 0) {
                if (blocked) ext_add(Cc, Bc);
                else ext_tall(Cc);
            }
            __syncthreads();
            Cc = Cn;
            Bc = Bn;
        }
    }

    // Update matrix U = -L21 L21^T (lower part) on the matrix cores, in units
    // of two tiles above each other; unit t is tiles (ti, tj), (ti + 1, tj) of
    // U's tile grid, column by column. Accumulators start at zero and take
    // the panel's columns in order; the children's entries that pass through
    // to U are added at the end, child by child in child order, before the
    // one store: each lane's places find a child's entry through the child's
    // inverse row map (this front's update row -> the child's, or -1).
    // Element e of a tile's result in lane l is row l % 16, column 4e + l /
    // 16: a column's rows are consecutive lanes.
    const int nuu = fused_update ? ((nbu + 1) >> 1) * ((nbu >> 1) + 1) : 0;  // sum over tj of ceil((nbu - tj) / 2)
    auto u_unit = [&](int t, int& ti, int& tj) {
        tj = 0;
        while (t >= (nbu - tj + 1) >> 1) {
            t -= (nbu - tj + 1) >> 1;
            tj++;
        }
        ti = tj + 2 * t;
    };
    auto u_store = [&](const int ti, const int tj, const d4& s0, const d4& s1) {
        const int a0 = (ti << 4) + lr, a1 = a0 + 16, b0 = (tj << 4) + lk;
        double w0[4], w1[4];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            w0[e] = -s0[e];
            w1[e] = -s1[e];
        }
        for (int k = 0; k < nch; k++) {
            const double* Uc;
            const int* inv;
            int uc;
            if (k < 2) {
                Uc = k ? F.cU[1] : F.cU[0];
                inv = k ? F.cinv[1] : F.cinv[0];
                uc = k ? F.cuc[1] : F.cuc[0];
            } else {
                const PatDev& T = I.P;
                const int ch = __builtin_amdgcn_readfirstlane(T.ch_list[F.ch0 + k]);
                Uc = I.U + T.sn_uofs[ch];
                inv = T.pinv + T.pinv_ofs[F.ch0 + k];
                uc = __builtin_amdgcn_readfirstlane(T.sn_nrow[ch]) - __builtin_amdgcn_readfirstlane(T.sn_ncol[ch]);
            }
            const int i0 = inv[min(a0, u - 1)], i1 = inv[min(a1, u - 1)];
            int ib[4];
            double v0[4], v1[4];
#pragma unroll
            for (int e = 0; e < 4; e++) ib[e] = inv[min(b0 + 4 * e, u - 1)];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                const int64_t col = (int64_t)max(ib[e], 0) * uc;
                v0[e] = Uc[col + max(i0, 0)];
                v1[e] = Uc[col + max(i1, 0)];
            }
            // (places outside U's lower part are not stored, so whatever
            // they take does not matter)
#pragma unroll
            for (int e = 0; e < 4; e++) {
                if (i0 >= 0 && ib[e] >= 0) w0[e] += v0[e];
                if (i1 >= 0 && ib[e] >= 0) w1[e] += v1[e];
            }
        }
        double* __restrict__ Us = F.U;
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int b = b0 + 4 * e;
            if (b <= a0 && a0 < u) Us[(int64_t)b * u + a0] = w0[e];
            if (b <= a1 && a1 < u) Us[(int64_t)b * u + a1] = w1[e];
        }
    };

    // Right-looking blocked Cholesky with one block of look-ahead: column
    // block kb+1 takes block kb's update first; then the panel waves factor
    // column block kb+1 while the others apply block kb's update to the
    // columns beyond it and to the update matrix. Every entry receives the
    // block updates in block order.
    if (blocked) {
        // what a lane adds to its row's address: rows here are lr, or lk + 4e,
        // modulo 16, and each panel row is lr modulo 16 as well
        const int rx = (lr & 7) << 1, fo = in_row(lr, lk);
        const int dof[2] = {in_row(lk, lr), in_row(lk + 4, lr)};
        auto npanel = [&](const int kb) { return min(maxp, max(1, (rt - (kb << 4) - 16 + 63) >> 6)); };
        // units of U below nreg live in registers of the waves that never
        // factor a panel block: unit s * ntw + (wave - np0) is slot s of a wave
        const int np0 = npanel(0), ntw = nwave - np0;
        const int nreg = min(nuu, US * ntw);
        const int ns = wave >= np0 ? (nreg - (wave - np0) + ntw - 1) / ntw : 0;  // this wave's slots
        d4 s0[US], s1[US];
        int uij[US];                  // (ti << 16) | tj
        int pa[US], pb[US];           // the operands' places in a column block
#pragma unroll
        for (int s = 0; s < US; s++) {
            s0[s] = s1[s] = d4{0.0, 0.0, 0.0, 0.0};
            uij[s] = pa[s] = pb[s] = 0;
        }
        if (ns > 0) {
#pragma unroll
            for (int s = 0; s < US; s++) {
                int ti = 0, tj = 0;
                if (s < ns) u_unit(s * ntw + wave - np0, ti, tj);
                uij[s] = (ti << 16) | tj;
                pa[s] = (cp + (ti << 4) + lr) * kRow;
                pb[s] = (cp + (tj << 4) + lr) * kRow;
            }
        }
        // Block kb's update of tiles (ti, tj), (ti + 1, tj) of the panel: the
        // result's element e in lane l is row 4e + l / 16, column l % 16. The
        // strict upper part of a diagonal tile takes values nothing reads.
        struct Unit {
            Frag b, a0, a1;
            double p0[4], p1[4];
            double* D;
            int o1;
        };
        auto unit_load = [&](Unit& X, const int kb, const int ti, const int tj) {
            const double* const Lk = P + block_base(kb, rt) + lr * kRow;
            X.o1 = ti + 1 < nbr ? 16 * kRow : 0;
            X.b = frag_load(Lk + (tj << 4) * kRow, fo);
            X.a0 = frag_load(Lk + (ti << 4) * kRow, fo);
            X.a1 = frag_load(Lk + (ti << 4) * kRow + X.o1, fo);
            X.D = P + block_base(tj, rt) + ((ti << 4) + lk) * kRow;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                X.p0[e] = X.D[4 * e * kRow + dof[e & 1]];
                X.p1[e] = X.D[4 * e * kRow + dof[e & 1] + X.o1];
            }
        };
        auto unit_store = [&](const Unit& X, const d4& t0, const d4& t1) {
            if (X.o1) {
#pragma unroll
                for (int e = 0; e < 4; e++) X.D[(4 * e + 16) * kRow + dof[e & 1]] = X.p1[e] - t1[e];
            }
#pragma unroll
            for (int e = 0; e < 4; e++) X.D[4 * e * kRow + dof[e & 1]] = X.p0[e] - t0[e];
        };
        for (int ph = 0;; ph++) {
            // even phases 2 kb: panel block kb beside the rest of block
            // kb-1's update; odd phases: block kb's update of column block kb+1
            const bool la = ph & 1;
            const int kb = ph >> 1, np = la || kb == nbc ? 0 : npanel(kb);
            if (wave < np) {
                // Column block kb of the panel in one pass: every 16-lane row
                // of a panel wave holds the diagonal block (lane i: row j0+i)
                // and runs the pivot chain on it, and each lane also carries
                // one row below the block (wave w, lane l: row
                // j0+16+64w+l). Step j scales column j and broadcasts its
                // entries of the diagonal rows across the 16-lane rows; the
                // same broadcast values serve the rank-one update of the
                // diagonal rows and the substitution step of the rows below.
                // Each entry sees the same operations in the same order as a
                // pivot chain followed by a row-by-row triangular solve.
                const int j0 = kb << 4, w = min(16, c - j0);
                const int prow = j0 + 16 + (wave << 6) + lane;
                double* const Pa = P + block_base(kb, rt) + (j0 + lr) * kRow;
                double* const Px = P + block_base(kb, rt) + (min(prow, rt - 16 + lr)) * kRow;
                double a[16], x[16];
#pragma unroll
                for (int k = 0; k < 16; k += 2) {
                    const double2 va = *(const double2*)(Pa + (k ^ rx)), vx = *(const double2*)(Px + (k ^ rx));
                    a[slot(k)] = va.x;
                    a[slot(k + 1)] = va.y;
                    x[slot(k)] = vx.x;
                    x[slot(k + 1)] = vx.y;
                }
                double myinv = 0.0;
                unsigned badv = 0;  // the same in every lane
                // No branches inside a group of four steps (a failing pivot
                // is recorded and replaced by one), so the updates of step j
                // can be scheduled alongside the pivot of step j+1; steps
                // past the last column meet zero rows and columns.
                static_for<4>([&](auto G) {
                    constexpr int g = G;
                    if (4 * g < w) {
                        static_for<4>([&](auto Q) {
                            constexpr int j = 4 * g + decltype(Q)::value;
                            const double dp = row_bcast<j>(a[j]);
                            const bool ok = dp > 0.0 && isfinite(dp);
                            badv |= ok ? 0u : 1u << j;
                            double inv, ljj;
                            pivot_roots(ok ? dp : 1.0, inv, ljj);
                            a[j] = lr == j ? ljj : a[j] * inv;
                            myinv = lr == j ? inv : myinv;
                            x[j] *= inv;
                            double lj[16];
                            static_for<16>([&](auto K) {
                                constexpr int k = K;
                                if constexpr (k > j) lj[k] = row_bcast<k>(a[j]);
                            });
                            static_for<16>([&](auto K) {
                                constexpr int k = K;
                                if constexpr (k > j) {
                                    a[k] = fma(-a[j], lj[k], a[k]);
                                    x[k] = fma(-x[j], lj[k], x[k]);
                                }
                            });
                        });
                    }
                });
                // The rows below go to LDS for the updates and to HBM; the
                // factored diagonal block to HBM only (nothing reads it here
                // again, and the other panel waves load it in this phase).
                if (prow < rt) {
#pragma unroll
                    for (int k = 0; k < 16; k += 2) {
                        double2 vx;
                        vx.x = x[slot(k)];
                        vx.y = x[slot(k + 1)];
                        *(double2*)(Px + (k ^ rx)) = vx;
                    }
                }
                double* __restrict__ const Lp = Lst + (int64_t)j0 * ld;
                const int row = prow < c ? prow : prow - shift;
                if ((prow < c || prow >= cp) && row < r) {
                    unsigned o = row;  // 32-bit offsets from a scalar base
                    if (w == 16) {
#pragma unroll
                        for (int k = 0; k < 16; k++, o += ld) Lp[o] = x[k];
                    } else {
#pragma unroll
                        for (int k = 0; k < 15; k++, o += ld)
                            if (k < w) Lp[o] = x[k];
                    }
                }
                // the diagonal block's columns, dealt to the panel waves (the
                // places above the diagonal take whatever the lane holds
                // there; nothing reads them)
                if (lane < w) {
                    const unsigned mine = ((np == 1 ? 0xffffu : np == 2 ? 0x5555u : np == 3 ? 0x9249u : 0x1111u) << wave) &
                                          ((1u << w) - 1);
                    unsigned o = j0 + lane;
#pragma unroll
                    for (int k = 0; k < 16; k++, o += ld)
                        if ((mine >> k) & 1u) Lp[o] = a[k];
                    if (wave == 0) dinv[j0 + lane] = myinv;
                }
                if (wave == 0) {
                    const unsigned bad = __builtin_amdgcn_readfirstlane(badv) & ((1u << w) - 1);
                    if (bad && lane == 0) {
                        int* const status = I.status;
                        atomicMin(&status[1], F.col0 + j0 + __builtin_ctz(bad));
                        atomicMax(&status[0], KKT_ST_NOT_SPD);
                    }
                }
            } else if (la || kb > 0) {
                // units t, t + ts, ... of the columns [kb + 1, tj1), two at a
                // time: a chain of four dependent f64 matrix instructions
                // takes about 500 cycles whatever else the SIMD does
                const int ku = la ? kb : kb - 1, tj1 = la ? kb + 2 : nbc, ts = nwave - np;
                int tj = kb + 1, t = wave - np;
                while (tj < tj1) {
                    const int nu = (nbr - tj + 1) >> 1;
                    if (t >= nu) {
                        t -= nu;
                        tj++;
                        continue;
                    }
                    Unit X, Y;
                    d4 x0 = {0.0, 0.0, 0.0, 0.0}, x1 = x0;
                    unit_load(X, ku, tj + 2 * t, tj);
                    t += ts;
                    if (t < nu) {
                        d4 y0 = {0.0, 0.0, 0.0, 0.0}, y1 = y0;
                        unit_load(Y, ku, tj + 2 * t, tj);
                        t += ts;
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            x0 = mfma_f64_16x16x4(X.a0[q], X.b[q], x0);
                            x1 = mfma_f64_16x16x4(X.a1[q], X.b[q], x1);
                            y0 = mfma_f64_16x16x4(Y.a0[q], X.b[q], y0);
                            y1 = mfma_f64_16x16x4(Y.a1[q], X.b[q], y1);
                        }
                        unit_store(X, x0, x1);
                        unit_store(Y, y0, y1);
                    } else {
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            x0 = mfma_f64_16x16x4(X.a0[q], X.b[q], x0);
                            x1 = mfma_f64_16x16x4(X.a1[q], X.b[q], x1);
                        }
                        unit_store(X, x0, x1);
                    }
                }
            }
            if (!la && kb > 0 && ns > 0) {
                // this wave's slots of U, two at a time
                const double* const Lk = P + block_base(kb - 1, rt);
#pragma unroll
                for (int s = 0; s < US; s += 2) {
                    if (s < ns) {
                        constexpr int last = US - 1;
                        const int s2 = s < last ? s + 1 : s;
                        const int xo = (uij[s] >> 16) + 1 < nbu ? 16 * kRow : 0, yo = (uij[s2] >> 16) + 1 < nbu ? 16 * kRow : 0;
                        const Frag xb = frag_load(Lk + pb[s], fo), xa0 = frag_load(Lk + pa[s], fo),
                                   xa1 = frag_load(Lk + pa[s] + xo, fo);
                        const Frag yb = frag_load(Lk + pb[s2], fo), ya0 = frag_load(Lk + pa[s2], fo),
                                   ya1 = frag_load(Lk + pa[s2] + yo, fo);
#pragma unroll
                        for (int q = 0; q < 4; q++) {
                            s0[s] = mfma_f64_16x16x4(xb[q], xa0[q], s0[s]);
                            s1[s] = mfma_f64_16x16x4(xb[q], xa1[q], s1[s]);
                            if (s < last) {
                                s0[s2] = mfma_f64_16x16x4(yb[q], ya0[q], s0[s2]);
                                s1[s2] = mfma_f64_16x16x4(yb[q], ya1[q], s1[s2]);
                            }
                        }
                    }
                }
            }
            if (!la && kb == nbc) break;
            __syncthreads();
            if (ph == 2 * nbc - 2) ph++;  // no column block follows the last
        }
#pragma unroll
        for (int s = 0; s < US; s++)
            if (s < ns) u_store(uij[s] >> 16, uij[s] & 0xffff, s0[s], s1[s]);
        // the units of U that no wave held in registers
        for (int t = nreg + wave; t < nuu; t += nwave) {
            int ti, tj;
            u_unit(t, ti, tj);
            d4 t0 = {0.0, 0.0, 0.0, 0.0}, t1 = t0;
            const int qa0 = (cp + (ti << 4) + lr) * kRow;
            const int qa1 = ti + 1 < nbu ? qa0 + 16 * kRow : qa0;
            const int qb = (cp + (tj << 4) + lr) * kRow;
            for (int kb = 0; kb < nbc; kb++) {
                const double* const Lk = P + block_base(kb, rt);
                const Frag xb = frag_load(Lk + qb, fo), xa0 = frag_load(Lk + qa0, fo), xa1 = frag_load(Lk + qa1, fo);
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    t0 = mfma_f64_16x16x4(xb[q], xa0[q], t0);
                    t1 = mfma_f64_16x16x4(xb[q], xa1[q], t1);
                }
            }
            u_store(ti, tj, t0, t1);
        }
    } else {
        factor_tall(I, F, P, invd, nuu, u_unit, u_store);
    }
    // every wave is done with the panel in LDS and with its stores before
    // the caller reuses the LDS or publishes the front
    __syncthreads();
}

__global__ __launch_bounds__(kFactorThreads) void k_factor(const InstDev* __restrict__ insts,
                                                          const FrontDesc* __restrict__ fds, int fused_update) {
    extern __shared__ __align__(16) double P[];
    __shared__ double invd[16];
    const FrontDesc& F = fds[blockIdx.x];
    factor_front<2, 6, 1>(insts[F.inst], F, P, invd, fused_update != 0);
}

// the same front factorization by four waves (every entry takes the same
// operations in the same order as in k_factor)
__global__ __launch_bounds__(kFactorThreadsSmall) __attribute__((amdgpu_waves_per_eu(KKT_SMALL_WAVES_PER_EU)))
void k_factor_small(const InstDev* __restrict__ insts, const FrontDesc* __restrict__ fds, int fused_update) {
    extern __shared__ __align__(16) double P[];
    __shared__ double invd[16];
    const FrontDesc& F = fds[blockIdx.x];
    factor_front<2, 8, 2>(insts[F.inst], F, P, invd, fused_update != 0);
}

// ---------------------------------------------------------------------------
// update matrix of a front by 16-column strips (level schedule)
// ---------------------------------------------------------------------------
// 16x16 tile of L21 L21^T read from a stored panel (column-major, leading
// dimension ld, kmax columns): the same steps as over the zero-padded LDS
// panel, with columns >= kmax contributing zeros. Rows past rlim are read
// clamped (their results are not stored).
__device__ inline d4 tile_abt_g(const double* __restrict__ Lp, int ld, int i0, int j0, int kmax, int rlim,
                                int lane) {
    const int lr = lane & 15, lk = lane >> 4;
    const int iac = min(i0 + lr, rlim - 1), jbc = min(j0 + lr, rlim - 1);
    // every column's loads are issued before the first step (kmax <= 128:
    // at most 32 steps of 4); indices past the last step repeat it, so no
    // load is predicated, and only the steps below nq run
    const int nq = (kmax + 3) >> 2;
    double a[32], b[32];
#pragma unroll
    for (int q = 0; q < 32; q++) {
        const int col = min(4 * min(q, nq - 1) + lk, kmax - 1) * ld;
        a[q] = Lp[col + iac];
        b[q] = Lp[col + jbc];
    }
    d4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 32; q++) {
        if (q < nq) {
            const bool vk = 4 * q + lk < kmax;
            acc = mfma_f64_16x16x4(vk ? a[q] : 0.0, vk ? b[q] : 0.0, acc);
        }
    }
    return acc;
}

// One wave per 16 x 16 tile of U = -L21 L21^T (lower part), on the matrix
// cores from the stored panel, with the children's update entries that pass
// through to it added in the tile epilogue. Each entry of U receives the same
// operations, in the same order, as in the factor kernel's fused path, so the
// two paths agree bitwise. (A tile per wave keeps each wave to one round trip
// for its loads and one matrix-core chain.)
constexpr int kUpdThreads = 64;
__global__ __launch_bounds__(kUpdThreads) void k_update(const InstDev* __restrict__ insts,
                                                       const FrontDesc* __restrict__ fds,
                                                       const StripItem* __restrict__ items) {
    const StripItem it = items[xcd_block()];
    const FrontDesc& F = fds[it.item];
    const InstDev& I = insts[F.inst];
    const PatDev& T = I.P;
    const int c = F.c, r = F.r;
    const int u = r - c, ld = r | 1;
    const int lane = threadIdx.x;
    const double* __restrict__ Lp = F.L;
    double* __restrict__ Us = F.U;
    const int ti = it.tile >> 16, tj = it.tile & 0xffff;
    const int nch = F.nch;
    // the children's pass-through entries of this lane's places, through
    // their inverse row maps, added in child order before the one store
    auto child_vals = [&](const int k, const int a0, const int b, double* v, bool* in) {
        const double* Uc;
        const int* inv;
        int uc;
        if (k < 2) {
            Uc = k ? F.cU[1] : F.cU[0];
            inv = k ? F.cinv[1] : F.cinv[0];
            uc = k ? F.cuc[1] : F.cuc[0];
        } else {
            const int ch = __builtin_amdgcn_readfirstlane(T.ch_list[F.ch0 + k]);
            Uc = I.U + T.sn_uofs[ch];
            inv = T.pinv + T.pinv_ofs[F.ch0 + k];
            uc = __builtin_amdgcn_readfirstlane(T.sn_nrow[ch]) - __builtin_amdgcn_readfirstlane(T.sn_ncol[ch]);
        }
        const int ib = inv[min(b, u - 1)];
        int ia[4];
#pragma unroll
        for (int e = 0; e < 4; e++) ia[e] = inv[min(a0 + 4 * e, u - 1)];
#pragma unroll
        for (int e = 0; e < 4; e++) {
            const int a = a0 + 4 * e;
            in[e] = a < u && b <= a && ia[e] >= 0 && ib >= 0;
            v[e] = Uc[(int64_t)max(ib, 0) * uc + max(ia[e], 0)];
        }
    };
    const int b = (tj << 4) + (lane & 15);
    const int a0 = (ti << 4) + (lane >> 4);
    double v0[4] = {0.0, 0.0, 0.0, 0.0}, v1[4] = {0.0, 0.0, 0.0, 0.0};
    bool in0[4] = {false, false, false, false}, in1[4] = {false, false, false, false};
    if (nch > 0) child_vals(0, a0, b, v0, in0);
    if (nch > 1) child_vals(1, a0, b, v1, in1);
    const d4 acc = tile_abt_g(Lp, ld, c + (ti << 4), c + (tj << 4), c, r, lane);
    double w[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        w[e] = -acc[e];
        if (in0[e]) w[e] += v0[e];
        if (in1[e]) w[e] += v1[e];
    }
    for (int k = 2; k < nch; k++) {
        double vk[4];
        bool ink[4];
        child_vals(k, a0, b, vk, ink);
#pragma unroll
        for (int e = 0; e < 4; e++)
            if (ink[e]) w[e] += vk[e];
    }
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int a = a0 + 4 * e;
        if (a < u && b <= a) Us[(int64_t)b * u + a] = w[e];
    }
}

// ---------------------------------------------------------------------------
// large fronts: panels too tall for a workgroup's LDS (level schedule)
// ---------------------------------------------------------------------------
// The panel is assembled and factored in place in its HBM slot by one
// workgroup per front; the update matrix is then formed by k_update's tiles,
// which read the stored panel. Each entry of the panel takes the operations
// of the LDS front kernel's non-fused path in the same order (assembly, the
// pivot chain of each diagonal block, the row-by-row solve below it, the
// blocks' updates in block order), so the factor does not depend on where
// the panel lives. Columns past the panel read as zero, as the zero-padded
// LDS panel does. Large fronts have at most 64 columns.
constexpr int kBigThreads = 256;
constexpr int kBigMaxCols = kLargeFrontCols;

// Pivot chain of diagonal block j0 (width w) of a panel in HBM, by one wave:
// lane i of each 16-lane row ends with row j0 + i of L_kk in a[0 .. i] (and
// the scaled entries of rows past the block's columns), lanes 0 .. w-1 of
// invd the pivot reciprocals; the returned mask has bit j set for a failed
// pivot j (replaced by one).
__device__ inline unsigned big_diag_chain(const double* P, int ld, int r, int j0, int w, int lane, double* a,
                                          double* invd) {
    const int i = lane & 15;
    const bool live = j0 + i < r;
    const int row = min(j0 + i, r - 1);
#pragma unroll
    for (int k = 0; k < 16; k++) a[k] = (live && k < w) ? P[(int64_t)(j0 + k) * ld + row] : 0.0;
    unsigned bad = 0;
    static_for<16>([&](auto J) {
        constexpr int j = J;
        if (j < w) {
            double d = readfirstlane_d(row_bcast<j>(a[j]));
            if (!(d > 0.0) || !isfinite(d)) {
                bad |= 1u << j;
                d = 1.0;
            }
            double inv, ljj;
            pivot_roots(d, inv, ljj);
            a[j] = i == j ? ljj : a[j] * inv;
            if (lane == 0) invd[j] = inv;
            static_for<16>([&](auto K) {
                constexpr int k = K;
                if constexpr (k > j) a[k] = fma(-a[j], row_bcast<k>(a[j]), a[k]);
            });
        }
    });
    return bad;
}

// Assembly of large fronts: workgroup (f, b, z) takes column block b and
// rows 256 z .. 256 z + 255 of large front f: zeroes that part of its
// columns, writes K's entries there, then adds the children's update entries
// that land there, child by child (the entries of one child are distinct; a
// child's update columns mapping into the block, and its update rows mapping
// into the row range, are contiguous ranges, its relative rows being
// ascending). Every entry belongs to one workgroup and takes the same
// operations in the same order as with whole columns per workgroup. Bound by
// load latency: every round trip has its loads issued together (49 -> 27 us on
// a front of 64 x 1,460 with two children).
constexpr int kBigInitRows = 256;
__global__ __launch_bounds__(kBigThreads) void k_big_init(const InstDev* __restrict__ insts,
                                                        const FrontDesc* __restrict__ fds) {
    __shared__ int cnt[2][4];
    const FrontDesc& F = fds[blockIdx.x];
    const int c = F.c, r = F.r, ld = r | 1;
    const int b0 = blockIdx.y << 4, r0 = (int)blockIdx.z * kBigInitRows;
    if (b0 >= c || r0 >= r) return;
    const int b1 = min(c, b0 + 16), r1 = min(r, r0 + kBigInitRows);
    const InstDev& I = insts[F.inst];
    const PatDev& T = I.P;
    double* const P = F.L;
    const int tid = threadIdx.x;
    constexpr int nt = kBigThreads;
    static_assert(kBigInitRows == kBigThreads, "one row per thread");
    const int row = r0 + tid;
    double* const Pr = P + (int64_t)b0 * ld + min(row, r - 1);
    if (row < r1)
        for (int j = 0; j < b1 - b0; j++) Pr[(int64_t)j * ld] = 0.0;
    __syncthreads();
    constexpr int KU = 8;  // places in flight per thread
    for (int q0 = tid; q0 < F.nk; q0 += KU * nt) {
        int loc[KU];
#pragma unroll
        for (int e = 0; e < KU; e++) loc[e] = F.kl[min(q0 + e * nt, F.nk - 1)];
#pragma unroll
        for (int e = 0; e < KU; e++) {
            const int col = loc[e] >> 16, i = loc[e] & 0xffff;
            if (q0 + e * nt < F.nk && col >= b0 && col < b1 && i >= r0 && i < r1)
                P[(int64_t)col * ld + i] = F.kv[q0 + e * nt];
        }
    }
    for (int k = 0; k < F.nch; k++) {
        const int ch = T.ch_list[F.ch0 + k];
        const int cc = T.sn_ncol[ch];
        const int uc = T.sn_nrow[ch] - cc, nb = T.rel_np[ch];
        const double* const Uc = I.U + T.sn_uofs[ch];
        const int* const rl = T.rel + T.sn_rowofs[ch] + cc;
        // child update columns e0 .. e1-1 map into columns b0 .. b1-1, its
        // update rows a0 .. a1-1 into rows r0 .. r1-1: the ascending relative
        // rows below each bound, counted by all threads (four binary searches
        // one after the other are some 40 dependent loads)
        if (tid < 4) cnt[k & 1][tid] = 0;
        __syncthreads();
        int n0 = 0, n1 = 0, n2 = 0, n3 = 0;
        for (int q0 = tid; q0 < uc; q0 += KU * nt) {
            int v[KU];
#pragma unroll
            for (int e = 0; e < KU; e++) v[e] = q0 + e * nt < uc ? rl[min(q0 + e * nt, uc - 1)] : r;
#pragma unroll
            for (int e = 0; e < KU; e++) {
                n0 += v[e] < b0 && q0 + e * nt < nb;
                n1 += v[e] < b1 && q0 + e * nt < nb;
                n2 += v[e] < r0;
                n3 += v[e] < r1;
            }
        }
        atomicAdd(&cnt[k & 1][0], n0);
        atomicAdd(&cnt[k & 1][1], n1);
        atomicAdd(&cnt[k & 1][2], n2);
        atomicAdd(&cnt[k & 1][3], n3);
        __syncthreads();
        const int e0 = cnt[k & 1][0], ne = cnt[k & 1][1] - e0, a0 = cnt[k & 1][2], a1 = cnt[k & 1][3];
        // at most one of the child's rows per thread, sixteen columns
        const int a = a0 + tid;
        if (ne > 0 && a < a1) {
            const int ra = rl[a];
            int rb[16];
            double uv[16], pv[16];
#pragma unroll
            for (int j = 0; j < 16; j++) {
                const int b = e0 + min(j, ne - 1);
                rb[j] = rl[b];
                uv[j] = Uc[(int64_t)b * uc + a];
            }
#pragma unroll
            for (int j = 0; j < 16; j++) pv[j] = P[(int64_t)rb[j] * ld + ra];
#pragma unroll
            for (int j = 0; j < 16; j++)
                if (j < ne && a >= e0 + j) P[(int64_t)rb[j] * ld + ra] = pv[j] + uv[j];
        }
        __syncthreads();
    }
}

// Rows below diagonal block kb of large fronts: workgroup (f, g) recomputes
// the block's pivot chain from the panel (every workgroup the same values),
// then solves rows j0 + 16 + 256 g + tid (x = p L_kk^{-T}, the row-by-row
// arithmetic of the LDS kernel). The factored block itself is written by
// k_big_tiles, after every workgroup here has read it.
__global__ __launch_bounds__(kBigThreads) void k_big_trsm(const FrontDesc* __restrict__ fds, int kb) {
    __shared__ double Ld[16 * 17];
    __shared__ double invd[16];
    const FrontDesc& F = fds[blockIdx.x];
    const int c = F.c, r = F.r, ld = r | 1;
    const int j0 = kb << 4;
    const int rows0 = j0 + 16 + (int)blockIdx.y * kBigThreads;
    if (j0 >= c || rows0 >= r) return;
    const int w = min(16, c - j0);
    double* const P = F.L;
    const int tid = threadIdx.x, lane = tid & 63;
    if (tid < 64) {
        double a[16];
        big_diag_chain(P, ld, r, j0, w, lane, a, invd);
        const int i = lane & 15;
        if (lane < 16) {
#pragma unroll
            for (int k = 0; k < 16; k++) Ld[k * 17 + i] = a[k];  // column k, row j0 + i
        }
    }
    __syncthreads();
    const int i = rows0 + tid;
    if (i >= r) return;
    double x[16], lc[16];
#pragma unroll
    for (int k = 0; k < 16; k++) x[k] = k < w ? P[(int64_t)(j0 + k) * ld + i] : 0.0;
#pragma unroll
    for (int j = 0; j < 16; j++) {
        if (j < w) {
#pragma unroll
            for (int k = 0; k < 16; k++) lc[k] = Ld[j * 17 + k];
            x[j] *= invd[j];
#pragma unroll
            for (int k = j + 1; k < 16; k++) x[k] = fma(-x[j], lc[k], x[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < 16; k++)
        if (k < w) P[(int64_t)(j0 + k) * ld + i] = x[k];
}

// After k_big_trsm(kb): the later column blocks of large fronts take block
// kb's update on the matrix cores, one 16 x 16 tile per wave (workgroup
// (f, h) takes tiles 4h .. 4h+3 of front f), and workgroup (f, 0) writes the
// factored diagonal block kb, its pivot reciprocals and any failed pivot.
__global__ __launch_bounds__(kBigThreads) void k_big_tiles(const InstDev* __restrict__ insts,
                                                         const FrontDesc* __restrict__ fds, int kb) {
    __shared__ double invd[16];
    const FrontDesc& F = fds[blockIdx.x];
    const int c = F.c, r = F.r, ld = r | 1;
    const int j0 = kb << 4;
    if (j0 >= c) return;
    const int w = min(16, c - j0);
    double* const P = F.L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (blockIdx.y == 0 && wave == 0) {
        double a[16];
        const unsigned bad = big_diag_chain(P, ld, r, j0, w, lane, a, invd);
        if (bad && lane == 0) {
            int* const status = insts[F.inst].status;
            atomicMin(&status[1], F.col0 + j0 + __builtin_ctz(bad));
            atomicMax(&status[0], KKT_ST_NOT_SPD);
        }
        const int i = lane & 15;
        if (lane < 16 && j0 + i < r) {
#pragma unroll
            for (int k = 0; k < 16; k++)
                if (k < w && k <= i) P[(int64_t)(j0 + k) * ld + j0 + i] = a[k];
        }
        if (lane < w) F.dinv[j0 + lane] = invd[lane];
    }
    const int nbc = (c + 15) >> 4, nbr = (r + 15) >> 4;
    if (kb + 1 >= nbc) return;
    int ntile = 0;
    for (int jt = kb + 1; jt < nbc; jt++) ntile += nbr - jt;
    const int t = (int)blockIdx.y * (kBigThreads >> 6) + wave;
    if (t >= ntile) return;
    int ti, tj;
    tri_tile(t, kb + 1, nbr, ti, tj);
    const d4 acc = tile_abt(P, ld, ti << 4, tj << 4, j0, r, lane);
    const int col = (tj << 4) + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const int row = (ti << 4) + 4 * e + (lane >> 4);
        if (col < c && row >= col && row < r) P[(int64_t)col * ld + row] -= acc[e];
    }
}

// ---------------------------------------------------------------------------
// dependency-driven (persistent) scheduling
// ---------------------------------------------------------------------------
// Workgroups take tickets in a topological order of the fronts (children
// before parents), wait until the children have published, process the
// front, release their writes at agent scope and count themselves done in
// the parent. A workgroup holding ticket t only waits for fronts with smaller
// tickets, which are held by running workgroups, so the queue always drains.
// Every wait is bounded: past the limit it latches an error and proceeds.
//
// All control flow of the persistent loops is wave-uniform. The scheduling
// steps run on wave 0 with every lane active (the test is on an SGPR), and
// only lane 0 adds to a counter, through the value it adds rather than a
// branch. A lane-divergent test such as threadIdx.x == 0 at both ends of the
// loop lets the optimizer thread the back-edge past the barriers; the loop
// then exits lane by lane and the other lanes of wave 0 re-run the body with
// the previous ticket.
constexpr long kSpinLimit = 1L << 22;

__device__ inline bool sched_wave() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) == 0; }
__device__ inline int lane0() { return (threadIdx.x & 63) == 0 ? 1 : 0; }

// called by a whole wave; the counter is read into a scalar register
__device__ inline void wait_at_least(const int* p, int v, int* err) {
    for (long spins = 0;; ++spins) {
        const int cur = __builtin_amdgcn_readfirstlane(__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (cur >= v) break;
        if (spins > kSpinLimit) {
            atomicMax(err, 1);
            break;
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// called by a whole wave; adds exactly one
__device__ inline void publish_add(int* p) {
    __hip_atomic_fetch_add(p, lane0(), __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// The ticket is broadcast through LDS and then moved to a scalar register,
// so everything derived from it (front index, sizes, loop bounds) is
// wave-uniform and every barrier below sits in uniform control flow.
__device__ inline int take_ticket(int* ticket, int* slot) {
    if (sched_wave()) {
        // lane 0 adds one; its return value is the ticket whatever the lane order
        const int old = atomicAdd(ticket, lane0());
        *slot = __builtin_amdgcn_readfirstlane(old);
    }
    __syncthreads();
    const int t = __builtin_amdgcn_readfirstlane(*slot);
    __syncthreads();
    return t;
}

__global__ __launch_bounds__(kFactorQueueThreads) void k_factor_queue(const InstDev* __restrict__ insts,
                                                                const FrontDesc* __restrict__ fds, DepLists D) {
    extern __shared__ __align__(16) double P[];
    __shared__ double invd[16];
    __shared__ int slot;
    for (;;) {
        const int t = take_ticket(D.ticket, &slot);
        if (t >= D.nitems) break;
        const int need = __builtin_amdgcn_readfirstlane(D.nchild[t]);
        const int par = __builtin_amdgcn_readfirstlane(D.parent[t]);
        if (sched_wave()) wait_at_least(D.cnt + t, need, D.err);
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const FrontDesc& F = fds[t];
        factor_front<2, 6, 4>(insts[F.inst], F, P, invd, true);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __syncthreads();
        if (sched_wave() && par >= 0) publish_add(D.cnt + par);
    }
}

// ---------------------------------------------------------------------------
// triangular sweeps (y holds the permuted right-hand side, then the solution)
// ---------------------------------------------------------------------------
constexpr int kSolveThreads = 256;
static_assert(kSolveThreads == 256, "the sweep work splits assume 256 threads");

// skip modes of the sweeps: SKIP_NONE runs every front; SKIP_REFINE skips
// the fronts of instances whose refinement has stopped, SKIP_CG those whose
// CG has stopped (the queued rounds after a stop decision do nothing)
__device__ __forceinline__ bool front_idle(const FrontDesc& F, int skip) {
    return skip == SKIP_REFINE ? *F.done != 0 : (skip == SKIP_CG ? *F.cgdone != 0 : false);
}

// v_writelane_b32 by the name of its intrinsic, which this compiler gives no builtin
extern "C" __device__ int kkt_writelane(int v, int lane, int old) __asm("llvm.amdgcn.writelane.i32");
__device__ __forceinline__ double writelane_d(double v, int lane, double old) {
    const long long b = __double_as_longlong(v), o = __double_as_longlong(old);
    const int lo = kkt_writelane((int)b, lane, (int)o), hi = kkt_writelane((int)(b >> 32), lane, (int)(o >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// two neighbouring rows of a panel column (8-byte aligned; one 16-byte load).
// The address unit takes about 16 cycles per load instruction of a wave
// whatever its width (measured, one workgroup: a panel of 66 x 199 in 5,000
// cycles by 8-byte loads, 2,900 by 16-byte loads of row pairs).
typedef double rows2 __attribute__((ext_vector_type(2), aligned(8)));

__device__ __forceinline__ rows2 rows_at(const double* col, unsigned row) {
    return *(const rows2*)((const char*)col + 8u * row);
}

// Substitution by the wave that owns the pivot rows (lane l: rows 2 l and
// 2 l + 1, values acc0 and acc1): every lane takes its terms with the pivot
// lane's value as a scalar, so one multiply, two lane reads and two FMAs per
// column solve the column and update all 128 rows (about 50 cycles; a chain
// inside 16 lanes by DPP broadcasts costs as much and leaves the other rows'
// updates to be done). The solved values are collected in y0 and y1; sums of
// rows at and above a solved pivot are no longer meaningful. Four columns from K0
// on, of a block of nb (TAIL: fewer than four are left).
template <int K0, bool TAIL>
__device__ __forceinline__ void fwd_steps(double& acc0, double& acc1, double& y0, double& y1, const rows2 (&a)[16],
                                          const double d0, const double d1, const int l0, const int nb) {
    static_for<4>([&](auto K) {
        constexpr int k = K0 + K;
        const int l = l0 + (k >> 1);
        double v = readlane_d((k & 1) ? acc1 * d1 : acc0 * d0, l);
        if (TAIL) v = k < nb ? v : 0.0;
        if constexpr ((k & 1) != 0) y1 = writelane_d(v, l, y1);
        else y0 = writelane_d(v, l, y0);
        acc0 = fma(-a[k].x, v, acc0);
        acc1 = fma(-a[k].y, v, acc1);
    });
}

// Forward step of one front by NTH threads: thread t holds rows 2 t and
// 2 t + 1, their panel entries in registers, up to three blocks of 16 columns
// in flight (loaded as the panel lies in HBM: no LDS staging, and only vectors
// in LDS, so the registers alone limit the fronts per compute unit). Levels of
// few fronts are bound by one wave's chain and the load latency (a 66 x 198
// front: loads and children's sums 4,700 cycles, columns 52 cycles each; with
// the panel staged in LDS and 16-lane chains 19,000 in all, 10.4 -> 6.0 us a
// launch), the leaf levels by HBM (512 fronts of 79 x 227: 26.9 -> 22.5 us).
// MAXR: blocks in flight at most, two for fronts of more than 96 columns and in
// the queue, where a third does not fit the registers. A spilled value makes
// every hardware queue allocate scratch memory at the first launch of the
// kernel (the first solve of a 450-variable system on a new queue 240 us
// against 110), and costs more than the third block gives (500 stages of 54
// variables, fronts of up to 112 columns: 186 -> 161 us a solve).
template <int NTH, int NBLK, int MAXR>
__device__ __forceinline__ void fwd_body(const InstDev* __restrict__ insts, const FrontDesc& F,
                                         double* __restrict__ sh) {
    constexpr int VU = kSolveThreads / NTH, NR = NBLK < MAXR ? NBLK : NBLK < 7 ? MAXR : 2;
    const int c = F.c, r = F.r;
    const int ld = r | 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cp = rup16(c), re = even_up(r);
    double* const ys = sh;       // solved values, zero past c
    double* const s0 = ys + cp;  // the two children's update vectors by row
    double* const s1 = s0 + re;
    double* const ex = s1 + re;  // rows past the threads
    const int row = 2 * tid, rc = min(row, (r - 1) & ~1);
    // loads before the first wait: the first entries of the first two
    // children's update vectors, the right-hand side and pivot reciprocals,
    // and 32 columns of the thread's rows
    const int ch0 = F.ch0, nch = F.nch, ch1 = ch0 + nch;
    struct VChild {
        const double* Vc;
        const int* rl;
        int uc;
    };
    // child at ch_list position q; the first two from the front descriptor
    auto vchild = [&](const int q) {
        VChild C;
        const int k = q - ch0;
        if (k < 2) {
            C.uc = k ? F.cuc[1] : F.cuc[0];
            C.Vc = k ? F.cV[1] : F.cV[0];
            C.rl = k ? F.crl[1] : F.crl[0];
        } else {
            const InstDev& I = insts[F.inst];
            const PatDev& T = I.P;
            const int ch = __builtin_amdgcn_readfirstlane(T.ch_list[q]);
            const int cc = __builtin_amdgcn_readfirstlane(T.sn_ncol[ch]);
            C.uc = __builtin_amdgcn_readfirstlane(T.sn_nrow[ch]) - cc;
            C.Vc = I.V + T.sn_vofs[ch];
            C.rl = T.rel + T.sn_rowofs[ch] + cc;
        }
        return C;
    };
    VChild V0 = {}, V1 = {};
    double v0[VU], v1[VU];
    int r0[VU], r1[VU];
    if (nch > 0) {
        V0 = vchild(ch0);
#pragma unroll
        for (int h = 0; h < VU; h++) {
            const int a = min(tid + h * NTH, V0.uc - 1);
            v0[h] = V0.Vc[a];
            r0[h] = V0.rl[a];
        }
    }
    if (nch > 1) {
        V1 = vchild(ch0 + 1);
#pragma unroll
        for (int h = 0; h < VU; h++) {
            const int a = min(tid + h * NTH, V1.uc - 1);
            v1[h] = V1.Vc[a];
            r1[h] = V1.rl[a];
        }
    }
    double w0 = 0.0, w1 = 0.0, d0 = 0.0, d1 = 0.0;
    if (wave == 0) {
        const int i0 = min(row, c - 1), i1 = min(row + 1, c - 1);
        w0 = F.y[i0];
        w1 = F.y[i1];
        d0 = F.dinv[i0];
        d1 = F.dinv[i1];
    }
    const bool live = 128 * wave < r;
    const double* const Pl = F.L;
    rows2 a[NR][16];
    // (no load depends on a branch, so every wait counts exactly; columns
    // past the last are read from the last)
    auto load = [&](auto B) {
#pragma unroll
        for (int k = 0; k < 16; k++)
            a[B % NR][k] = rows_at(Pl + (B + 1 < NBLK ? 16 * B + k : min(16 * B + k, c - 1)) * ld, rc);
    };
    static_for<(NR < 2 ? NR : 2)>([&](auto B) { load(B); });
    double acc0 = row < c ? w0 : 0.0, acc1 = row + 1 < c ? w1 : 0.0;
    if (nch > 0) {
        for (int i = tid; i < re; i += NTH) s0[i] = s1[i] = 0.0;
        __syncthreads();
#pragma unroll
        for (int h = 0; h < VU; h++)
            if (tid + h * NTH < V0.uc) s0[r0[h]] = v0[h];
        for (int q = tid + VU * NTH; q < V0.uc; q += NTH) s0[V0.rl[q]] = V0.Vc[q];
#pragma unroll
        for (int h = 0; h < VU; h++)
            if (tid + h * NTH < V1.uc) s1[r1[h]] = v1[h];
        for (int q = tid + VU * NTH; q < V1.uc; q += NTH) s1[V1.rl[q]] = V1.Vc[q];
        __syncthreads();
        acc0 = (acc0 + s0[rc]) + s1[rc];
        acc1 = (acc1 + s0[rc + 1]) + s1[rc + 1];
        for (int i = tid + 2 * NTH; i < r; i += NTH) ex[i - 2 * NTH] = s0[i] + s1[i];
        for (int q = ch0 + 2; q < ch1; q += 2) {  // in the children's order, two at a time
            __syncthreads();
            for (int i = tid; i < re; i += NTH) s0[i] = s1[i] = 0.0;
            __syncthreads();
            const VChild A = vchild(q);
            for (int e = tid; e < A.uc; e += NTH) s0[A.rl[e]] = A.Vc[e];
            if (q + 1 < ch1) {
                const VChild B = vchild(q + 1);
                for (int e = tid; e < B.uc; e += NTH) s1[B.rl[e]] = B.Vc[e];
            }
            __syncthreads();
            acc0 = (acc0 + s0[rc]) + s1[rc];
            acc1 = (acc1 + s0[rc + 1]) + s1[rc + 1];
            for (int i = tid + 2 * NTH; i < r; i += NTH)
                ex[i - 2 * NTH] = (ex[i - 2 * NTH] + s0[i]) + s1[i];
        }
    } else {
        for (int i = tid + 2 * NTH; i < r; i += NTH) ex[i - 2 * NTH] = 0.0;
    }
    if constexpr (NR > 2) load(std::integral_constant<int, 2>{});
    // L11 y = w and the update rows, 16 columns at a time: the first wave
    // solves the columns (its own rows, at most 128 of them pivots, take
    // their terms in the same steps), the other waves take the solved values
    // one block behind. Every row subtracts its terms in ascending column
    // order.
    double y0 = 0.0, y1 = 0.0;
    static_for<NBLK>([&](auto B) {
        constexpr int j0 = 16 * B, l0 = 8 * B;
        const int nb = c - j0;
        if (wave == 0) {
            static_for<4>([&](auto Q) {
                if (B + 1 < NBLK || nb >= 4 * Q + 4)
                    fwd_steps<4 * Q, false>(acc0, acc1, y0, y1, a[B % NR], d0, d1, l0, nb);
                else if (nb > 4 * Q)
                    fwd_steps<4 * Q, true>(acc0, acc1, y0, y1, a[B % NR], d0, d1, l0, nb);
            });
            if (lane >= l0 && lane < l0 + 8) {
                ys[row] = y0;
                ys[row + 1] = y1;
            }
        }
        __syncthreads();
        if (wave > 0 && live) {  // (eight of the values at a time: registers)
#pragma unroll
            for (int h = 0; h < 16; h += 8) {
                double y[8];
#pragma unroll
                for (int k = 0; k < 8; k++) y[k] = ys[j0 + h + k];
#pragma unroll
                for (int k = 0; k < 8; k++) {
                    acc0 = fma(-a[B % NR][h + k].x, y[k], acc0);
                    acc1 = fma(-a[B % NR][h + k].y, y[k], acc1);
                }
            }
        }
        if constexpr (B + NR < NBLK) load(std::integral_constant<int, B + NR>{});
    });
    double* const Vs = F.V;
    if (row < c) F.y[row] = y0;
    else if (row < r) Vs[row - c] = acc0;
    if (row + 1 < c) F.y[row + 1] = y1;
    else if (row + 1 < r) Vs[row + 1 - c] = acc1;
    for (int i = tid + 2 * NTH; i < r; i += NTH) {
        double s = ex[i - 2 * NTH];
        for (int j = 0; j < c; j += 8) {
            double b[8];
#pragma unroll
            for (int k = 0; k < 8; k++) b[k] = Pl[min(j + k, c - 1) * ld + i];
#pragma unroll
            for (int k = 0; k < 8; k++) s = fma(-b[k], ys[j + k], s);
        }
        Vs[i - c] = s;
    }
}

// one body per number of column blocks (c <= 128)
template <int NTH, int MAXR>
__device__ __forceinline__ void fwd_front(const InstDev* __restrict__ insts, const FrontDesc& F, const int skip_done,
                                          double* __restrict__ sh) {
    if (front_idle(F, skip_done)) return;
    switch ((F.c + 15) >> 4) {
        case 1: return fwd_body<NTH, 1, MAXR>(insts, F, sh);
        case 2: return fwd_body<NTH, 2, MAXR>(insts, F, sh);
        case 3: return fwd_body<NTH, 3, MAXR>(insts, F, sh);
        case 4: return fwd_body<NTH, 4, MAXR>(insts, F, sh);
        case 5: return fwd_body<NTH, 5, MAXR>(insts, F, sh);
        case 6: return fwd_body<NTH, 6, MAXR>(insts, F, sh);
        case 7: return fwd_body<NTH, 7, MAXR>(insts, F, sh);
        default: return fwd_body<NTH, 8, MAXR>(insts, F, sh);
    }
}

// Columns k0 + 3 down to k0 of a 16-column block by one wave (lane l0 + k of x
// holds column k; TAIL: the block has nb < k0 + 4). o collects the solution,
// xl the terms of the columns 64 to the left (HI).
template <int K0, bool TAIL, bool HI>
__device__ __forceinline__ void bwd_steps(double& x, double& xl, double& o, const double (&a)[16],
                                          const double (&al)[16], const double d, const int l0, const int nb) {
    static_for<4>([&](auto K) {
        constexpr int k = K0 + 3 - decltype(K)::value;
        double v = readlane_d(x * d, l0 + k);
        if (TAIL) v = k < nb ? v : 0.0;
        o = writelane_d(v, l0 + k, o);
        x = fma(-a[k], v, x);
        if constexpr (HI) xl = fma(-al[k], v, xl);
    });
}

// L11^T x = t by one wave, from the last column down (c <= 128): lane l
// carries columns l and l + 64 in x0 and x1 and their pivot reciprocals in
// d0 and d1; P holds the panel (odd leading dimension ld). Steps as in
// fwd_steps. The first 64 columns' coefficients are read ahead of the
// solution (tri_bwd_load, while the other waves still sum), so the steps wait
// for no load.
__device__ __forceinline__ void tri_bwd_load(double (&a)[4][16], const double* __restrict__ P, const int ld,
                                             const int c, const int lane) {
    const double* const p = P + min(lane, c - 1) * ld;
    static_for<4>([&](auto B) {
        if (16 * B < c) {
#pragma unroll
            for (int k = 0; k < 16; k++) a[B][k] = p[min(16 * B + k, c - 1)];
        }
    });
}
__device__ __forceinline__ void tri_bwd_wave(const double (&a)[4][16], const double* __restrict__ P, const int ld,
                                             const int c, const double d0, const double d1, double& x0, double& x1,
                                             const int lane) {
    double o0 = 0.0, o1 = 0.0;
    if (c > 64) {
        const double* const p0 = P + lane * ld;
        const double* const p1 = P + min(lane + 64, c - 1) * ld;
        for (int j = (c - 1) & ~15; j >= 64; j -= 16) {
            const int nb = c - j;
            double u[16], v[16];
#pragma unroll
            for (int k = 0; k < 16; k++) {
                u[k] = p1[min(j + k, c - 1)];
                v[k] = p0[min(j + k, c - 1)];
            }
            static_for<4>([&](auto Q) {
                if (nb > 12 - 4 * Q) bwd_steps<12 - 4 * Q, true, true>(x1, x0, o1, u, v, d1, j - 64, nb);
            });
        }
    }
    static_for<4>([&](auto Q) {
        constexpr int B = 3 - decltype(Q)::value;
        const int nb = c - 16 * B;
        if (nb >= 16) {
            static_for<4>([&](auto R) {
                bwd_steps<12 - 4 * R, false, false>(x0, x0, o0, a[B], a[B], d0, 16 * B, nb);
            });
        } else if (nb > 0) {
            static_for<4>([&](auto R) {
                if (nb > 12 - 4 * R) bwd_steps<12 - 4 * R, true, false>(x0, x0, o0, a[B], a[B], d0, 16 * B, nb);
            });
        }
    });
    x0 = o0;
    x1 = o1;
}

// Backward step of one front: the panel is staged in LDS (odd leading
// dimension) by contiguous 16-byte loads, the dot products run over all
// threads, the triangle by one wave. A 66 x 198 front takes 5,800 cycles to
// stage, 3,000 for the products and 3,800 for the triangle (one row's chain
// after another by DPP broadcasts: 12,500); 11.0 -> 7.3 us a launch of few
// fronts with four waves, 6.6 with eight, two lanes then sharing a column's
// four sums. Taking the rectangle from HBM to registers instead costs more where
// few fronts run (its strands load at a third of the rate; about 10 us) and
// wins only on levels of more fronts than compute units (bwd_front_wide).
// PU: panel loads per thread in flight while staging; NTH: 512 threads, or
// 256 where every panel is at most kSweepHalfLds (several fronts share a
// compute unit) and in the queue. REST: what is left of the panel PU at a time
// too (the queue, whose 256 threads take whole panels; on the level launches,
// with little left, it costs 1 to 2 %). The sums do not depend on any of them.
template <int PU, int NTH, bool REST>
__device__ __forceinline__ void bwd_front(const FrontDesc& F, double* __restrict__ sh) {
    constexpr int HS = NTH / kSolveThreads, NS = 4 / HS;  // lanes per g, strands per lane
    const int c = F.c, r = F.r;
    const int u = r - c;
    double* const yb = F.y - F.col0;  // the instance's work vector
    const int ld = r | 1;
    constexpr int nt = NTH;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // G consecutive lanes per column (G c <= 256 for c <= 128)
    const int lg = c <= 16 ? 4 : c <= 32 ? 3 : c <= 64 ? 2 : 1, G = 1 << lg;
    const int nz = (u + 4 * G - 1) & -(4 * G);
    double* P = sh;
    double* z = sh + even_up(ld * c);
    double* t = z + nz;
    // row i of the update part at z[place(i)]: a lane's four rows of a step
    // (G apart) side by side
    auto place = [&](const int i) {
        return ((i >> (lg + 2)) << (lg + 2)) + ((i & (G - 1)) << 2) + ((i >> lg) & 3);
    };
    const int* __restrict__ rw = F.rw;
    // The update rows' indices are loaded first, so the gather of their
    // values waits only for them while the panel loads stay in flight.
    int ri = u > 0 ? rw[min(tid, u - 1)] : 0;
    const double2* __restrict__ s2 = (const double2*)(const double*)F.L;
    double2* d2 = (double2*)P;
    const int n2 = even_up(ld * c) >> 1;
    double2 pv[PU];
#pragma unroll
    for (int k = 0; k < PU; k++) pv[k] = s2[min(tid + k * nt, n2 - 1)];
    double d0 = 0.0, d1 = 0.0, y0 = 0.0, y1 = 0.0;
    if (wave == 0) {
        d0 = F.dinv[min(lane, c - 1)];
        d1 = F.dinv[min(lane + 64, c - 1)];
        y0 = F.y[min(lane, c - 1)];
        y1 = F.y[min(lane + 64, c - 1)];
    }
    pin(ri);
    double zy = u > 0 ? yb[ri] : 0.0;
#pragma unroll
    for (int k = 0; k < PU; k++) pin(pv[k]);
#pragma unroll
    for (int k = 0; k < PU; k++)
        if (tid + k * nt < n2) d2[tid + k * nt] = pv[k];
    if constexpr (REST) {
        for (int q = tid + PU * nt; q < n2; q += PU * nt) {
#pragma unroll
            for (int k = 0; k < PU; k++) pv[k] = s2[min(q + k * nt, n2 - 1)];
#pragma unroll
            for (int k = 0; k < PU; k++) pin(pv[k]);
#pragma unroll
            for (int k = 0; k < PU; k++)
                if (q + k * nt < n2) d2[q + k * nt] = pv[k];
        }
    } else {
        for (int q = tid + PU * nt; q < n2; q += nt) d2[q] = s2[q];
    }
    pin(zy);
    if (tid < nz) z[place(tid)] = tid < u ? zy : 0.0;
    for (int i = tid + nt; i < nz; i += nt) z[place(i)] = i < u ? yb[rw[i]] : 0.0;
    __syncthreads();
    // t = y1 - L21^T z: lane g of a column's G takes rows g, g + G, g + 2 G,
    // g + 3 G of every 4 G into four running sums while all four are there,
    // the rest into the first; a group's sums are combined in a fixed order.
    // Four steps' LDS reads go out together.
    {
        constexpr int sp = HS == 2 ? 1 : 0;
        const int k = tid >> (lg + sp), g = tid & (G - 1), half = sp ? (tid >> lg) & 1 : 0;
        const int T = u - 3 * G - g > 0 ? (u - 3 * G - g + 4 * G - 1) >> (lg + 2) : 0;
        double a[NS];
#pragma unroll
        for (int h = 0; h < NS; h++) a[h] = 0.0;
        if (k < c) {
            const double* const col = P + k * ld + c + g + G * NS * half;
            const double* const zg = z + 4 * g + NS * half;
            int s = 0;
            for (; s + 4 <= T; s += 4) {
                double p[4][NS], q[4][NS];
#pragma unroll
                for (int e = 0; e < 4; e++)
#pragma unroll
                    for (int h = 0; h < NS; h++) {
                        p[e][h] = col[4 * G * (s + e) + G * h];
                        q[e][h] = zg[4 * G * (s + e) + h];
                    }
#pragma unroll
                for (int e = 0; e < 4; e++)
#pragma unroll
                    for (int h = 0; h < NS; h++) a[h] = fma(p[e][h], q[e][h], a[h]);
            }
            for (; s < T; s++)
#pragma unroll
                for (int h = 0; h < NS; h++) a[h] = fma(col[4 * G * s + G * h], zg[4 * G * s + h], a[h]);
            if (half == 0)
                for (int h = 0; g + 4 * G * T + G * h < u; h++)
                    a[0] = fma(col[4 * G * T + G * h], zg[4 * G * T + h], a[0]);
        }
        double part;
        if constexpr (HS == 1) {
            part = (a[0] + a[1]) + (a[2] + a[3]);
        } else {
            part = a[0] + a[1];
            part += __shfl_xor(part, G);
        }
        for (int off = G >> 1; off > 0; off >>= 1) part += __shfl_xor(part, off);
        if (k < c && g == 0 && half == 0) t[k] = part;
    }
    double a[4][16];
    if (wave == 0) tri_bwd_load(a, P, ld, c, lane);
    __syncthreads();
    if (wave == 0) {
        double x0 = lane < c ? y0 - t[lane] : 0.0;
        double x1 = lane + 64 < c ? y1 - t[lane + 64] : 0.0;
        tri_bwd_wave(a, P, ld, c, d0, d1, x0, x1, lane);
        if (lane < c) F.y[lane] = x0;
        if (lane + 64 < c) F.y[lane + 64] = x1;
    }
}

// sum of a column's 4 G strands (strand g + G q holds rows g + G q, g + G q +
// 4 G, ... of the column): the four strands of each g, then g by halves
template <int G>
__device__ __forceinline__ double strand_sum(const double* __restrict__ w) {
    double p[G];
#pragma unroll
    for (int g = 0; g < G; g++) p[g] = (w[g] + w[g + G]) + (w[g + 2 * G] + w[g + 3 * G]);
#pragma unroll
    for (int h = G >> 1; h > 0; h >>= 1)
#pragma unroll
        for (int g = 0; g < h; g++) p[g] += p[g + h];
    return p[0];
}

// Backward step of one front of a level of more fronts than compute units: the
// rectangle goes from HBM to registers straight into the dot products (a lane
// holds two neighbouring strands of a column: 8 strands a column above 64
// columns, 16, 32 or 64 at most 64, 32, 16, so two passes cover every front)
// and only the triangle is staged in LDS, so two workgroups share a compute
// unit where a whole panel leaves room for one (512 fronts of 79 x 227: 24 ->
// 18.5 us). Every sum takes the order of bwd_front (same bits). Bound by HBM
// and the address unit (16 cycles a load).
__device__ __forceinline__ void bwd_front_wide(const FrontDesc& F, double* __restrict__ sh) {
    constexpr int nt = kSolveThreads, NT = 6, NP = 2;
    const int c = F.c, r = F.r, u = r - c;
    double* const yb = F.y - F.col0;  // the instance's work vector
    const int ld = r | 1, ldt = c | 1;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lg = c <= 16 ? 4 : c <= 32 ? 3 : c <= 64 ? 2 : 1, G = 1 << lg, S = 4 * G;
    double* const P = sh;
    double* const z = P + even_up(ldt * c);
    double* const w = z + even_up(u);
    const int* const rw = F.rw;
    const double* const Pl = F.L;
    // loads, before the first wait: the update rows' indices (the gather of
    // their values waits for them alone), the first rows of the strands and
    // 64 columns of the triangle
    const int ri = u > 0 ? rw[min(tid, u - 1)] : 0;
    const int cpp = nt >> (lg + 1);  // columns per pass
    const int e = 2 * (tid & (2 * G - 1)), col = tid >> (lg + 1), g = e & (G - 1);
    const int wcol = (64 * wave) >> (lg + 1);  // the wave's first
    rows2 v0[NP][NT], v1[NP][NT];
    auto load = [&](rows2 (&v)[NP][NT], const int t0) {
        static_for<NP>([&](auto p) {
            if (p * cpp + wcol < c) {
                const double* const b = Pl + (min(p * cpp + col, c - 1) * ld + c);
#pragma unroll
                for (int t = 0; t < NT; t++) v[p][t] = *(const rows2*)(b + min(e + S * (t0 + t), u - 1));
            }
        });
    };
    const int nT = (u + S - 1) >> (lg + 2);  // rows per strand, at most
    if (u > 0) load(v0, 0);
    rows2 ta[16];
    auto tri_load = [&](const int j0) {
#pragma unroll
        for (int k = 0; k < 16; k++)
            if (j0 + 4 * k + wave < c)
                ta[k] = rows_at(Pl + (j0 + 4 * k + wave) * ld, min(2 * lane, (c - 1) & ~1));
    };
    auto tri_store = [&](const int j0) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            const int j = j0 + 4 * k + wave;
            if (j < c) {
                double* const d = P + j * ldt + 2 * lane;
                if (2 * lane < c) d[0] = ta[k].x;
                if (2 * lane + 1 < c) d[1] = ta[k].y;
            }
        }
    };
    tri_load(0);
    double d0 = 0.0, d1 = 0.0, y0 = 0.0, y1 = 0.0;
    if (wave == 0) {
        d0 = F.dinv[min(lane, c - 1)];
        d1 = F.dinv[min(lane + 64, c - 1)];
        y0 = F.y[min(lane, c - 1)];
        y1 = F.y[min(lane + 64, c - 1)];
    }
    const double zy = u > 0 ? yb[ri] : 0.0;
    if (nT > NT) load(v1, NT);
    tri_store(0);
    if (c > 64) tri_load(64);
    if (tid < u) z[tid] = zy;
    for (int i = tid + nt; i < u; i += nt) z[i] = yb[rw[i]];
    __syncthreads();
    // t = y1 - L21^T z. Lane g of a column's G takes rows four G at a time,
    // one per strand, while four are left (T steps); what remains of its rows
    // goes to its first strand.
    auto steps = [&](const int g) { return u - 3 * G - g > 0 ? (u - 3 * G - g + S - 1) >> (lg + 2) : 0; };
    const int T0 = steps(g), T1 = steps(g + 1);
    double s0[NP] = {0.0, 0.0}, s1[NP] = {0.0, 0.0};
    if (u > 0) {
        auto terms = [&](const rows2 (&v)[NP][NT], const int t0) {
            double za[NT], zb[NT];
#pragma unroll
            for (int t = 0; t < NT; t++) {
                const int i = min(e + S * (t0 + t), (u - 1) & ~1);
                za[t] = z[i];
                zb[t] = z[i + 1];
            }
#pragma unroll
            for (int t = 0; t < NT; t++) {
                za[t] = t0 + t < T0 ? za[t] : 0.0;
                zb[t] = t0 + t < T1 ? zb[t] : 0.0;
            }
            static_for<NP>([&](auto p) {
                if (p * cpp + wcol < c) {
#pragma unroll
                    for (int t = 0; t < NT; t++) {
                        s0[p] = fma(t0 + t < T0 ? v[p][t].x : 0.0, za[t], s0[p]);
                        s1[p] = fma(t0 + t < T1 ? v[p][t].y : 0.0, zb[t], s1[p]);
                    }
                }
            });
        };
        double ra[NP][3], rb[NP][3];
        const int i0 = g + S * T0, i1 = g + 1 + S * T1;
        if (e < G) {
            static_for<NP>([&](auto p) {
                if (p * cpp + wcol < c) {
                    const double* const b = Pl + (min(p * cpp + col, c - 1) * ld + c);
#pragma unroll
                    for (int k = 0; k < 3; k++) {
                        ra[p][k] = b[min(i0 + G * k, u - 1)];
                        rb[p][k] = b[min(i1 + G * k, u - 1)];
                    }
                }
            });
        }
        for (int t0 = 0; t0 < nT; t0 += 2 * NT) {
            terms(v0, t0);
            if (t0 + 2 * NT < nT) load(v0, t0 + 2 * NT);
            if (t0 + NT < nT) terms(v1, t0 + NT);
            if (t0 + 3 * NT < nT) load(v1, t0 + 3 * NT);
        }
        if (e < G) {
            double za[3], zb[3];
#pragma unroll
            for (int k = 0; k < 3; k++) {
                za[k] = i0 + G * k < u ? z[i0 + G * k] : 0.0;
                zb[k] = i1 + G * k < u ? z[i1 + G * k] : 0.0;
            }
            static_for<NP>([&](auto p) {
                if (p * cpp + wcol < c) {
#pragma unroll
                    for (int k = 0; k < 3; k++) {
                        s0[p] = fma(ra[p][k], za[k], s0[p]);
                        s1[p] = fma(rb[p][k], zb[k], s1[p]);
                    }
                }
            });
        }
    }
    if (c > 64) tri_store(64);
    const int ws = S + 1;
#pragma unroll
    for (int p = 0; p < NP; p++)
        if (p * cpp + col < c) {
            w[(p * cpp + col) * ws + e] = s0[p];
            w[(p * cpp + col) * ws + e + 1] = s1[p];
        }
    __syncthreads();
    if (wave == 0) {
        double x0 = 0.0, x1 = 0.0;
        const double* const w0 = w + min(lane, c - 1) * ws;
        if (G == 2) {
            x0 = strand_sum<2>(w0);
            x1 = strand_sum<2>(w + min(lane + 64, c - 1) * ws);
        } else if (G == 4) {
            x0 = strand_sum<4>(w0);
        } else if (G == 8) {
            x0 = strand_sum<8>(w0);
        } else {
            x0 = strand_sum<16>(w0);
        }
        x0 = lane < c ? y0 - x0 : 0.0;
        x1 = lane + 64 < c ? y1 - x1 : 0.0;
        double a[4][16];
        tri_bwd_load(a, P, ldt, c, lane);
        tri_bwd_wave(a, P, ldt, c, d0, d1, x0, x1, lane);
        if (lane < c) F.y[lane] = x0;
        if (lane + 64 < c) F.y[lane + 64] = x1;
    }
}

// Forward sweep of large fronts. k_big_fwd, one workgroup per front: the
// children's update vectors are added child by child (the update part in the
// front's own HBM slot), the c x c triangle is solved by one wave, its
// coefficients in registers (y_j = w_j / l_jj, then w_i -= l_ij y_j for i > j,
// in column order). k_big_fwd_rows: the update rows take -L21 y by one thread
// per row (column order), over as many workgroups as they fill. By one
// workgroup in all, its loads one after another, the pass took 46 us on a
// front of 64 x 1,460; 12 us now.
template <int K0, bool TAIL>
__device__ __forceinline__ void row_steps(double& w, double& y, const double (&a)[16], const double d, const int l0,
                                          const int nb) {
    static_for<4>([&](auto K) {
        constexpr int k = K0 + K;
        double v = readlane_d(w * d, l0 + k);
        if (TAIL) v = k < nb ? v : 0.0;
        y = writelane_d(v, l0 + k, y);
        w = fma(-a[k], v, w);
    });
}
__global__ __launch_bounds__(kBigThreads) void k_big_fwd(const InstDev* __restrict__ insts,
                                                       const FrontDesc* __restrict__ fds, int skip_done) {
    __shared__ double w[kBigMaxCols];
    const FrontDesc& F = fds[blockIdx.x];
    if (front_idle(F, skip_done)) return;
    const InstDev& I = insts[F.inst];
    const PatDev& T = I.P;
    const int c = F.c, r = F.r, u = r - c, ld = r | 1;
    const double* const P = F.L;
    double* const V = F.V;
    constexpr int nt = kBigThreads, VU = 8;
    const int tid = threadIdx.x, lane = tid & 63;
    double a[4][16], d = 0.0;
    if (tid < 64) {
        static_for<4>([&](auto B) {
#pragma unroll
            for (int k = 0; k < 16; k++) a[B][k] = P[(int64_t)min(16 * B + k, c - 1) * ld + min(lane, c - 1)];
        });
        d = F.dinv[min(lane, c - 1)];
    }
    if (tid < c) w[tid] = F.y[tid];
    for (int i = tid; i < u; i += nt) V[i] = 0.0;
    __syncthreads();
    for (int k = 0; k < F.nch; k++) {
        const int ch = T.ch_list[F.ch0 + k];
        const int cc = T.sn_ncol[ch];
        const int uc = T.sn_nrow[ch] - cc;
        const double* const Vc = I.V + T.sn_vofs[ch];
        const int* const rl = T.rel + T.sn_rowofs[ch] + cc;
        // (a child's entries are distinct: VU of them per thread in flight)
        for (int q0 = tid; q0 < uc; q0 += VU * nt) {
            int ra[VU];
            double v[VU], t[VU];
#pragma unroll
            for (int e = 0; e < VU; e++) {
                const int q = min(q0 + e * nt, uc - 1);
                ra[e] = rl[q];
                v[e] = Vc[q];
            }
#pragma unroll
            for (int e = 0; e < VU; e++) t[e] = u > 0 ? V[max(ra[e] - c, 0)] : 0.0;
#pragma unroll
            for (int e = 0; e < VU; e++) {
                if (q0 + e * nt >= uc) continue;
                if (ra[e] < c) w[ra[e]] += v[e];
                else V[ra[e] - c] = t[e] + v[e];
            }
        }
        __syncthreads();
    }
    if (tid < 64) {
        double x = lane < c ? w[lane] : 0.0, y = 0.0;
        static_for<4>([&](auto B) {
            const int nb = c - 16 * B;
            static_for<4>([&](auto Q) {
                if (nb >= 4 * Q + 4) row_steps<4 * Q, false>(x, y, a[B], d, 16 * B, nb);
                else if (nb > 4 * Q) row_steps<4 * Q, true>(x, y, a[B], d, 16 * B, nb);
            });
        });
        if (lane < c) F.y[lane] = y;
    }
}
__global__ __launch_bounds__(kBigThreads) void k_big_fwd_rows(const FrontDesc* __restrict__ fds, int skip_done) {
    const FrontDesc& F = fds[blockIdx.x];
    const int c = F.c, r = F.r, u = r - c, ld = r | 1;
    const int row = (int)blockIdx.y * kBigThreads + threadIdx.x;
    if ((int)blockIdx.y * kBigThreads >= u) return;
    if (front_idle(F, skip_done)) return;
    __shared__ double y[kBigMaxCols];
    if (threadIdx.x < kBigMaxCols) y[threadIdx.x] = (int)threadIdx.x < c ? F.y[threadIdx.x] : 0.0;
    const int i = min(row, u - 1);
    const double* const P = (const double*)F.L + c + i;
    double acc = F.V[i];
    double a[4][16];
    static_for<4>([&](auto B) {
#pragma unroll
        for (int k = 0; k < 16; k++) a[B][k] = P[(int64_t)min(16 * B + k, c - 1) * ld];
    });
    __syncthreads();
    static_for<4>([&](auto B) {
        if (16 * B < c) {
#pragma unroll
            for (int k = 0; k < 16; k++)
                if (16 * B + k < c) acc = fma(-a[B][k], y[16 * B + k], acc);
        }
    });
    if (row < u) F.V[row] = acc;
}

// Backward sweep of large fronts. k_big_bwd_dot: y1 - L21^T z, one wave per
// column (lanes over rows, a fixed butterfly); k_big_bwd: the triangle by one
// wave, one workgroup per front. With the dot products in the front's one
// workgroup, a row index, its value and the panel entry at a time, the pass
// took 113 us on a front of 64 x 1,460; 9 us now.
__global__ __launch_bounds__(kBigThreads) void k_big_bwd_dot(const FrontDesc* __restrict__ fds, int skip_done) {
    constexpr int RU = 8;  // rows per lane in flight
    const FrontDesc& F = fds[blockIdx.x];
    const int c = F.c, r = F.r, u = r - c, ld = r | 1;
    const int lane = threadIdx.x & 63;
    const int j = __builtin_amdgcn_readfirstlane((int)blockIdx.y * (kBigThreads >> 6) + (int)(threadIdx.x >> 6));
    if (j >= c || u == 0) return;
    if (front_idle(F, skip_done)) return;
    const double* const col = (const double*)F.L + (int64_t)j * ld + c;
    const double* const yb = F.y - F.col0;  // the instance's work vector
    const int* const rw = F.rw;
    double s = 0.0;
    for (int a0 = lane; a0 < u; a0 += 64 * RU) {
        int ri[RU];
        double p[RU], z[RU];
#pragma unroll
        for (int e = 0; e < RU; e++) {
            const int a = min(a0 + 64 * e, u - 1);
            ri[e] = rw[a];
            p[e] = col[a];
        }
#pragma unroll
        for (int e = 0; e < RU; e++) z[e] = yb[ri[e]];
#pragma unroll
        for (int e = 0; e < RU; e++)
            if (a0 + 64 * e < u) s = fma(p[e], z[e], s);
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if (lane == 0) F.y[j] = F.y[j] - s;
}
__global__ __launch_bounds__(kBigThreads) void k_big_bwd(const FrontDesc* __restrict__ fds, int skip_done) {
    __shared__ double Ls[kBigMaxCols * (kBigMaxCols + 1)];
    const FrontDesc& F = fds[blockIdx.x];
    if (front_idle(F, skip_done)) return;
    const int c = F.c, r = F.r, ld = r | 1, ldl = c | 1;
    const double* const P = F.L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double t[16];
#pragma unroll
    for (int k = 0; k < 16; k++) t[k] = P[(int64_t)min(4 * k + wave, c - 1) * ld + min(lane, c - 1)];
    double x0 = 0.0, x1 = 0.0, d = 0.0;
    if (wave == 0) {
        x0 = lane < c ? F.y[min(lane, c - 1)] : 0.0;
        d = F.dinv[min(lane, c - 1)];
    }
#pragma unroll
    for (int k = 0; k < 16; k++)
        if (4 * k + wave < c && lane < c) Ls[(4 * k + wave) * ldl + lane] = t[k];
    __syncthreads();
    if (wave == 0) {
        double a[4][16];
        tri_bwd_load(a, Ls, ldl, c, lane);
        tri_bwd_wave(a, Ls, ldl, c, d, d, x0, x1, lane);
        if (lane < c) F.y[lane] = x0;
    }
}

template <int NTH>
__global__ __launch_bounds__(NTH, 2) void k_fwd(const InstDev* __restrict__ insts,
                                                      const FrontDesc* __restrict__ fds, int skip_done) {
    extern __shared__ __align__(16) double sh[];
    fwd_front<NTH, 3>(insts, fds[blockIdx.x], skip_done, sh);
}

template <int PU, int NTH>
__global__ __launch_bounds__(NTH) void k_bwd(const FrontDesc* __restrict__ fds, int skip_done) {
    extern __shared__ __align__(16) double sh[];
    const FrontDesc& F = fds[blockIdx.x];
    if (front_idle(F, skip_done)) return;
    bwd_front<PU, NTH, false>(F, sh);
}

__global__ __launch_bounds__(kSolveThreads, 2) void k_bwd_wide(const FrontDesc* __restrict__ fds, int skip_done) {
    extern __shared__ __align__(16) double sh[];
    const FrontDesc& F = fds[blockIdx.x];
    if (front_idle(F, skip_done)) return;
    bwd_front_wide(F, sh);
}

// Both sweeps in one launch: tickets 0..N-1 are the forward sweep in
// topological order, tickets N..2N-1 the backward sweep in reverse order. A
// front's backward step waits for its parent's (a root waits for its own
// forward step, the last of its tree).
__global__ __launch_bounds__(kSolveThreads, 2) void k_sweeps_queue(const InstDev* __restrict__ insts,
                                                               const FrontDesc* __restrict__ fds, DepLists D,
                                                               int skip_done) {
    extern __shared__ __align__(16) double sh[];
    __shared__ int slot;
    const int N = D.nitems;
    for (;;) {
        const int t = take_ticket(D.ticket, &slot);
        if (t >= 2 * N) break;
        const bool fwd = t < N;
        const int k = fwd ? t : 2 * N - 1 - t;
        const int par = __builtin_amdgcn_readfirstlane(D.parent[k]);
        if (sched_wave()) {
            if (fwd) wait_at_least(D.cnt + k, __builtin_amdgcn_readfirstlane(D.nchild[k]), D.err);
            else if (par >= 0) wait_at_least(D.bdone + par, 1, D.err);
            else wait_at_least(D.fdone + k, 1, D.err);
        }
        __syncthreads();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const FrontDesc& F = fds[k];
        if (fwd) fwd_front<kSolveThreads, 2>(insts, F, skip_done, sh);
        else if (!front_idle(F, skip_done)) bwd_front<16, kSolveThreads, true>(F, sh);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __syncthreads();
        if (sched_wave()) {
            if (!fwd) publish_add(D.bdone + k);
            else if (par >= 0) publish_add(D.cnt + par);
            else publish_add(D.fdone + k);
        }
    }
}

// ---------------------------------------------------------------------------
// permutations between original and pivot order (row blocks of 256)
// ---------------------------------------------------------------------------
// y[k] = src[perm[k]] with src = b (PIN_B) or r (PIN_R)
__global__ __launch_bounds__(256) void k_perm_in(const InstDev* __restrict__ insts, Calls C,
                                                 const WorkItem* __restrict__ items, int mode) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (mode == PIN_R && I.rs->done) return;
    const int k = it.id + threadIdx.x;
    if (k >= I.P.n) return;
    const double* src = mode == PIN_B ? C.b + I.n_off : I.r;
    I.y[k] = src[I.P.perm[k]];
}

// POUT_X: x[perm[k]] = y[k]; POUT_X_UPDATE: xprev = x, x += y[iperm];
// POUT_DX: dx[perm[k]] = y[k]
__global__ __launch_bounds__(256) void k_perm_out(const InstDev* __restrict__ insts, Calls C,
                                                  const WorkItem* __restrict__ items, int mode) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (mode == POUT_X_UPDATE && I.rs->done) return;
    const int k = it.id + threadIdx.x;
    if (k >= I.P.n) return;
    const int i = I.P.perm[k];
    const double v = I.y[k];
    if (mode == POUT_X) {
        C.x[I.n_off + i] = v;
    } else if (mode == POUT_X_UPDATE) {
        double* x = C.x + I.n_off;
        const double xo = x[i];
        I.xprev[i] = xo;
        x[i] = xo + v;
    } else {
        C.dx[I.n_off + i] = v;
    }
}

// ---------------------------------------------------------------------------
// residual r = b - K x and backward-error reductions (original numbering)
// ---------------------------------------------------------------------------
__global__ void k_refine_reset(const InstDev* __restrict__ insts, int ninst, double tol, int maxit,
                               int* __restrict__ ndone) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q == 0) *ndone = 0;
    if (q >= ninst) return;
    RefineState* S = insts[q].rs;
    S->omega = S->omega_prev = INFINITY;
    S->eta = S->eta_prev = INFINITY;
    S->relres = S->relres_prev = INFINITY;
    S->tol = tol;
    S->maxit = maxit;
    S->it = 0;
    S->done = 0;
    S->revert = 0;
}

// block maxima of five values, written to this block's slot (no atomics:
// the decision kernel takes the maximum over the slots)
__device__ inline void block_max5(double v0, double v1, double v2, double v3, double v4, double* out) {
    __shared__ double red[5][256];
    const int tid = threadIdx.x;
    red[0][tid] = v0; red[1][tid] = v1; red[2][tid] = v2; red[3][tid] = v3; red[4][tid] = v4;
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if (tid < h)
            for (int q = 0; q < 5; q++) red[q][tid] = fmax(red[q][tid], red[q][tid + h]);
        __syncthreads();
    }
    if (tid < 5) out[tid] = red[tid][0];
}

// 16 lanes per row (coalesced reads of the row's entries); each 16-lane
// group takes NR rows, 16 apart, and issues the loads of all of them before
// the first wait: many short independent rows in flight hide the dependent
// loads (row bounds, then columns, then x), and each block's reduction is
// shared by 16 NR rows.
__global__ __launch_bounds__(256) void k_residual(const InstDev* __restrict__ insts, Calls C,
                                                  const WorkItem* __restrict__ items) {
    constexpr int NR = 16 / kResidualSplit;  // rows per 16-lane group
    const WorkItem it = items[blockIdx.x / kResidualSplit];
    const InstDev& I = insts[it.inst];
    if (I.rs->done) return;  // uniform per block
    const double* __restrict__ x = C.x + I.n_off;
    const double* __restrict__ b = C.b + I.n_off;
    const int n = I.P.n;
    const int g = threadIdx.x >> 4, l = threadIdx.x & 15;
    double ra = 0.0, om = 0.0, rs = 0.0, xa = 0.0, ba = 0.0;
    const int row0 = it.id + (blockIdx.x % kResidualSplit) * 16 * NR + g;
    // rows past the end load the last row (valid addresses) and are discarded
    int64_t pb[NR], pe[NR];
#pragma unroll
    for (int j = 0; j < NR; j++) {
        const int i = min(row0 + 16 * j, n - 1);
        pb[j] = I.P.sp_ptr[i];
        pe[j] = I.P.sp_ptr[i + 1];
    }
    // the first three entries of each lane and row in one round (values,
    // columns, then the gathered x), clamped so no load is predicated; the
    // terms are then summed in the lane's order, as in the loop for the rest
    constexpr int RU = 3;
    double kv[NR][RU], xv[NR][RU];
    int cl[NR][RU];
#pragma unroll
    for (int j = 0; j < NR; j++)
#pragma unroll
        for (int q = 0; q < RU; q++) {
            const int64_t p = min(pb[j] + l + 16 * q, pe[j] - 1);
            kv[j][q] = I.kcsr[p];
            cl[j][q] = I.P.sp_col[p];
        }
#pragma unroll
    for (int j = 0; j < NR; j++)
#pragma unroll
        for (int q = 0; q < RU; q++) xv[j][q] = x[cl[j][q]];
#pragma unroll
    for (int j = 0; j < NR; j++) {
        double sum = 0.0, den = 0.0, ks = 0.0;
#pragma unroll
        for (int q = 0; q < RU; q++) {
            if (pb[j] + l + 16 * q < pe[j]) {
                const double t = kv[j][q] * xv[j][q];
                sum += t;
                den += fabs(t);
                ks += fabs(kv[j][q]);
            }
        }
        for (int64_t p = pb[j] + l + 16 * RU; p < pe[j]; p += 16) {
            const double kp = I.kcsr[p];
            const double t = kp * x[I.P.sp_col[p]];
            sum += t;
            den += fabs(t);
            ks += fabs(kp);
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) {
            sum += __shfl_xor(sum, o, 16);
            den += __shfl_xor(den, o, 16);
            ks += __shfl_xor(ks, o, 16);
        }
        const int i = row0 + 16 * j;
        if (l == 0 && i < n) {
            const double bi = b[i];
            const double ri = bi - sum;
            I.r[i] = ri;
            const double ai = fabs(ri);
            den += fabs(bi);
            ra = fmax(ra, ai);
            om = fmax(om, den > 0.0 ? ai / den : (ai > 0.0 ? INFINITY : 0.0));
            rs = fmax(rs, ks);
            xa = fmax(xa, fabs(x[i]));
            ba = fmax(ba, fabs(bi));
        }
    }
    const int slot = (it.id >> 8) * kResidualSplit + (int)(blockIdx.x % kResidualSplit);
    block_max5(ra, om, rs, xa, ba, I.rpart + 5 * slot);
}

// One workgroup per instance: the maxima over the residual blocks' slots
// (order-independent), then eta / omega and the refinement stop rule
// (omega <= tol, maxit corrections, or omega not halving; in the last case
// the previous iterate wins if omega grew).
// With rep, the instance's report goes to the host (also of an instance that
// has stopped before: the host reads the reports of the last check only), so
// no copy follows the check.
__global__ __launch_bounds__(256) void k_refine_decide(const InstDev* __restrict__ insts, int* ndone,
                                                       RefineReport* __restrict__ rep, const int* __restrict__ err) {
    const InstDev& I = insts[blockIdx.x];
    RefineState* S = I.rs;
    auto report = [&]() {
        if (!rep) return;
        RefineReport r;
        r.rs = *S;
        r.status[0] = I.status[0];
        r.status[1] = I.status[1];
        r.err = *err;
        rep[blockIdx.x] = r;
    };
    if (S->done) {  // uniform per block
        if (threadIdx.x == 0) report();
        return;
    }
    const int nslots = ((I.P.n + 255) >> 8) * kResidualSplit;
    double m[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
    // eight slots per thread in flight at once; a maximum is unchanged by
    // repeats, so indices past the end repeat the last slot
    constexpr int UNR = 8;
    const double* __restrict__ rp = I.rpart;
    for (int t0 = threadIdx.x; t0 < nslots; t0 += blockDim.x * UNR) {
        double v[UNR][5];
#pragma unroll
        for (int k = 0; k < UNR; k++) {
            const int t = min(t0 + k * (int)blockDim.x, nslots - 1);
#pragma unroll
            for (int q = 0; q < 5; q++) v[k][q] = rp[5 * t + q];
        }
#pragma unroll
        for (int k = 0; k < UNR; k++)
#pragma unroll
            for (int q = 0; q < 5; q++) m[q] = fmax(m[q], v[k][q]);
    }
    __shared__ double red[5][256];
    for (int q = 0; q < 5; q++) red[q][threadIdx.x] = m[q];
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h)
            for (int q = 0; q < 5; q++) red[q][threadIdx.x] = fmax(red[q][threadIdx.x], red[q][threadIdx.x + h]);
        __syncthreads();
    }
    if (threadIdx.x != 0) return;
    const double rmax = red[0][0], om = red[1][0], kn = red[2][0], xm = red[3][0], bm = red[4][0];
    const double den = kn * xm + bm;
    S->eta_prev = S->eta;
    S->relres_prev = S->relres;
    S->omega_prev = S->omega;
    S->eta = den > 0.0 ? rmax / den : 0.0;
    S->relres = bm > 0.0 ? rmax / bm : rmax;
    S->omega = om;
    bool stop = om <= S->tol || S->it >= S->maxit;
    if (S->it > 0 && om > 0.5 * S->omega_prev) {
        stop = true;
        if (om > S->omega_prev) S->revert = 1;
    }
    if (stop) {
        S->done = 1;
        atomicAdd(ndone, 1);
    } else {
        S->it += 1;
    }
    report();
}

__global__ __launch_bounds__(256) void k_refine_revert(const InstDev* __restrict__ insts, Calls C,
                                                       const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (!I.rs->revert) return;
    const int i = it.id + threadIdx.x;
    if (i >= I.P.n) return;
    C.x[I.n_off + i] = I.xprev[i];
}

__global__ __launch_bounds__(256) void k_matvec(const InstDev* __restrict__ insts, const double* __restrict__ x,
                                                double* __restrict__ y, const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    if (i >= I.P.n) return;
    double sum = 0.0;
    for (int64_t p = I.P.sp_ptr[i]; p < I.P.sp_ptr[i + 1]; p++) sum += I.kcsr[p] * x[I.P.sp_col[p]];
    y[i] = sum;
}

// ---------------------------------------------------------------------------
// Schur-complement CG (eq. (schurcomp)). The m-vectors (c, r, p, q, dy) are in
// the numbering of J's rows; the n-vectors handed to the sweeps are in pivot
// order, so J^T v is written straight into the sweep vector (pivot position k
// holds column perm[k]) and J t reads the sweep output through j_colp.
//
// Iteration k is three launches around the sweep pair:
//   k_cg_dir  the stop tests of the iterate dy_k, then p_k = r_k + beta_k p_{k-1}
//             (row owners) and y = J^T p_k for the sweeps, each entry of p_k
//             formed on the fly by the same fma as its stored value;
//   k_cg_q    q = J K_gamma^{-1} J^T p_k and the partial sums of p.q;
//   k_cg_upd  alpha = r.r / p.q, dy += alpha p, r -= alpha q, and the partial
//             sums of r.r and maxima of |dy|.
// Each scalar (r.r, p.q, the norms) is reduced from the previous launch's
// per-workgroup partial sums by every workgroup that needs it, in one fixed
// order, so every workgroup takes the same decision without any
// synchronisation inside a launch; workgroup 0 of the instance records it.
// Every kernel returns at once when the instance's CG has stopped, so the
// iterations can be queued without reading decisions back.
//
// Reduction slots of one single factor (4 per part of a 256-row block of n, of
// which there are kRowSplit, and 4 per block of m):
//   N-region red[4 (kRowSplit b + part) + k], n-side blocks: 0 max row sum of
//                                          |A| (k_cg_rows, every part), 1 max
//                                          |f| (k_cg_fg, part 0); 2 max |r|,
//                                          3 max |J^T r| (k_cg_dir, eta test,
//                                          part 0); 0, 1 of every part again
//                                          for the final residual
//   M-region red[mslot0 + 4 b + k]:        0 r.r, 1 max |dy| (k_cg_c with
//                                          dy = 0, then k_cg_upd); 2 max |g|,
//                                          3 max row sum of |J| (k_cg_c)
//   Q-region red[qslot0 + 2 b + k]:        p.q (k_cg_q, stride 1); the final
//                                          residual's max |g - J dx|, |dy|
// ---------------------------------------------------------------------------
// deterministic block sum of v (every thread gets the sum)
__device__ inline double block_sum(double v) {
    __shared__ double sred[256];
    const int tid = threadIdx.x;
    sred[tid] = v;
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if (tid < h) sred[tid] += sred[tid + h];
        __syncthreads();
    }
    const double t = sred[0];
    __syncthreads();
    return t;
}

__device__ inline double block_max(double v) {
    __shared__ double smax[256];
    const int tid = threadIdx.x;
    smax[tid] = v;
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if (tid < h) smax[tid] = fmax(smax[tid], smax[tid + h]);
        __syncthreads();
    }
    const double t = smax[0];
    __syncthreads();
    return t;
}

__device__ __forceinline__ int cg_nb(int len) { return (len + 255) >> 8; }
// (the n-side region holds kRowSplit records per 256-row block)
__device__ __forceinline__ int cg_mslot0(const InstDev& I) { return 4 * kRowSplit * cg_nb(I.P.n); }
__device__ __forceinline__ int cg_qslot0(const InstDev& I) { return cg_mslot0(I) + 4 * cg_nb(I.P.m); }

// fixed-order sum / maximum over slot k of nb blocks (stride `stride`), eight
// loads in flight (indices past the end repeat the last slot: a maximum does
// not change, and a sum leaves them out)
template <class Use>
__device__ __forceinline__ void slots_each(const double* red, int nb, int stride, int k, Use&& use) {
    for (int b0 = threadIdx.x; b0 < nb; b0 += 8 * (int)blockDim.x) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; u++) t[u] = red[stride * min(b0 + u * (int)blockDim.x, nb - 1) + k];
#pragma unroll
        for (int u = 0; u < 8; u++)
            if (b0 + u * (int)blockDim.x < nb) use(t[u]);
    }
}
__device__ inline double slots_sum(const double* red, int nb, int stride, int k) {
    double v = 0.0;
    slots_each(red, nb, stride, k, [&](double t) { v += t; });
    return block_sum(v);
}
__device__ inline double slots_max(const double* red, int nb, int stride, int k) {
    double v = 0.0;
    slots_each(red, nb, stride, k, [&](double t) { v = fmax(v, t); });
    return block_max(v);
}
// maximum of the negated slots (a minimum, for slots that may all be positive)
__device__ inline double slots_max_neg(const double* red, int nb, int stride, int k) {
    double v = -INFINITY;
    for (int b = threadIdx.x; b < nb; b += blockDim.x) v = fmax(v, -red[stride * b + k]);
    return block_max(v);
}

// sum_q a[q] * v[idx[q]] over q in [q0, q1), four loads in flight per round,
// terms added in q order
template <class F>
__device__ __forceinline__ double gather_dot(int q0, int q1, const double* __restrict__ a,
                                             const int* __restrict__ idx, F&& v) {
    double s = 0.0;
    for (int q = q0; q < q1; q += 4) {
        int id[4];
        double av[4], xv[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int qc = min(q + u, q1 - 1);
            id[u] = idx[qc];
            av[u] = a[qc];
        }
#pragma unroll
        for (int u = 0; u < 4; u++) xv[u] = v(id[u]);
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (q + u < q1) s += av[u] * xv[u];
    }
    return s;
}

// Columns of J with more than kLongColumn entries (a stage's coupling
// variables hold about 70 where most columns hold three or four) are summed by
// 16-lane groups in workgroups of their own behind a kernel's row blocks; one
// lane alone takes two dependent memory round trips per four entries while
// its wave waits. Lane l loads terms l, l + 16, ...; every lane then adds all
// terms in column order, taking them from the lanes by row broadcasts, so the
// sum has the bits of the one-lane loop. (Distillation pattern, n = 142,000,
// 10,000 columns of 70 entries: k_cg_dir 35.8 -> 16.3 us; n = 21,371:
// k_aug_rhs 30.6 -> 6.2 us.)
__device__ __forceinline__ bool long_column(int q0, int q1) { return q1 - q0 > kLongColumn; }

// the column of this thread's group in workgroup b of the long columns (pivot
// position), or -1
__device__ __forceinline__ int group_column(const PatDev& P, int b) {
    const int h = b * 16 + (int)(threadIdx.x >> 4);
    return h < P.nlong ? P.jtp_long[h] : -1;
}

// term(q, a, x, y): entry q's coefficient and values; add(a, x, y) in column
// order (by every lane; terms past the end are zero)
template <class Term, class Add>
__device__ __forceinline__ void column_terms(int q0, int q1, Term&& term, Add&& add) {
    const int l = threadIdx.x & 15;
    for (int q = q0; q < q1; q += 64) {
        double a[4], x[4], y[4];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int qu = q + 16 * u + l;
            term(min(qu, q1 - 1), a[u], x[u], y[u]);
            a[u] = qu < q1 ? a[u] : 0.0;
            x[u] = qu < q1 ? x[u] : 0.0;
            y[u] = qu < q1 ? y[u] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (q + 16 * u < q1)
                static_for<16>([&](auto K) {
                    constexpr int k = K;
                    add(row_bcast<k>(a[u]), row_bcast<k>(x[u]), row_bcast<k>(y[u]));
                });
    }
}

// Sums over the entries p0 .. p1 - 1 of a row of a symmetric row list (or of a
// column of J) by a 16-lane group: lane l takes entries l, l + 16, ..., four
// of its entries in flight; term(p) gives an entry's coefficient and gathered
// value, add(a, t) takes it and their product. The lanes' sums are then
// combined by the caller.
template <class Term, class Add>
__device__ __forceinline__ void lane_terms(int64_t p0, int64_t p1, int l, Term&& term, Add&& add) {
    for (int64_t p = p0 + l; p < p1; p += 64) {
        double a[4], x[4];
#pragma unroll
        for (int u = 0; u < 4; u++) term(min(p + 16 * u, p1 - 1), a[u], x[u]);
#pragma unroll
        for (int u = 0; u < 4; u++)
            if (p + 16 * u < p1) add(a[u], a[u] * x[u]);
    }
}
__device__ __forceinline__ double sum16(double v) {
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v += __shfl_xor(v, o, 16);
    return v;
}
// Row kernels by 16-lane groups: kRowSplit workgroups of 256 threads share a
// 256-row item, each group takes kRowsPerGroup of their rows (one thread per
// row reads a wave's 64 rows, 20 to 140 entries each, uncoalesced and one
// round trip after another: measured on n = 142,000 k_cg_res_n 200 -> 46 us,
// on n = 21,371 k_aug_res_n 73 -> 16 us).
constexpr int kRowsPerGroup = 16 / kRowSplit;
// row t (0 .. kRowsPerGroup - 1) of this thread's group
__device__ __forceinline__ int group_row(const WorkItem& it, int t) {
    return it.id + (int)(blockIdx.x % kRowSplit) * 16 * kRowsPerGroup + 16 * t + (int)(threadIdx.x >> 4);
}
__device__ __forceinline__ int row_slot(const WorkItem& it) {
    return (it.id >> 8) * kRowSplit + (int)(blockIdx.x % kRowSplit);
}

// L-region red[lslot0 + b]: max |J^T r| over the 16 columns of long-column
// workgroup b (k_cg_dir, eta test)
__device__ __forceinline__ int cg_lslot0(const InstDev& I) { return cg_qslot0(I) + 2 * cg_nb(I.P.m); }

// f_gamma = f + gamma J^T g in pivot order (sweep vector and a copy for dx),
// the maximum of |f_i|, and the CG record's set-up (workgroup 0).
__global__ __launch_bounds__(256) void k_cg_fg(const InstDev* __restrict__ insts, Calls C,
                                               const WorkItem* __restrict__ items, int nitems, double tol, int maxit,
                                               double eta_tol) {
    const double* __restrict__ g = C.g;
    auto out = [&](const InstDev& I, int k, double sum) {
        const double v = C.f[I.n_off + I.P.perm[k]] + C.gamma * sum;
        I.fg[k] = v;
        I.y[k] = v;
    };
    if ((int)blockIdx.x >= nitems) {  // long columns
        const InstDev& I = insts[0];
        const int k = group_column(I.P, blockIdx.x - nitems);
        if (k < 0) return;
        double s = 0.0;
        column_terms(
            I.P.jtp_ptr[k], I.P.jtp_ptr[k + 1],
            [&](int q, double& a, double& x, double& y) {
                const int row = I.P.jtp_row[q];
                const bool eq = !C.eqm || C.eqm[row];
                a = eq ? I.jtv[q] : 0.0;
                x = eq ? g[row] : 0.0;
                y = 0.0;
            },
            [&](double a, double x, double) { s += a * x; });
        if ((threadIdx.x & 15) == 0) out(I, k, s);
        return;
    }
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (it.id == 0 && threadIdx.x == 0) {
        CgState* G = I.cg;
        G->tol = tol;
        G->maxit = maxit;
        G->eta_tol = eta_tol;
        G->it = 0;
        G->status = 0;
        G->done = 0;
        G->eta_stop = 0;
        G->eta = 0.0;
    }
    const int k = it.id + threadIdx.x;
    double fa = 0.0;
    if (k < I.P.n) {
        const int q0 = I.P.jtp_ptr[k], q1 = I.P.jtp_ptr[k + 1];
        if (!long_column(q0, q1)) {
            double s = 0.0;
            for (int q = q0; q < q1; q++) {
                const int row = I.P.jtp_row[q];
                if (C.eqm && !C.eqm[row]) continue;  // general HyKKT: equality rows only
                s += I.jtv[q] * g[row];
            }
            out(I, k, s);
        }
        fa = fabs(C.f[I.n_off + I.P.perm[k]]);
    }
    fa = block_max(fa);
    if (threadIdx.x == 0) I.red[4 * kRowSplit * (it.id >> 8) + 1] = fa;
}

// the maximum over the primal rows of the saddle matrix of sum_j |K0_ij| +
// sum_r |J_ri| (general HyKKT: equality rows of J only), original numbering
__global__ __launch_bounds__(256) void k_cg_rows(const InstDev* __restrict__ insts, Calls C,
                                                 const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x / kRowSplit];
    const InstDev& I = insts[it.inst];
    const int l = threadIdx.x & 15;
    double arow = 0.0;
#pragma unroll
    for (int t = 0; t < kRowsPerGroup; t++) {
        const int j = group_row(it, t);
        double s = 0.0;
        if (j < I.P.n) {
            lane_terms(
                I.P.sp_ptr[j], I.P.sp_ptr[j + 1], l,
                [&](int64_t p, double& a, double& x) {
                    a = I.k0csr[p];
                    x = 0.0;
                },
                [&](double a, double) { s += fabs(a); });
            lane_terms(
                I.P.jt_ptr[j], I.P.jt_ptr[j + 1], l,
                [&](int64_t q, double& a, double& x) {
                    a = !C.eqm || C.eqm[I.P.jt_row[q]] ? I.jraw[I.P.jt_e[q]] : 0.0;
                    x = 0.0;
                },
                [&](double a, double) { s += fabs(a); });
        }
        arow = fmax(arow, sum16(s));
    }
    arow = block_max(arow);
    if (threadIdx.x == 0) I.red[4 * row_slot(it)] = arow;
}

// After the sweeps: c = J K_gamma^{-1} f_gamma - g; r = c; p_old = 0; dy = 0;
// partial sums of c.c and the m-side norms.
__global__ __launch_bounds__(256) void k_cg_c(const InstDev* __restrict__ insts, Calls C,
                                              const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    double cc = 0.0, ga = 0.0, jrow = 0.0;
    if (i < I.P.m) {
        const int p0 = I.P.j_ptr[i], p1 = I.P.j_ptr[i + 1];
        const double* __restrict__ y = I.y;
        // general HyKKT: the inequality rows are not in the Schur system; their
        // entries of c, r, p and dy stay 0
        const bool eq = !C.eqm || C.eqm[i];
        const double s = gather_dot(p0, p1, I.jraw, I.P.j_colp, [&](int c) { return y[c]; });
        if (eq)
            for (int p = p0; p < p1; p++) jrow += fabs(I.jraw[p]);
        const double gi = eq ? C.g[I.m_off + i] : 0.0;
        const double ci = eq ? s - gi : 0.0;
        I.cvec[i] = ci;
        I.rvec[i] = ci;
        I.pvec2[i] = 0.0;
        C.dy[I.m_off + i] = 0.0;
        cc = ci * ci;
        ga = fabs(gi);
    }
    cc = block_sum(cc);
    ga = block_max(ga);
    jrow = block_max(jrow);
    if (threadIdx.x == 0) {
        double* s = I.red + cg_mslot0(I) + 4 * (it.id >> 8);
        s[0] = cc;
        s[1] = 0.0;  // ||dy_0||_inf
        s[2] = ga;
        s[3] = jrow;
    }
}

// Iteration k: stop tests of dy_k (r_k . r_k from the M-region partials),
// p_k = r_k + beta_k p_{k-1} for the instance's rows (row i by thread i of the
// n-side blocks; the Schur system needs m <= n) and y[k'] = (J^T p_k)_{perm[k']}.
// Stops: ||r_k||_2 <= tol ||c||_2 (converged) or k == maxit (NOT_CONVERGED).
// With eta_tol > 0 the maxima of |r_k| and |J^T r_k| go to the N-region for
// k_cg_eta_test.
__global__ __launch_bounds__(256) void k_cg_dir(const InstDev* __restrict__ insts,
                                                const WorkItem* __restrict__ items, int nitems, int k, int* ndone) {
    const bool longs = (int)blockIdx.x >= nitems;  // long columns (behind the row blocks)
    const WorkItem it = longs ? WorkItem{0, -1} : items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    CgState* G = I.cg;
    if (G->done) return;  // uniform per block
    const int nbm = cg_nb(I.P.m);
    const double rr = slots_sum(I.red + cg_mslot0(I), nbm, 4, 0);
    const double cnorm = k == 0 ? sqrt(rr) : G->cnorm;
    const bool conv = k == 0 ? rr == 0.0 : sqrt(rr) <= G->tol * cnorm;
    const bool lead = it.id == 0 && threadIdx.x == 0;
    if (conv || k >= G->maxit) {
        if (lead) {
            G->rr_new = rr;
            if (k == 0) G->cnorm = cnorm;
            G->it = k;
            G->status = conv ? 0 : 6;  // not converged after maxit iterations
            G->done = 1;
            atomicAdd(ndone, 1);
        }
        return;
    }
    const double beta = k == 0 ? 0.0 : rr / G->rrs[(k - 1) & 1];
    if (lead) {
        G->rrs[k & 1] = rr;
        G->rr_new = rr;
        G->it = k;
        if (k == 0) G->cnorm = cnorm;
    }
    const int parity = k & 1;
    double* __restrict__ pn = parity ? I.pvec2 : I.pvec;
    const double* __restrict__ po = parity ? I.pvec : I.pvec2;
    const double* __restrict__ r = I.rvec;
    const bool eta_test = G->eta_tol > 0.0;
    double ra = 0.0, ja = 0.0;
    if (longs) {
        const int kk = group_column(I.P, blockIdx.x - nitems);
        if (kk >= 0) {
            double s = 0.0, t = 0.0;
            column_terms(
                I.P.jtp_ptr[kk], I.P.jtp_ptr[kk + 1],
                [&](int q, double& a, double& x, double& y) {
                    const int row = I.P.jtp_row[q];
                    a = I.jtv[q];
                    y = r[row];
                    x = fma(beta, po[row], y);
                },
                [&](double a, double x, double y) {
                    s += a * x;
                    t += a * y;
                });
            if ((threadIdx.x & 15) == 0) I.y[kk] = s;
            ja = fabs(t);
        }
    } else {
        const int kk = it.id + threadIdx.x;
        if (kk < I.P.m) {
            pn[kk] = fma(beta, po[kk], r[kk]);
            ra = fabs(r[kk]);
        }
        const int q0 = kk < I.P.n ? I.P.jtp_ptr[kk] : 0, q1 = kk < I.P.n ? I.P.jtp_ptr[kk + 1] : 0;
        if (kk < I.P.n && !long_column(q0, q1)) {
            double s = 0.0, t = 0.0;
            for (int q = q0; q < q1; q += 4) {
                int row[4];
                double a[4], rv[4], pv[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int qc = min(q + u, q1 - 1);
                    row[u] = I.P.jtp_row[qc];
                    a[u] = I.jtv[qc];
                }
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    rv[u] = r[row[u]];
                    pv[u] = po[row[u]];
                }
#pragma unroll
                for (int u = 0; u < 4; u++)
                    if (q + u < q1) {
                        s += a[u] * fma(beta, pv[u], rv[u]);
                        t += a[u] * rv[u];
                    }
            }
            I.y[kk] = s;
            ja = fabs(t);
        }
    }
    if (!eta_test) return;  // uniform per launch
    ra = block_max(ra);
    ja = block_max(ja);
    if (threadIdx.x == 0) {
        if (longs) {
            I.red[cg_lslot0(I) + blockIdx.x - nitems] = ja;
            return;
        }
        double* sl = I.red + 4 * kRowSplit * (it.id >> 8);
        sl[2] = ra;
        sl[3] = ja;
    }
}

// eta_tol > 0, one workgroup per instance, between k_cg_dir and the sweeps:
// for dx = K_gamma^{-1}(f_gamma - J^T dy) the saddle system's residual is
// (gamma J^T r, r), so
//   max(gamma ||J^T r||_inf, ||r||_inf) / (||A||_inf ||dy||_inf + ||(f, g)||_inf)
// bounds its normwise backward error from above (the denominator leaves out
// ||dx||); the CG stops at dy_k when the bound is <= eta_tol.
__global__ __launch_bounds__(256) void k_cg_eta_test(const InstDev* __restrict__ insts, Calls C, int k,
                                                     int* ndone) {
    const InstDev& I = insts[blockIdx.x];
    CgState* G = I.cg;
    if (G->done || !(G->eta_tol > 0.0)) return;  // uniform
    const int nbn = cg_nb(I.P.n), nbm = cg_nb(I.P.m);
    const double* Nr = I.red;
    const double* Mr = I.red + cg_mslot0(I);
    const double norm_a = fmax(slots_max(Nr, kRowSplit * nbn, 4, 0), slots_max(Mr, nbm, 4, 3));
    const double norm_rhs = fmax(slots_max(Nr, nbn, 4 * kRowSplit, 1), slots_max(Mr, nbm, 4, 2));
    const double rmax = slots_max(Nr, nbn, 4 * kRowSplit, 2);
    const double jrmax = fmax(slots_max(Nr, nbn, 4 * kRowSplit, 3), slots_max(I.red + cg_lslot0(I), (I.P.nlong + 15) >> 4, 1, 0));
    const double dymax = slots_max(Mr, nbm, 4, 1);
    if (threadIdx.x == 0) {
        G->norm_a = norm_a;
        G->norm_rhs = norm_rhs;
        G->rmax = rmax;
        G->dymax = dymax;
        if (fmax(C.gamma * jrmax, rmax) <= G->eta_tol * (norm_a * dymax + norm_rhs)) {
            G->it = k;
            G->done = 1;
            G->eta_stop = 1;
            atomicAdd(ndone, 1);
        }
    }
}

// q = J t with t = K_gamma^{-1} J^T p_k (the sweep output, pivot order) and the
// partial sums of p_k . q
__global__ __launch_bounds__(256) void k_cg_q(const InstDev* __restrict__ insts, Calls C,
                                              const WorkItem* __restrict__ items, int k) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (I.cg->done) return;  // uniform per block
    const double* __restrict__ pn = (k & 1) ? I.pvec2 : I.pvec;
    const int i = it.id + threadIdx.x;
    double v = 0.0;
    if (i < I.P.m) {
        const double* __restrict__ y = I.y;
        double s = gather_dot(I.P.j_ptr[i], I.P.j_ptr[i + 1], I.jraw, I.P.j_colp, [&](int c) { return y[c]; });
        if (C.eqm && !C.eqm[i]) s = 0.0;  // general HyKKT: equality rows only
        I.qvec[i] = s;
        v = pn[i] * s;
    }
    v = block_sum(v);
    if (threadIdx.x == 0) I.red[cg_qslot0(I) + (it.id >> 8)] = v;
}

// alpha = r_k . r_k / p_k . q (p_k^T S p_k <= 0: BREAKDOWN), dy += alpha p_k,
// r -= alpha q, and the partial sums of r.r and maxima of |dy|.
__global__ __launch_bounds__(256) void k_cg_upd(const InstDev* __restrict__ insts, Calls C,
                                                const WorkItem* __restrict__ items, int k, int* ndone) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    CgState* G = I.cg;
    if (G->done) return;  // uniform per block
    const int nbm = cg_nb(I.P.m);
    const double pq = slots_sum(I.red + cg_qslot0(I), nbm, 1, 0);
    if (!(pq > 0.0)) {
        if (it.id == 0 && threadIdx.x == 0) {
            G->pq = pq;
            G->it = k;
            G->status = 7;  // breakdown
            G->done = 1;
            atomicAdd(ndone, 1);
        }
        return;
    }
    const double a = G->rrs[k & 1] / pq;
    const double* __restrict__ pn = (k & 1) ? I.pvec2 : I.pvec;
    const int i = it.id + threadIdx.x;
    double rr = 0.0, da = 0.0;
    if (i < I.P.m) {
        double* dy = C.dy + I.m_off;
        const double d = fma(a, pn[i], dy[i]);
        dy[i] = d;
        const double ri = fma(-a, I.qvec[i], I.rvec[i]);
        I.rvec[i] = ri;
        rr = ri * ri;
        da = fabs(d);
    }
    rr = block_sum(rr);
    da = block_max(da);
    if (threadIdx.x == 0) {
        double* s = I.red + cg_mslot0(I) + 4 * (it.id >> 8);
        s[0] = rr;
        s[1] = da;
    }
}

// right-hand side of the last solve: y[k] = f_gamma[k] - (J^T dy)_{perm[k]}
__global__ __launch_bounds__(256) void k_cg_dxrhs(const InstDev* __restrict__ insts, Calls C,
                                                  const WorkItem* __restrict__ items, int nitems) {
    const bool longs = (int)blockIdx.x >= nitems;
    const WorkItem it = longs ? WorkItem{0, -1} : items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const double* __restrict__ dy = C.dy + I.m_off;
    const int k = longs ? group_column(I.P, blockIdx.x - nitems) : it.id + (int)threadIdx.x;
    if (k < 0 || k >= I.P.n) return;
    const int q0 = I.P.jtp_ptr[k], q1 = I.P.jtp_ptr[k + 1];
    if (longs) {
        double s = 0.0;
        column_terms(
            q0, q1,
            [&](int q, double& a, double& x, double& y) {
                a = I.jtv[q];
                x = dy[I.P.jtp_row[q]];
                y = 0.0;
            },
            [&](double a, double x, double) { s += a * x; });
        if ((threadIdx.x & 15) == 0) I.y[k] = I.fg[k] - s;
    } else if (!long_column(q0, q1)) {
        I.y[k] = I.fg[k] - gather_dot(q0, q1, I.jtv, I.P.jtp_row, [&](int r) { return dy[r]; });
    }
}

// Saddle-system residual of (dx, dy): rows of the primal block,
// f - K0 dx - J^T dy (original numbering), with the maxima of |res| and |dx|.
__global__ __launch_bounds__(256) void k_cg_res_n(const InstDev* __restrict__ insts, Calls C,
                                                  const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x / kRowSplit];
    const InstDev& I = insts[it.inst];
    const int l = threadIdx.x & 15;
    const double* __restrict__ dx = C.dx + I.n_off;
    const double* __restrict__ dy = C.dy + I.m_off;
    double ra = 0.0, xa = 0.0;
#pragma unroll
    for (int t = 0; t < kRowsPerGroup; t++) {
        const int j = group_row(it, t);
        double s = 0.0;
        if (j < I.P.n) {
            lane_terms(
                I.P.sp_ptr[j], I.P.sp_ptr[j + 1], l,
                [&](int64_t p, double& a, double& x) {
                    a = I.k0csr[p];
                    x = dx[I.P.sp_col[p]];
                },
                [&](double, double ax) { s += ax; });
            lane_terms(
                I.P.jt_ptr[j], I.P.jt_ptr[j + 1], l,
                [&](int64_t q, double& a, double& x) {
                    a = I.jraw[I.P.jt_e[q]];
                    x = dy[I.P.jt_row[q]];
                },
                [&](double, double ax) { s += ax; });
        }
        s = sum16(s);
        if (l == 0 && j < I.P.n) {
            ra = fmax(ra, fabs(C.f[I.n_off + j] - s));
            xa = fmax(xa, fabs(dx[j]));
        }
    }
    ra = block_max(ra);
    xa = block_max(xa);
    if (threadIdx.x == 0) {
        double* sl = I.red + 4 * row_slot(it);
        sl[0] = ra;
        sl[1] = xa;
    }
}

// constraint rows, g - J dx, with |dy|
__global__ __launch_bounds__(256) void k_cg_res_m(const InstDev* __restrict__ insts, Calls C,
                                                  const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    double ra = 0.0, ya = 0.0;
    if (i < I.P.m && (!C.eqm || C.eqm[i])) {  // general HyKKT: equality rows only
        const double* __restrict__ dx = C.dx + I.n_off;
        double s = 0.0;
        for (int p = I.P.j_ptr[i]; p < I.P.j_ptr[i + 1]; p++) s += I.jraw[p] * dx[I.P.j_col[p]];
        ra = fabs(C.g[I.m_off + i] - s);
        ya = fabs(C.dy[I.m_off + i]);
    }
    ra = block_max(ra);
    ya = block_max(ya);
    if (threadIdx.x == 0) {
        double* s = I.red + cg_qslot0(I) + 2 * (it.id >> 8);
        s[0] = ra;
        s[1] = ya;
    }
}

// one workgroup per instance: eta = ||res||_inf / (||A||_inf ||(dx, dy)||_inf
// + ||(f, g)||_inf) from the residual kernels' maxima and the norms kept in
// the record by k_cg_norms
__global__ __launch_bounds__(256) void k_cg_eta(const InstDev* __restrict__ insts) {
    const InstDev& I = insts[blockIdx.x];
    CgState* G = I.cg;
    const int nbn = cg_nb(I.P.n), nbm = cg_nb(I.P.m);
    const double* Nr = I.red;
    const double* Qr = I.red + cg_qslot0(I);
    const double r1 = slots_max(Nr, kRowSplit * nbn, 4, 0), x1 = slots_max(Nr, kRowSplit * nbn, 4, 1);
    const double r2 = slots_max(Qr, nbm, 2, 0), y2 = slots_max(Qr, nbm, 2, 1);
    if (threadIdx.x == 0) {
        const double den = G->norm_a * fmax(x1, y2) + G->norm_rhs;
        const double res = fmax(r1, r2);
        G->eta = den > 0.0 ? res / den : (res > 0.0 ? INFINITY : 0.0);
    }
}

// one workgroup per instance, before the iterations: ||A||_inf (the n-side
// part) and ||f||_inf from k_cg_fg's partials, kept in the record (the eta
// test and the final residual overwrite the N-region)
__global__ __launch_bounds__(256) void k_cg_norms(const InstDev* __restrict__ insts) {
    const InstDev& I = insts[blockIdx.x];
    CgState* G = I.cg;
    const int nbn = cg_nb(I.P.n), nbm = cg_nb(I.P.m);
    const double* Mr = I.red + cg_mslot0(I);
    const double an = fmax(slots_max(I.red, kRowSplit * nbn, 4, 0), slots_max(Mr, nbm, 4, 3));
    const double fm = fmax(slots_max(I.red, nbn, 4 * kRowSplit, 1), slots_max(Mr, nbm, 4, 2));
    if (threadIdx.x == 0) {
        G->norm_a = an;
        G->norm_rhs = fm;
    }
}

// ---------------------------------------------------------------------------
// Augmented system of eq. (kkt:augmented) with no equality rows (the Lifted-KKT
// form, H = J, D_s = Sigma_s), regularised on the Hessian block as the
// condensed matrix K = W + Sigma_x + delta I + J^T Sigma_s J is:
//   [[K0, 0, J^T], [0, Sigma_s, I], [J, I, 0]] [dx; ds; dz] = -[r1; r2; r4],
// K0 = W + Sigma_x + delta I. Condensation (eq. (kkt:condensed)) gives
// K dx = -(r1 + J^T (Sigma_s r4 - r2)), and the slack and multiplier steps
// follow as ds = -r4 - J dx, dz = -r2 - Sigma_s ds. The refinement on the
// full system (section "Hybrid linear solver") takes the residual e of the
// augmented system and solves for the correction the same way.
// Slots: N-region 8 per part of a 256-row block, kRowSplit parts a block
// (k_aug_res_n), M-region 8 per block after it.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int aug_mslot0(const InstDev& I) { return 8 * kRowSplit * cg_nb(I.P.n); }

// b_j = p1_j - sum_q J_qj (p2_q - Sigma_s,q p4_q) with p = -r (mode 0) or
// p = e (mode 1); pivot-ordered threads, b in original numbering
__global__ __launch_bounds__(256) void k_aug_rhs(const InstDev* __restrict__ insts, AugCall A,
                                                 const WorkItem* __restrict__ items, int nitems, int mode) {
    const bool longs = (int)blockIdx.x >= nitems;
    const WorkItem it = longs ? WorkItem{0, -1} : items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (mode == 1 && I.aug->done) return;  // uniform per block
    const int k = longs ? group_column(I.P, blockIdx.x - nitems) : it.id + (int)threadIdx.x;
    if (k < 0 || k >= I.P.n) return;
    const int n = I.P.n, m = I.P.m;
    const int j = I.P.perm[k];
    const double* __restrict__ p2 = mode ? I.aug_e + n : A.r2;
    const double* __restrict__ p4 = mode ? I.aug_e + n + m : A.r4;
    const double sgn = mode ? 1.0 : -1.0;
    const int q0 = I.P.jtp_ptr[k], q1 = I.P.jtp_ptr[k + 1];
    double s = 0.0;
    if (longs) {
        column_terms(
            q0, q1,
            [&](int q, double& a, double& x, double& y) {
                const int row = I.P.jtp_row[q];
                a = I.jtv[q];
                x = sgn * p2[row] - I.ssv[row] * (sgn * p4[row]);
                y = 0.0;
            },
            [&](double a, double x, double) { s += a * x; });
        if ((threadIdx.x & 15) != 0) return;
    } else {
        if (long_column(q0, q1)) return;
        s = gather_dot(q0, q1, I.jtv, I.P.jtp_row,
                       [&](int row) { return sgn * p2[row] - I.ssv[row] * (sgn * p4[row]); });
    }
    const double p1 = mode ? I.aug_e[j] : -A.r1[j];
    I.aug_b[j] = p1 - s;
}

// mode 0: ds = p4 - J dx, dz = p2 - Sigma_s ds with p = -r.
// mode 1: t = K^{-1} b is in aug_t; the iterate moves to aug_prev and
// dx += t, ds += e4 - J t, dz += e2 - Sigma_s (e4 - J t).
__global__ __launch_bounds__(256) void k_aug_recover_m(const InstDev* __restrict__ insts, AugCall A,
                                                       const WorkItem* __restrict__ items, int mode) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (mode == 1 && I.aug->done) return;
    const int i = it.id + threadIdx.x;
    if (i >= I.P.m) return;
    const int n = I.P.n, m = I.P.m;
    const double* __restrict__ v = mode ? I.aug_t : A.dx;
    double s = 0.0;
    for (int p = I.P.j_ptr[i]; p < I.P.j_ptr[i + 1]; p++) s += I.jraw[p] * v[I.P.j_col[p]];
    const double p2 = mode ? I.aug_e[n + i] : -A.r2[i];
    const double p4 = mode ? I.aug_e[n + m + i] : -A.r4[i];
    const double ds = p4 - s;
    const double dz = p2 - I.ssv[i] * ds;
    if (mode == 0) {
        A.ds[i] = ds;
        A.dz[i] = dz;
    } else {
        const double so = A.ds[i], zo = A.dz[i];
        I.aug_prev[n + i] = so;
        I.aug_prev[n + m + i] = zo;
        A.ds[i] = so + ds;
        A.dz[i] = zo + dz;
    }
}

__global__ __launch_bounds__(256) void k_aug_update_x(const InstDev* __restrict__ insts, AugCall A,
                                                      const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (I.aug->done) return;
    const int j = it.id + threadIdx.x;
    if (j >= I.P.n) return;
    const double xo = A.dx[j];
    I.aug_prev[j] = xo;
    A.dx[j] = xo + I.aug_t[j];
}

__global__ void k_aug_reset(const InstDev* __restrict__ insts, int ninst, double tol, int maxit) {
    const int q = blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= ninst) return;
    AugState* S = insts[q].aug;
    S->eta = S->eta_prev = S->omega = S->omega_prev = INFINITY;
    S->tol = tol;
    S->maxit = maxit;
    S->it = 0;
    S->done = 0;
    S->revert = 0;
}

// ratio for the componentwise backward error (0/0 taken as 0)
__device__ __forceinline__ double aug_ratio(double r, double den) {
    return den > 0.0 ? r / den : (r > 0.0 ? INFINITY : 0.0);
}

// primal rows: e1 = -r1 - K0 dx - J^T dz, with |K0||dx| + |J|^T|dz| + |r1|,
// the row sums of |A| and the maxima of |dx| and |r1|
__global__ __launch_bounds__(256) void k_aug_res_n(const InstDev* __restrict__ insts, AugCall A,
                                                   const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x / kRowSplit];
    const InstDev& I = insts[it.inst];
    if (I.aug->done) return;
    const int l = threadIdx.x & 15;
    double ea = 0.0, om = 0.0, ar = 0.0, xa = 0.0, ba = 0.0;
#pragma unroll
    for (int t = 0; t < kRowsPerGroup; t++) {
        const int j = group_row(it, t);
        double s = 0.0, den = 0.0, rs = 0.0;
        auto add = [&](double a, double ax) {
            s += ax;
            den += fabs(ax);
            rs += fabs(a);
        };
        if (j < I.P.n) {
            lane_terms(
                I.P.sp_ptr[j], I.P.sp_ptr[j + 1], l,
                [&](int64_t p, double& a, double& x) {
                    a = I.k0csr[p];
                    x = A.dx[I.P.sp_col[p]];
                },
                add);
            lane_terms(
                I.P.jt_ptr[j], I.P.jt_ptr[j + 1], l,
                [&](int64_t q, double& a, double& x) {
                    a = I.jraw[I.P.jt_e[q]];
                    x = A.dz[I.P.jt_row[q]];
                },
                add);
        }
        s = sum16(s);
        den = sum16(den);
        rs = sum16(rs);
        if (l == 0 && j < I.P.n) {
            const double p1 = -A.r1[j];
            const double e1 = p1 - s;
            I.aug_e[j] = e1;
            ea = fmax(ea, fabs(e1));
            om = fmax(om, aug_ratio(fabs(e1), den + fabs(p1)));
            ar = fmax(ar, rs);
            xa = fmax(xa, fabs(A.dx[j]));
            ba = fmax(ba, fabs(p1));
        }
    }
    ea = block_max(ea);
    om = block_max(om);
    ar = block_max(ar);
    xa = block_max(xa);
    ba = block_max(ba);
    if (threadIdx.x == 0) {
        double* sl = I.red + 8 * row_slot(it);
        sl[0] = ea;
        sl[1] = om;
        sl[2] = ar;
        sl[3] = xa;
        sl[4] = ba;
    }
}

// slack rows e2 = -r2 - Sigma_s ds - dz and constraint rows e4 = -r4 - J dx - ds
__global__ __launch_bounds__(256) void k_aug_res_m(const InstDev* __restrict__ insts, AugCall A,
                                                   const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (I.aug->done) return;
    const int i = it.id + threadIdx.x;
    const int n = I.P.n, m = I.P.m;
    double ea = 0.0, om = 0.0, ar = 0.0, xa = 0.0, ba = 0.0;
    if (i < m) {
        const double sg = I.ssv[i], ds = A.ds[i], dz = A.dz[i];
        const double p2 = -A.r2[i], p4 = -A.r4[i];
        const double t2 = sg * ds;
        const double e2 = p2 - t2 - dz;
        double s = 0.0, den4 = 0.0, rs4 = 0.0;
        for (int p = I.P.j_ptr[i]; p < I.P.j_ptr[i + 1]; p++) {
            const double a = I.jraw[p], t = a * A.dx[I.P.j_col[p]];
            s += t;
            den4 += fabs(t);
            rs4 += fabs(a);
        }
        const double e4 = p4 - s - ds;
        I.aug_e[n + i] = e2;
        I.aug_e[n + m + i] = e4;
        ea = fmax(fabs(e2), fabs(e4));
        om = fmax(aug_ratio(fabs(e2), fabs(t2) + fabs(dz) + fabs(p2)),
                  aug_ratio(fabs(e4), den4 + fabs(ds) + fabs(p4)));
        ar = fmax(sg + 1.0, rs4 + 1.0);
        xa = fmax(fabs(ds), fabs(dz));
        ba = fmax(fabs(p2), fabs(p4));
    }
    ea = block_max(ea);
    om = block_max(om);
    ar = block_max(ar);
    xa = block_max(xa);
    ba = block_max(ba);
    if (threadIdx.x == 0) {
        double* sl = I.red + aug_mslot0(I) + 8 * (it.id >> 8);
        sl[0] = ea;
        sl[1] = om;
        sl[2] = ar;
        sl[3] = xa;
        sl[4] = ba;
    }
}

// one workgroup per instance: eta and omega of the augmented system, and the
// stop rule of the refinement (omega <= tol, maxit corrections, or omega not
// halving; the previous iterate wins if omega grew)
__global__ __launch_bounds__(256) void k_aug_decide(const InstDev* __restrict__ insts) {
    const InstDev& I = insts[blockIdx.x];
    AugState* S = I.aug;
    if (S->done) return;
    const int nbn = cg_nb(I.P.n), nbm = cg_nb(I.P.m);
    const double* Nr = I.red;
    const double* Mr = I.red + aug_mslot0(I);
    double v[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 5; k++) {
        slots_each(Nr, kRowSplit * nbn, 8, k, [&](double t) { v[k] = fmax(v[k], t); });
        slots_each(Mr, nbm, 8, k, [&](double t) { v[k] = fmax(v[k], t); });
    }
    __shared__ double top[5];
    block_max5(v[0], v[1], v[2], v[3], v[4], top);
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 0; k < 5; k++) v[k] = top[k];
    const double den = v[2] * v[3] + v[4];
    S->eta_prev = S->eta;
    S->omega_prev = S->omega;
    S->eta = den > 0.0 ? v[0] / den : (v[0] > 0.0 ? INFINITY : 0.0);
    S->omega = v[1];
    bool stop = S->omega <= S->tol || S->it >= S->maxit;
    if (S->it > 0 && S->omega > 0.5 * S->omega_prev) {
        stop = true;
        if (S->omega > S->omega_prev) S->revert = 1;
    }
    if (stop) S->done = 1;
    else S->it += 1;
}

__global__ __launch_bounds__(256) void k_aug_revert_n(const InstDev* __restrict__ insts, AugCall A,
                                                      const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (!I.aug->revert) return;
    const int j = it.id + threadIdx.x;
    if (j < I.P.n) A.dx[j] = I.aug_prev[j];
}

__global__ __launch_bounds__(256) void k_aug_revert_m(const InstDev* __restrict__ insts, AugCall A,
                                                      const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    if (!I.aug->revert) return;
    const int i = it.id + threadIdx.x;
    if (i >= I.P.m) return;
    A.ds[i] = I.aug_prev[I.P.n + i];
    A.dz[i] = I.aug_prev[I.P.n + I.P.m + i];
}

// ---------------------------------------------------------------------------
// Interior-point loop (section "INTERIOR-POINT METHOD": the smoothed KKT
// system eq. (smoothkkt), Newton steps eq. (newtonstep) through the
// augmented system, fraction-to-boundary steps) on the convex QP
//   min 1/2 x^T W x + c^T x  s.t.  J x + s = u, s >= 0,
// multipliers z, D_s = S^{-1} Z. Per iteration (vectors in original numbering):
//   r1 = W x + c + J^T z, r4 = J x + s - u, gap = s^T z / m,
//   err = max(||r1|| / (1 + ||c||), ||r4|| / (1 + ||u||), gap) (inf-norms),
//   mu = sigma gap, r2 = z - mu / s, tau = max(tau_min, 1 - mu),
//   the Newton step (dx, ds, dz) from the augmented system, the largest
//   alpha_p, alpha_d <= 1 keeping s and z above (1 - tau) of their values.
// W x comes from the factor's kept K0 = W + delta I (Sigma_x = 0).
// Slots: red[4 (kRowSplit b + part) + k] for the n-side (nbn blocks; k_ipm_norm_n
// uses the first nbn records), red[4 kRowSplit nbn + 4 b + k] for the m-side.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int ipm_m0(const InstDev& I) { return 4 * kRowSplit * cg_nb(I.P.n); }

// n-side: max |c|; m-side: max |u|; then the record (one workgroup per
// instance reduces in the second kernel)
__global__ __launch_bounds__(256) void k_ipm_norm_n(const InstDev* __restrict__ insts, IpmCall P,
                                                    const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int j = it.id + threadIdx.x;
    const double v = block_max(j < I.P.n ? fabs(P.c[j]) : 0.0);
    if (threadIdx.x == 0) P.red[4 * (it.id >> 8)] = v;
}
__global__ __launch_bounds__(256) void k_ipm_norm_m(const InstDev* __restrict__ insts, IpmCall P,
                                                    const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    const double v = block_max(i < I.P.m ? fabs(P.u[i]) : 0.0);
    if (threadIdx.x == 0) P.red[ipm_m0(I) + 4 * (it.id >> 8)] = v;
}
__global__ __launch_bounds__(256) void k_ipm_init(const InstDev* __restrict__ insts, IpmCall P, double tol, int maxit,
                                                  double sigma, double tau_min) {
    const InstDev& I = insts[0];
    const double cm = slots_max(P.red, cg_nb(I.P.n), 4, 0);
    const double um = slots_max(P.red + ipm_m0(I), cg_nb(I.P.m), 4, 0);
    if (threadIdx.x != 0) return;
    IpmState* S = P.st;
    S->cn = 1.0 + cm;
    S->un = 1.0 + um;
    S->tol = tol;
    S->maxit = maxit;
    S->sigma = sigma;
    S->tau_min = tau_min;
    S->it = 0;
    S->done = 0;
    S->status = 0;
    S->mu = S->gap = S->err = S->r1max = S->r4max = S->ap = S->ad = S->delta = 0.0;
}

// D_s = z / s, the slack weights of the refactor
__global__ __launch_bounds__(256) void k_ipm_dsw(const InstDev* __restrict__ insts, IpmCall P,
                                                 const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    if (i < I.P.m) P.dsw[i] = P.z[i] / P.s[i];
}

// r1 = (K0 - delta I) x + c + J^T z
__global__ __launch_bounds__(256) void k_ipm_res_n(const InstDev* __restrict__ insts, IpmCall P,
                                                   const WorkItem* __restrict__ items, double delta) {
    const WorkItem it = items[blockIdx.x / kRowSplit];
    const InstDev& I = insts[it.inst];
    const int l = threadIdx.x & 15;
    double ra = 0.0;
#pragma unroll
    for (int u = 0; u < kRowsPerGroup; u++) {
        const int j = group_row(it, u);
        double s = 0.0, t = 0.0;
        if (j < I.P.n) {
            lane_terms(
                I.P.sp_ptr[j], I.P.sp_ptr[j + 1], l,
                [&](int64_t p, double& a, double& x) {
                    a = I.k0csr[p];
                    x = P.x[I.P.sp_col[p]];
                },
                [&](double, double ax) { s += ax; });
            lane_terms(
                I.P.jt_ptr[j], I.P.jt_ptr[j + 1], l,
                [&](int64_t q, double& a, double& x) {
                    a = P.jv[I.P.jt_e[q]];
                    x = P.z[I.P.jt_row[q]];
                },
                [&](double, double ax) { t += ax; });
        }
        s = sum16(s);
        t = sum16(t);
        if (l == 0 && j < I.P.n) {
            const double r = s - delta * P.x[j] + P.c[j] + t;
            P.r1[j] = r;
            ra = fmax(ra, fabs(r));
        }
    }
    ra = block_max(ra);
    if (threadIdx.x == 0) P.red[4 * row_slot(it)] = ra;
}

// r4 = J x + s - u, partial s^T z
__global__ __launch_bounds__(256) void k_ipm_res_m(const InstDev* __restrict__ insts, IpmCall P,
                                                   const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    double ra = 0.0, sz = 0.0;
    if (i < I.P.m) {
        double t = 0.0;
        for (int p = I.P.j_ptr[i]; p < I.P.j_ptr[i + 1]; p++) t += P.jv[p] * P.x[I.P.j_col[p]];
        const double r = t + P.s[i] - P.u[i];
        P.r4[i] = r;
        ra = fabs(r);
        sz = P.s[i] * P.z[i];
    }
    ra = block_max(ra);
    sz = block_sum(sz);
    if (threadIdx.x == 0) {
        double* sl = P.red + ipm_m0(I) + 4 * (it.id >> 8);
        sl[0] = ra;
        sl[1] = sz;
    }
}

// the stop test and mu, tau of this iteration
__global__ __launch_bounds__(256) void k_ipm_decide(const InstDev* __restrict__ insts, IpmCall P, double delta) {
    const InstDev& I = insts[0];
    const int nbn = cg_nb(I.P.n), nbm = cg_nb(I.P.m);
    const double r1 = slots_max(P.red, kRowSplit * nbn, 4, 0);
    const double r4 = slots_max(P.red + ipm_m0(I), nbm, 4, 0);
    const double sz = slots_sum(P.red + ipm_m0(I), nbm, 4, 1);
    if (threadIdx.x != 0) return;
    IpmState* S = P.st;
    S->r1max = r1;
    S->r4max = r4;
    S->delta = fmax(S->delta, delta);
    S->gap = I.P.m > 0 ? sz / I.P.m : 0.0;
    S->err = fmax(fmax(r1 / S->cn, r4 / S->un), S->gap);
    if (S->err <= S->tol) {
        S->done = 1;
    } else if (S->it >= S->maxit) {
        S->done = 1;
        S->status = 6;  // not converged
    } else {
        S->mu = S->sigma * S->gap;
        S->tau = fmax(S->tau_min, 1.0 - S->mu);
    }
}

// r2 = z - mu / s
__global__ __launch_bounds__(256) void k_ipm_r2(const InstDev* __restrict__ insts, IpmCall P,
                                                const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    if (i < I.P.m) P.r2[i] = P.z[i] - P.st->mu / P.s[i];
}

// fraction to the boundary: per block the smallest -tau v / dv over dv < 0
// (2 when no entry decreases), for s and for z
__global__ __launch_bounds__(256) void k_ipm_alpha(const InstDev* __restrict__ insts, IpmCall P,
                                                   const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    const double tau = P.st->tau;
    double as = 2.0, az = 2.0;
    if (i < I.P.m) {
        if (P.ds[i] < 0.0) as = -tau * P.s[i] / P.ds[i];
        if (P.dz[i] < 0.0) az = -tau * P.z[i] / P.dz[i];
    }
    as = -block_max(-as);
    az = -block_max(-az);
    if (threadIdx.x == 0) {
        double* sl = P.red + ipm_m0(I) + 4 * (it.id >> 8);
        sl[2] = as;
        sl[3] = az;
    }
}

__global__ __launch_bounds__(256) void k_ipm_alpha_fin(const InstDev* __restrict__ insts, IpmCall P) {
    const InstDev& I = insts[0];
    const int nbm = cg_nb(I.P.m);
    const double as = -slots_max_neg(P.red + ipm_m0(I), nbm, 4, 2);
    const double az = -slots_max_neg(P.red + ipm_m0(I), nbm, 4, 3);
    if (threadIdx.x != 0) return;
    P.st->ap = fmin(1.0, as);
    P.st->ad = fmin(1.0, az);
    P.st->it += 1;
}

// x += alpha_p dx (n-side blocks); s += alpha_p ds, z += alpha_d dz (m-side)
__global__ __launch_bounds__(256) void k_ipm_update_n(const InstDev* __restrict__ insts, IpmCall P,
                                                      const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int j = it.id + threadIdx.x;
    if (j < I.P.n) P.x[j] = fma(P.st->ap, P.dx[j], P.x[j]);
}
__global__ __launch_bounds__(256) void k_ipm_update_m(const InstDev* __restrict__ insts, IpmCall P,
                                                      const WorkItem* __restrict__ items) {
    const WorkItem it = items[blockIdx.x];
    const InstDev& I = insts[it.inst];
    const int i = it.id + threadIdx.x;
    if (i < I.P.m) {
        P.s[i] = fma(P.st->ap, P.ds[i], P.s[i]);
        P.z[i] = fma(P.st->ad, P.dz[i], P.z[i]);
    }
}

// ---------------------------------------------------------------------------
// Stage-structured solver: the condensed matrix of a dynamic program is
// block-banded (section "Future Works"); with stage-contiguous variables and
// couplings between consecutive stages only, K is block tridiagonal and is
// factored here by block cyclic reduction: the stages at odd positions of the
// active chain are eliminated together (one workgroup each), the rest form
// the next, half as long, chain. This is a Cholesky factorization of K in
// the cyclic-reduction order, with dense blocks: per eliminated stage k with
// active neighbours l and r, the front [D_k; K(l,k); K(r,k)] is factored,
//   L_k = chol(D_k),  L(l,k) = K(l,k) L_k^{-T},  L(r,k) = K(r,k) L_k^{-T},
// and it leaves to the next level the updates L(l,k) L(l,k)^T (to D_l),
// L(r,k) L(r,k)^T (to D_r) and the fill K(r,l) = -L(r,k) L(l,k)^T. Every
// launch also runs one workgroup per stage that stays in the chain, which
// applies the updates of the previous level to its D (so each stage takes at
// most two updates, from the level just before). K itself comes from the
// general assembly (kcsr), so its entries are the same bits as the
// supernodal path's.
// ---------------------------------------------------------------------------
// 1/d: the hardware reciprocal estimate refined by two steps of Newton's
// iteration r <- r + r (1 - d r), each of which doubles the correct bits
__device__ __forceinline__ double recip_f64(double d) {
    double r = __builtin_amdgcn_rcp(d);
    r = fma(r, fma(-d, r, 1.0), r);
    r = fma(r, fma(-d, r, 1.0), r);
    return r;
}

__global__ void k_fill_f64(double* __restrict__ p, double v, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ __launch_bounds__(256) void k_cr_scatter(const InstDev* __restrict__ insts, CrArrays A,
                                                    const CrScatter* __restrict__ items, int64_t nitems) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nitems) return;
    const CrScatter it = items[t];
    const double v = insts[it.inst].kcsr[it.pos];
    if (it.dst >= 0) A.D[it.dst] = v;
    else A.C[-it.dst - 1] = v;
}

// One workgroup per task of one level (NB: stage widths <= 16 NB). A task
// eliminates its stage or applies the previous level's updates to a stage
// that stays. Thread (ti, tc) = (tid % 16, tid / 16)
// holds the front entries of rows ti + 16 a and columns tc + 16 b in
// registers. The front's rows: [0, s_k) stage k, then l, then r; columns
// [0, s_k). Right-looking Cholesky, one barrier per column: the owners of
// column j publish it (unscaled) to LDS, every thread reads the pivot and
// updates its entries right of j, the owners scale their part of column j.
// Then the update block Q = P P^T of the rows below (P = [L(l,k); L(r,k)])
// from LDS, register-tiled the same way (lower half only).
template <int NB>
__global__ __launch_bounds__(256) void k_cr_factor(const InstDev* __restrict__ insts, CrArrays AR, int task0) {
    constexpr int RA = 3 * NB;  // row slots of the front (<= 48 NB rows)
    constexpr int QA = 2 * NB;  // row / column slots of the update block (<= 32 NB)
    constexpr int CB = 48 * NB;
    extern __shared__ __align__(16) double sh[];
    const CrTask T = AR.tasks[task0 + blockIdx.x];
    const int tid = threadIdx.x, ti = tid & 15, tc = tid >> 4;
    const int sk = T.sk;
    const int64_t u0 = T.npull > 0 ? AR.pulls[T.pull0].u : -1;
    const int64_t u1 = T.npull > 1 ? AR.pulls[T.pull0 + 1].u : -1;
    const double* Dk = (T.from_work ? AR.L : AR.D) + T.d;
    double* Lk = AR.L + T.d;
    if (!T.elim) {
        // a stage that stays: D_k -= the previous level's updates (lower part)
        double v[NB][NB], w0[NB][NB], w1[NB][NB];
#pragma unroll
        for (int a = 0; a < NB; a++)
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const int i = ti + 16 * a, c = tc + 16 * b;
                const bool ok = i < sk && c < sk && i >= c;
                const int64_t idx = (int64_t)c * sk + i;
                v[a][b] = ok ? Dk[idx] : 0.0;
                w0[a][b] = ok && u0 >= 0 ? AR.U[u0 + idx] : 0.0;
                w1[a][b] = ok && u1 >= 0 ? AR.U[u1 + idx] : 0.0;
            }
#pragma unroll
        for (int a = 0; a < NB; a++)
#pragma unroll
            for (int b = 0; b < NB; b++) {
                const int i = ti + 16 * a, c = tc + 16 * b;
                if (i < sk && c < sk && i >= c) Lk[(int64_t)c * sk + i] = (v[a][b] - w0[a][b]) - w1[a][b];
            }
        return;
    }
    const InstDev& I = insts[T.inst];
    const int sl = T.sl, sr = T.sr, np = sl + sr, mr = sk + np;
    // all loads issued before any is used: the rows below the stage (one load
    // each, K(l,k) = K(k,l)^T and K(r,k)), then D_k and its updates
    double m[RA][NB];
#pragma unroll
    for (int a = 0; a < RA; a++)
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const int i = ti + 16 * a, c = tc + 16 * b;
            const bool below = c < sk && i >= sk && i < mr;
            const int64_t at = i < sk + sl ? T.kl + (int64_t)(i - sk) * sk + c : T.kr + (int64_t)c * sr + (i - sk - sl);
            m[a][b] = below ? AR.C[at] : 0.0;
        }
    double dv[NB][NB], w0[NB][NB], w1[NB][NB];
#pragma unroll
    for (int a = 0; a < NB; a++)
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const int i = ti + 16 * a, c = tc + 16 * b;
            const bool ok = i < sk && c < sk && i >= c;
            const int64_t idx = (int64_t)c * sk + i;
            dv[a][b] = ok ? Dk[idx] : 0.0;
            w0[a][b] = ok && u0 >= 0 ? AR.U[u0 + idx] : 0.0;
            w1[a][b] = ok && u1 >= 0 ? AR.U[u1 + idx] : 0.0;
        }
#pragma unroll
    for (int a = 0; a < NB; a++)
#pragma unroll
        for (int b = 0; b < NB; b++)
            if (ti + 16 * a < sk) m[a][b] = (dv[a][b] - w0[a][b]) - w1[a][b];
    // Right-looking Cholesky in unscaled form: step j subtracts M(i,j)
    // M(c,j) / M(j,j) from M(i,c), and the columns are scaled by the square
    // roots of their pivots (kept in LDS) in one pass at the end, which keeps
    // the square roots off the per-column chain. The update of step j
    // touches entry (i, c) with i >= c > j. With i = ti + 16 a and c = tc +
    // 16 b that is: slot pairs a > b always (given c > j), a == b when ti >=
    // tc, a < b never; so the pairs are fixed at compile time and the rest is
    // masked by selects (no branches in the loop).
    double* colbuf = sh;            // two column buffers of CB rows
    double* piv = sh + 2 * CB;      // the pivots (after substitution of failed ones)
    bool rowok[RA];
#pragma unroll
    for (int a = 0; a < RA; a++) rowok[a] = ti + 16 * a < mr;
    const bool diag_ok = ti >= tc;
    int par = 0;
#pragma unroll
    for (int jb = 0; jb < NB; jb++) {
        for (int jj = 0; jj < 16; jj++) {
            const int j = 16 * jb + jj;
            if (j >= sk) break;
            double* cb = colbuf + par * CB;
            if (tc == jj) {
#pragma unroll
                for (int a = jb; a < RA; a++) cb[ti + 16 * a] = m[a][jb];
            }
            __syncthreads();
            // every read of the column first, then the pivot
            double d = cb[j];
            double cv[RA], cc[NB];
#pragma unroll
            for (int a = jb; a < RA; a++) cv[a] = cb[ti + 16 * a];
#pragma unroll
            for (int b = jb; b < NB; b++) cc[b] = cb[tc + 16 * b];
            if (!(d > 0.0) || !isfinite(d)) {
                if (tid == 0) {
                    atomicMin(&I.status[1], T.var0 + j);
                    atomicMax(&I.status[0], KKT_ST_NOT_SPD);
                }
                d = 1.0;
            }
            if (tid == 0) piv[j] = d;
            const double inv_d = recip_f64(d);
#pragma unroll
            for (int a = jb; a < RA; a++) cv[a] = rowok[a] ? cv[a] : 0.0;
#pragma unroll
            for (int b = jb; b < NB; b++) {
                const int c = tc + 16 * b;
                const double lc = (c > j && c < sk) ? cc[b] * inv_d : 0.0;
                m[b][b] = fma(-(diag_ok ? cv[b] : 0.0), lc, m[b][b]);
#pragma unroll
                for (int a = b + 1; a < RA; a++) m[a][b] = fma(-cv[a], lc, m[a][b]);
            }
            par ^= 1;
        }
    }
    __syncthreads();
    // scale: L(i,c) = M(i,c) / sqrt(d_c) below the diagonal, sqrt(d_c) on it
#pragma unroll
    for (int b = 0; b < NB; b++) {
        const int c = tc + 16 * b;
        const double dc = c < sk ? piv[c] : 1.0;
        const double ls = sqrt(dc), inv_ls = recip_f64(ls);
#pragma unroll
        for (int a = 0; a < RA; a++) {
            const int i = ti + 16 * a;
            m[a][b] = i == c ? ls : m[a][b] * inv_ls;
        }
    }
    // L_k to L (lower), L(l,k) and L(r,k) to P, and P = the rows below into LDS
    double* Pb = sh + 2 * CB + 16 * NB;  // s_k columns of np rows
#pragma unroll
    for (int a = 0; a < RA; a++)
#pragma unroll
        for (int b = 0; b < NB; b++) {
            const int i = ti + 16 * a, c = tc + 16 * b;
            if (c >= sk || i >= mr) continue;
            if (i < sk) {
                if (i >= c) Lk[(int64_t)c * sk + i] = m[a][b];
            } else {
                Pb[c * np + (i - sk)] = m[a][b];
                if (i < sk + sl) AR.P[T.pl + (int64_t)c * sl + (i - sk)] = m[a][b];
                else AR.P[T.pr + (int64_t)c * sr + (i - sk - sl)] = m[a][b];
            }
        }
    if (np == 0) return;  // uniform: the last stage of its instance
    __syncthreads();
    // Q = P P^T, lower half: UL = Q(l, l), UR = Q(r, r), fill F = -Q(r, l)
    double q[QA][QA];
#pragma unroll
    for (int a = 0; a < QA; a++)
#pragma unroll
        for (int b = 0; b <= a; b++) q[a][b] = 0.0;
    // Pb holds s_k np entries plus 32 NB of padding, so these reads stay in
    // bounds for every slot; slots past np are masked to zero. The reads of
    // column c + 1 are issued before the products of column c.
    bool pok[QA], qok[QA];
#pragma unroll
    for (int a = 0; a < QA; a++) {
        pok[a] = ti + 16 * a < np;
        qok[a] = tc + 16 * a < np;
    }
    double pr[QA], pc[QA];
#pragma unroll
    for (int a = 0; a < QA; a++) {
        pr[a] = Pb[ti + 16 * a];
        pc[a] = Pb[tc + 16 * a];
    }
    for (int c = 0; c < sk; c++) {
        const int cn = c + 1 < sk ? c + 1 : c;
        double prn[QA], pcn[QA];
#pragma unroll
        for (int a = 0; a < QA; a++) {
            prn[a] = Pb[cn * np + ti + 16 * a];
            pcn[a] = Pb[cn * np + tc + 16 * a];
        }
#pragma unroll
        for (int a = 0; a < QA; a++) {
            pr[a] = pok[a] ? pr[a] : 0.0;
            pc[a] = qok[a] ? pc[a] : 0.0;
        }
#pragma unroll
        for (int a = 0; a < QA; a++)
#pragma unroll
            for (int b = 0; b <= a; b++) q[a][b] = fma(pr[a], pc[b], q[a][b]);
#pragma unroll
        for (int a = 0; a < QA; a++) {
            pr[a] = prn[a];
            pc[a] = pcn[a];
        }
    }
#pragma unroll
    for (int a = 0; a < QA; a++)
#pragma unroll
        for (int b = 0; b <= a; b++) {
            const int p = ti + 16 * a, p2 = tc + 16 * b;
            if (p >= np || p2 >= np || p < p2) continue;
            if (p < sl) AR.U[T.ul + (int64_t)p2 * sl + p] = q[a][b];
            else if (p2 >= sl) AR.U[T.ur + (int64_t)(p2 - sl) * sr + (p - sl)] = q[a][b];
            else AR.C[T.f + (int64_t)p2 * sr + (p - sl)] = -q[a][b];
        }
}

// L y = t by one wave (s columns, column-major with s rows in LDS): lane l
// carries rows l and l + 64 in t0 and t1 and their pivot reciprocals in d0
// and d1; steps as in fwd_steps, a block's coefficients read while the block
// before it is solved
template <int K0, bool TAIL, bool HI>
__device__ __forceinline__ void cr_steps(double& t, double& th, double& y, const double (&a)[16],
                                         const double (&ah)[16], const double d, const int l0, const int nb) {
    static_for<4>([&](auto K) {
        constexpr int k = K0 + K;
        double v = readlane_d(t * d, l0 + k);
        if (TAIL) v = k < nb ? v : 0.0;
        y = writelane_d(v, l0 + k, y);
        t = fma(-a[k], v, t);
        if constexpr (HI) th = fma(-ah[k], v, th);
    });
}
__device__ __forceinline__ void tri_fwd_wave(const double* __restrict__ L, const int s, const double d0,
                                             const double d1, double& t0, double& t1, const int lane) {
    static_assert(kCrMaxStage <= 128, "two rows per lane");
    double y0 = 0.0, y1 = 0.0;
    const double *const p0 = L + min(lane, s - 1), *const p1 = L + min(lane + 64, s - 1);
    double a[2][16], b[2][16];
    auto load = [&](auto Q, const int j) {
#pragma unroll
        for (int k = 0; k < 16; k++) {
            a[Q][k] = p0[min(j + k, s - 1) * s];
            b[Q][k] = p1[min(j + k, s - 1) * s];
        }
    };
    load(std::integral_constant<int, 0>{}, 0);
    static_for<4>([&](auto B) {
        const int nb = s - 16 * B;
        if (nb > 0) {
            load(std::integral_constant<int, (B + 1) & 1>{}, 16 * B + 16);
            static_for<4>([&](auto R) {
                if (nb >= 4 * R + 4) cr_steps<4 * R, false, true>(t0, t1, y0, a[B & 1], b[B & 1], d0, 16 * B, nb);
                else if (nb > 4 * R) cr_steps<4 * R, true, true>(t0, t1, y0, a[B & 1], b[B & 1], d0, 16 * B, nb);
            });
        }
    });
    for (int j = 64; j < s; j += 16) {
        const int nb = s - j;
        if (j > 64) load(std::integral_constant<int, 0>{}, j);
        static_for<4>([&](auto R) {
            if (nb >= 4 * R + 4) cr_steps<4 * R, false, false>(t1, t1, y1, b[0], b[0], d1, j - 64, nb);
            else if (nb > 4 * R) cr_steps<4 * R, true, false>(t1, t1, y1, b[0], b[0], d1, j - 64, nb);
        });
    }
    t0 = y0;
    t1 = y1;
}

// Stages L_k (s_k x s_k, column-major) into LDS: every thread issues its
// loads before the first store.
__device__ inline void cr_stage_block(double* __restrict__ dst, const double* __restrict__ src, int n) {
    constexpr int PER = (kCrMaxStage * kCrMaxStage + 255) / 256;
    double v[PER];
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int q = threadIdx.x + 256 * u;
        v[u] = q < n ? src[q] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int q = threadIdx.x + 256 * u;
        if (q < n) dst[q] = v[u];
    }
}

// y (s_k rows) -= sum over columns c = g, g + 4, ... of P(:, c) x_c, P
// column-major with s_k rows: this thread's part for rows r and r + 64
__device__ inline void cr_matvec_part(const double* __restrict__ P, int rows, int cols,
                                      const double* __restrict__ x, int r, int g, double& s0, double& s1) {
    constexpr int U = kCrMaxStage / 4;
    double xv[U], p0[U], p1[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int c = g + 4 * u;
        xv[u] = c < cols ? x[c] : 0.0;
        p0[u] = c < cols && r < rows ? P[(int64_t)c * rows + r] : 0.0;
        p1[u] = c < cols && r + 64 < rows ? P[(int64_t)c * rows + r + 64] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
        s0 = fma(p0[u], xv[u], s0);
        s1 = fma(p1[u], xv[u], s1);
    }
}

// this thread's part of (P^T x)(r), (P^T x)(r + 64) over rows a = g, g + 4,
// ... of P (column-major, prow rows)
__device__ inline void cr_matvec_t_part(const double* __restrict__ P, int prow, int cols,
                                        const double* __restrict__ x, int r, int g, double& s0, double& s1) {
    constexpr int U = kCrMaxStage / 4;
    double xv[U], p0[U], p1[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const int a = g + 4 * u;
        xv[u] = a < prow ? x[a] : 0.0;
        p0[u] = a < prow && r < cols ? P[(int64_t)r * prow + a] : 0.0;
        p1[u] = a < prow && r + 64 < cols ? P[(int64_t)(r + 64) * prow + a] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
        s0 = fma(p0[u], xv[u], s0);
        s1 = fma(p1[u], xv[u], s1);
    }
}

// Forward solve L y = b, per level: a task eliminating its stage takes t_k -
// the previous level's contributions, then y_k = L_k^{-1} t_k by
// substitution in wave 0 (tri_fwd_wave: 12.9 us a launch of few stages of 66,
// 18.5 with one LDS column read ahead per step); a
// task of a stage that stays only subtracts the contributions. On
// level 0 t_k starts from b (mode 0) or the refinement residual (mode 1,
// stopped instances skipped); later levels from t.
__global__ __launch_bounds__(256) void k_cr_fwd(const InstDev* __restrict__ insts, CrArrays AR, int task0,
                                                Calls C, int mode, int level0) {
    __shared__ double Ls[kCrMaxStage * kCrMaxStage];
    __shared__ double red[4][128];
    __shared__ double inv[kCrMaxStage];
    const CrTask T = AR.tasks[task0 + blockIdx.x];
    const InstDev& I = insts[T.inst];
    if (mode == 1 && I.rs->done) return;  // uniform per block
    const bool elim = T.elim != 0;
    const int tid = threadIdx.x, r = tid & 63, g = tid >> 6, sk = T.sk;
    double s0 = 0.0, s1 = 0.0;
    for (int u = 0; u < T.npull; u++) {
        const CrPull Pu = AR.pulls[T.pull0 + u];
        cr_matvec_part(AR.P + Pu.p, sk, Pu.si, AR.t + Pu.vi, r, g, s0, s1);
    }
    red[g][r] = s0;
    red[g][r + 64] = s1;
    if (elim) {
        cr_stage_block(Ls, AR.L + T.d, sk * sk);
        if (tid < sk) inv[tid] = 1.0 / AR.L[T.d + (int64_t)tid * sk + tid];
    }
    __syncthreads();
    if (tid >= 64) return;
    const double* src = level0 ? (mode == 0 ? C.b + T.v0 : I.r + T.var0) : AR.t + T.v0;
    const int i0 = r, i1 = r + 64;
    double t0 = i0 < sk ? src[i0] - ((red[0][i0] + red[1][i0]) + (red[2][i0] + red[3][i0])) : 0.0;
    double t1 = i1 < sk ? src[i1] - ((red[0][i1] + red[1][i1]) + (red[2][i1] + red[3][i1])) : 0.0;
    if (elim) {
        tri_fwd_wave(Ls, sk, inv[min(i0, sk - 1)], inv[min(i1, sk - 1)], t0, t1, r);
    }
    if (i0 < sk) AR.t[T.v0 + i0] = t0;
    if (i1 < sk) AR.t[T.v0 + i1] = t1;
}

// Backward solve L^T x = y, levels in reverse, eliminated stages only: x_k =
// L_k^{-T} (y_k - L(l,k)^T x_l - L(r,k)^T x_r), the neighbours being
// eliminated later (their x already in t), the triangle as in the supernodal
// sweep (10.3 us a launch of few stages of 66, 16.7 step by step from LDS).
// x_k goes to t and to the output:
// mode 0 x = x_k; mode 1 xprev = x, x += x_k.
__global__ __launch_bounds__(256) void k_cr_bwd(const InstDev* __restrict__ insts, CrArrays AR, int task0, Calls C,
                                                int mode) {
    __shared__ double Ls[kCrMaxStage * kCrMaxStage];
    __shared__ double red[4][128];
    __shared__ double inv[kCrMaxStage];
    const CrTask T = AR.tasks[task0 + blockIdx.x];
    const InstDev& I = insts[T.inst];
    if (!T.elim || (mode == 1 && I.rs->done)) return;  // uniform per block
    const int tid = threadIdx.x, r = tid & 63, g = tid >> 6, sk = T.sk;
    double s0 = 0.0, s1 = 0.0;
    if (T.sl > 0) cr_matvec_t_part(AR.P + T.pl, T.sl, sk, AR.t + T.vl, r, g, s0, s1);
    if (T.sr > 0) cr_matvec_t_part(AR.P + T.pr, T.sr, sk, AR.t + T.vr, r, g, s0, s1);
    red[g][r] = s0;
    red[g][r + 64] = s1;
    cr_stage_block(Ls, AR.L + T.d, sk * sk);
    if (tid < sk) inv[tid] = 1.0 / AR.L[T.d + (int64_t)tid * sk + tid];
    __syncthreads();
    if (tid >= 64) return;
    const int i0 = r, i1 = r + 64;
    double t0 = i0 < sk ? AR.t[T.v0 + i0] - ((red[0][i0] + red[1][i0]) + (red[2][i0] + red[3][i0])) : 0.0;
    double t1 = i1 < sk ? AR.t[T.v0 + i1] - ((red[0][i1] + red[1][i1]) + (red[2][i1] + red[3][i1])) : 0.0;
    double a[4][16];
    tri_bwd_load(a, Ls, sk, sk, r);
    tri_bwd_wave(a, Ls, sk, sk, inv[min(i0, sk - 1)], inv[min(i1, sk - 1)], t0, t1, r);
    double* x = C.x + T.v0;
    if (i0 < sk) {
        AR.t[T.v0 + i0] = t0;
        if (mode == 0) {
            x[i0] = t0;
        } else {
            const double xo = x[i0];
            I.xprev[T.var0 + i0] = xo;
            x[i0] = xo + t0;
        }
    }
    if (i1 < sk) {
        AR.t[T.v0 + i1] = t1;
        if (mode == 0) {
            x[i1] = t1;
        } else {
            const double xo = x[i1];
            I.xprev[T.var0 + i1] = xo;
            x[i1] = xo + t1;
        }
    }
}

// ---------------------------------------------------------------------------
// workspace redirection (allocation-free solve): copies of a factor's instance
// descriptor and front descriptors whose per-solve vectors point into a
// caller-provided workspace
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_ws_redirect(const InstDev* __restrict__ src_inst,
                                                     const FrontDesc* __restrict__ src_fd, int nf, SolveWs w) {
    const InstDev& S = src_inst[0];
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t == 0) {
        InstDev D = S;
        D.y = w.y;
        D.V = w.V;
        D.r = w.r;
        D.xprev = w.xprev;
        D.rpart = w.rpart;
        D.rs = w.rs;
        w.inst[0] = D;
    }
    if (t >= nf) return;
    FrontDesc F = src_fd[t];
    F.y = w.y + F.col0;
    F.V = w.V + (F.V - S.V);
    for (int j = 0; j < 2; j++)
        if (j < F.nch) F.cV[j] = w.V + (F.cV[j] - S.V);
    F.done = &w.rs->done;
    w.fd[t] = F;
}

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------
hipError_t set_kernel_attributes() {
    const int lds = kMaxDynLds;
    hipError_t e = hipFuncSetAttribute((const void*)k_factor, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)k_factor_small, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)k_factor_queue, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)k_cr_factor<1>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)k_cr_factor<2>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)k_cr_factor<3>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)k_cr_factor<4>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    e = hipFuncSetAttribute((const void*)k_cr_factor<5>, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    if (e != hipSuccess) return e;
    for (const void* k : {(const void*)k_fwd<64>, (const void*)k_fwd<128>, (const void*)k_fwd<256>, (const void*)k_sweeps_queue, (const void*)k_bwd<16, 256>, (const void*)k_bwd<16, 512>, (const void*)k_bwd_wide})
        if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxSweepLds);
    return e;
}

static inline unsigned blocks_for(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

void launch_aug_rhs(const InstDev* insts, const AugCall& A, const WorkItem* ncols, int nitems, int nlong, int mode,
                    hipStream_t st) {
    if (nitems > 0) k_aug_rhs<<<nitems + (nlong + 15) / 16, kBlock, 0, st>>>(insts, A, ncols, nitems, mode);
}
void launch_aug_recover(const InstDev* insts, const AugCall& A, const WorkItem* ncols, int nn, const WorkItem* mrows,
                        int nm, int mode, hipStream_t st) {
    if (mode == 1 && nn > 0) k_aug_update_x<<<nn, kBlock, 0, st>>>(insts, A, ncols);
    if (nm > 0) k_aug_recover_m<<<nm, kBlock, 0, st>>>(insts, A, mrows, mode);
}
void launch_aug_reset(const InstDev* insts, int ninst, double tol, int maxit, hipStream_t st) {
    if (ninst > 0) k_aug_reset<<<blocks_for(ninst, 64), 64, 0, st>>>(insts, ninst, tol, maxit);
}
void launch_aug_check(const InstDev* insts, const AugCall& A, const WorkItem* ncols, int nn, const WorkItem* mrows,
                      int nm, int ninst, hipStream_t st) {
    if (nn > 0) k_aug_res_n<<<nn * kRowSplit, kBlock, 0, st>>>(insts, A, ncols);
    if (nm > 0) k_aug_res_m<<<nm, kBlock, 0, st>>>(insts, A, mrows);
    if (ninst > 0) k_aug_decide<<<ninst, kBlock, 0, st>>>(insts);
}
void launch_aug_revert(const InstDev* insts, const AugCall& A, const WorkItem* ncols, int nn, const WorkItem* mrows,
                       int nm, hipStream_t st) {
    if (nn > 0) k_aug_revert_n<<<nn, kBlock, 0, st>>>(insts, A, ncols);
    if (nm > 0) k_aug_revert_m<<<nm, kBlock, 0, st>>>(insts, A, mrows);
}
void launch_ipm_start(const InstDev* insts, const IpmCall& P, const WorkItem* ncols, int nn, const WorkItem* mrows,
                      int nm, double tol, int maxit, double sigma, double tau_min, hipStream_t st) {
    if (nn > 0) k_ipm_norm_n<<<nn, kBlock, 0, st>>>(insts, P, ncols);
    if (nm > 0) k_ipm_norm_m<<<nm, kBlock, 0, st>>>(insts, P, mrows);
    k_ipm_init<<<1, kBlock, 0, st>>>(insts, P, tol, maxit, sigma, tau_min);
}
void launch_ipm_dsw(const InstDev* insts, const IpmCall& P, const WorkItem* mrows, int nm, hipStream_t st) {
    if (nm > 0) k_ipm_dsw<<<nm, kBlock, 0, st>>>(insts, P, mrows);
}
void launch_ipm_residuals(const InstDev* insts, const IpmCall& P, const WorkItem* ncols, int nn, const WorkItem* mrows,
                          int nm, double delta, hipStream_t st) {
    if (nn > 0) k_ipm_res_n<<<nn * kRowSplit, kBlock, 0, st>>>(insts, P, ncols, delta);
    if (nm > 0) k_ipm_res_m<<<nm, kBlock, 0, st>>>(insts, P, mrows);
    k_ipm_decide<<<1, kBlock, 0, st>>>(insts, P, delta);
}
void launch_ipm_r2(const InstDev* insts, const IpmCall& P, const WorkItem* mrows, int nm, hipStream_t st) {
    if (nm > 0) k_ipm_r2<<<nm, kBlock, 0, st>>>(insts, P, mrows);
}
void launch_ipm_step(const InstDev* insts, const IpmCall& P, const WorkItem* ncols, int nn, const WorkItem* mrows,
                     int nm, hipStream_t st) {
    if (nm > 0) k_ipm_alpha<<<nm, kBlock, 0, st>>>(insts, P, mrows);
    k_ipm_alpha_fin<<<1, kBlock, 0, st>>>(insts, P);
    if (nn > 0) k_ipm_update_n<<<nn, kBlock, 0, st>>>(insts, P, ncols);
    if (nm > 0) k_ipm_update_m<<<nm, kBlock, 0, st>>>(insts, P, mrows);
}
void launch_fill_f64(double* p, double v, int64_t n, hipStream_t st) {
    if (n > 0) k_fill_f64<<<blocks_for(n, kBlock), kBlock, 0, st>>>(p, v, n);
}
void launch_cr_scatter(const InstDev* insts, const CrArrays& A, const CrScatter* items, int64_t nitems,
                       hipStream_t st) {
    if (nitems > 0) k_cr_scatter<<<blocks_for(nitems, kBlock), kBlock, 0, st>>>(insts, A, items, nitems);
}
void launch_cr_factor(const InstDev* insts, const CrArrays& A, int task0, int ntask, int nb, size_t lds,
                      hipStream_t st) {
    if (ntask <= 0) return;
    switch (nb) {
        case 1: k_cr_factor<1><<<ntask, kBlock, lds, st>>>(insts, A, task0); break;
        case 2: k_cr_factor<2><<<ntask, kBlock, lds, st>>>(insts, A, task0); break;
        case 3: k_cr_factor<3><<<ntask, kBlock, lds, st>>>(insts, A, task0); break;
        case 4: k_cr_factor<4><<<ntask, kBlock, lds, st>>>(insts, A, task0); break;
        default: k_cr_factor<5><<<ntask, kBlock, lds, st>>>(insts, A, task0); break;
    }
}
void launch_cr_fwd(const InstDev* insts, const CrArrays& A, int task0, int ntask, const Calls& C, int mode,
                   int level0, hipStream_t st) {
    if (ntask > 0) k_cr_fwd<<<ntask, 256, 0, st>>>(insts, A, task0, C, mode, level0);
}
void launch_cr_bwd(const InstDev* insts, const CrArrays& A, int task0, int ntask, const Calls& C, int mode,
                   hipStream_t st) {
    if (ntask > 0) k_cr_bwd<<<ntask, 256, 0, st>>>(insts, A, task0, C, mode);
}
void launch_ws_redirect(const InstDev* src_inst, const FrontDesc* src_fd, int nf, const SolveWs& w, hipStream_t st) {
    k_ws_redirect<<<blocks_for(nf > 0 ? nf : 1, 256), 256, 0, st>>>(src_inst, src_fd, nf, w);
}
void launch_copy_segments(const CopySeg* segs, int nseg, hipStream_t st) {
    if (nseg > 0) k_copy_segments<<<nseg * kCopyParts, 256, 0, st>>>(segs);
}
void launch_fill_i32(int* p, int v, int64_t n, hipStream_t st) {
    if (n > 0) k_fill_i32<<<blocks_for(n, kBlock), kBlock, 0, st>>>(p, v, n);
}
void launch_status_init(int* status, int ninst, hipStream_t st) {
    if (ninst > 0) k_status_init<<<blocks_for(ninst, kBlock), kBlock, 0, st>>>(status, ninst);
}
void launch_jscale(const InstDev* insts, const Calls& C, const WorkItem* items, int nitems, hipStream_t st) {
    if (nitems > 0) k_jscale<<<nitems, kBlock, 0, st>>>(insts, C, items);
}
void launch_keep_lifted(const InstDev* insts, const Calls& C, const WorkItem* jentries, int nj, const WorkItem* mrows,
                        int nm, hipStream_t st) {
    if (nj > 0) k_keep_lifted<<<nj, kBlock, 0, st>>>(insts, C, jentries, 0);
    if (nm > 0) k_keep_lifted<<<nm, kBlock, 0, st>>>(insts, C, mrows, 1);
}
void launch_jcopy(const InstDev* insts, const Calls& C, const WorkItem* items, int nitems, hipStream_t st) {
    if (nitems > 0) k_jcopy<<<nitems, kBlock, 0, st>>>(insts, C, items);
}
void launch_assemble_heavy(const InstDev* insts, const Calls& C, const WorkItem* items, int nitems, hipStream_t st) {
    if (nitems > 0) k_assemble_heavy<<<(nitems + 15) / 16, kBlock, 0, st>>>(insts, C, items, nitems);
}
void launch_assemble(const InstDev* insts, const Calls& C, const WorkItem* items, int nitems, hipStream_t st) {
    if (nitems > 0) k_assemble<<<nitems, kBlock, 0, st>>>(insts, C, items);
}
void launch_factor(const InstDev* insts, const FrontDesc* fds, int nitems, size_t lds, int fused_update,
                   hipStream_t st) {
    if (nitems > 0) k_factor<<<nitems, kFactorThreads, lds, st>>>(insts, fds, fused_update);
}
void launch_factor_small(const InstDev* insts, const FrontDesc* fds, int nitems, size_t lds, int fused_update,
                         hipStream_t st) {
    if (nitems > 0) k_factor_small<<<nitems, kFactorThreadsSmall, lds, st>>>(insts, fds, fused_update);
}
void launch_big_factor(const InstDev* insts, const FrontDesc* fds, int nitems, int max_cols, int max_rows,
                       hipStream_t st) {
    if (nitems <= 0) return;
    const int nbc = (max_cols + 15) / 16, nbr = (max_rows + 15) / 16;
    k_big_init<<<dim3(nitems, nbc, (max_rows + kBigInitRows - 1) / kBigInitRows), kBigThreads, 0, st>>>(insts, fds);
    for (int kb = 0; kb < nbc; kb++) {
        const int below = max_rows - 16 * kb - 16;
        if (below > 0) k_big_trsm<<<dim3(nitems, (below + kBigThreads - 1) / kBigThreads), kBigThreads, 0, st>>>(fds, kb);
        int ntile = 0;
        for (int jt = kb + 1; jt < nbc; jt++) ntile += nbr - jt;
        const int wpg = kBigThreads / 64;
        k_big_tiles<<<dim3(nitems, std::max(1, (ntile + wpg - 1) / wpg)), kBigThreads, 0, st>>>(insts, fds, kb);
    }
}
void launch_big_fwd(const InstDev* insts, const FrontDesc* fds, int nitems, int max_rows, int skip_done, hipStream_t st) {
    if (nitems <= 0) return;
    k_big_fwd<<<nitems, kBigThreads, 0, st>>>(insts, fds, skip_done);
    const int nb = (max_rows + kBigThreads - 1) / kBigThreads;
    k_big_fwd_rows<<<dim3(nitems, nb), kBigThreads, 0, st>>>(fds, skip_done);
}
void launch_big_bwd(const FrontDesc* fds, int nitems, int max_cols, int skip_done, hipStream_t st) {
    if (nitems <= 0) return;
    const int wpg = kBigThreads / 64;
    k_big_bwd_dot<<<dim3(nitems, (max_cols + wpg - 1) / wpg), kBigThreads, 0, st>>>(fds, skip_done);
    k_big_bwd<<<nitems, kBigThreads, 0, st>>>(fds, skip_done);
}
void launch_update(const InstDev* insts, const FrontDesc* fds, const StripItem* items, int nitems, hipStream_t st) {
    if (nitems > 0) k_update<<<nitems, kUpdThreads, 0, st>>>(insts, fds, items);
}
void launch_factor_queue(const InstDev* insts, const FrontDesc* fds, const DepLists& D, int grid, size_t lds,
                         hipStream_t st) {
    if (D.nitems > 0) k_factor_queue<<<grid, kFactorQueueThreads, lds, st>>>(insts, fds, D);
}
void launch_sweeps_queue(const InstDev* insts, const FrontDesc* fds, const DepLists& D, int grid, size_t lds,
                         int skip_done, hipStream_t st) {
    if (D.nitems > 0) k_sweeps_queue<<<grid, kSolveThreads, lds, st>>>(insts, fds, D, skip_done);
}
void launch_fwd(const InstDev* insts, const FrontDesc* fds, int nitems, int maxr, bool narrow, size_t lds, int skip_done, hipStream_t st) {
    if (nitems <= 0) return;
    // a wave holds 128 rows
    if (narrow) k_fwd<64><<<nitems, 64, lds, st>>>(insts, fds, skip_done);
    else if (maxr <= 256) k_fwd<128><<<nitems, 128, lds, st>>>(insts, fds, skip_done);
    else k_fwd<256><<<nitems, 256, lds, st>>>(insts, fds, skip_done);
}
void launch_bwd(const FrontDesc* fds, int nitems, int form, size_t lds, int skip_done, hipStream_t st) {
    if (nitems <= 0) return;
    if (form == BWD_WIDE) k_bwd_wide<<<nitems, kSolveThreads, lds, st>>>(fds, skip_done);
    else if (form == BWD_LIGHT) k_bwd<16, 256><<<nitems, 256, lds, st>>>(fds, skip_done);
    else k_bwd<16, 512><<<nitems, 512, lds, st>>>(fds, skip_done);
}
void launch_perm_in(const InstDev* insts, const Calls& C, const WorkItem* rows, int nitems, int mode, hipStream_t st) {
    if (nitems > 0) k_perm_in<<<nitems, kBlock, 0, st>>>(insts, C, rows, mode);
}
void launch_perm_out(const InstDev* insts, const Calls& C, const WorkItem* rows, int nitems, int mode, hipStream_t st) {
    if (nitems > 0) k_perm_out<<<nitems, kBlock, 0, st>>>(insts, C, rows, mode);
}
void launch_refine_reset(const InstDev* insts, int ninst, double tol, int maxit, int* ndone, hipStream_t st) {
    k_refine_reset<<<blocks_for(ninst, 64), 64, 0, st>>>(insts, ninst, tol, maxit, ndone);
}
void launch_residual(const InstDev* insts, const Calls& C, const WorkItem* rows, int nitems, hipStream_t st) {
    if (nitems > 0) k_residual<<<nitems * kResidualSplit, kBlock, 0, st>>>(insts, C, rows);
}
void launch_refine_decide(const InstDev* insts, int ninst, int* ndone, RefineReport* rep, const int* err,
                          hipStream_t st) {
    if (ninst > 0) k_refine_decide<<<ninst, 256, 0, st>>>(insts, ndone, rep, err);
}
void launch_refine_revert(const InstDev* insts, const Calls& C, const WorkItem* rows, int nitems, hipStream_t st) {
    if (nitems > 0) k_refine_revert<<<nitems, kBlock, 0, st>>>(insts, C, rows);
}
void launch_matvec(const InstDev* insts, const double* x, double* y, const WorkItem* rows, int nitems, hipStream_t st) {
    if (nitems > 0) k_matvec<<<nitems, kBlock, 0, st>>>(insts, x, y, rows);
}
void launch_cg_fg(const InstDev* insts, const Calls& C, const WorkItem* ncols, int nitems, int nlong, double tol,
                  int maxit, double eta_tol, hipStream_t st) {
    if (nitems > 0) k_cg_fg<<<nitems + (nlong + 15) / 16, kBlock, 0, st>>>(insts, C, ncols, nitems, tol, maxit, eta_tol);
    if (nitems > 0) k_cg_rows<<<nitems * kRowSplit, kBlock, 0, st>>>(insts, C, ncols);
}
void launch_cg_c(const InstDev* insts, const Calls& C, const WorkItem* mrows, int nitems, int ninst, hipStream_t st) {
    if (nitems > 0) k_cg_c<<<nitems, kBlock, 0, st>>>(insts, C, mrows);
    if (ninst > 0) k_cg_norms<<<ninst, kBlock, 0, st>>>(insts);
}
void launch_cg_dir(const InstDev* insts, const WorkItem* ncols, int nitems, int nlong, int k, int* ndone,
                   hipStream_t st) {
    if (nitems > 0) k_cg_dir<<<nitems + (nlong + 15) / 16, kBlock, 0, st>>>(insts, ncols, nitems, k, ndone);
}
void launch_cg_eta_test(const InstDev* insts, const Calls& C, int ninst, int k, int* ndone, hipStream_t st) {
    if (ninst > 0) k_cg_eta_test<<<ninst, kBlock, 0, st>>>(insts, C, k, ndone);
}
void launch_cg_q(const InstDev* insts, const Calls& C, const WorkItem* mrows, int nitems, int k, hipStream_t st) {
    if (nitems > 0) k_cg_q<<<nitems, kBlock, 0, st>>>(insts, C, mrows, k);
}
void launch_cg_upd(const InstDev* insts, const Calls& C, const WorkItem* mrows, int nitems, int k, int* ndone,
                   hipStream_t st) {
    if (nitems > 0) k_cg_upd<<<nitems, kBlock, 0, st>>>(insts, C, mrows, k, ndone);
}
void launch_cg_dxrhs(const InstDev* insts, const Calls& C, const WorkItem* ncols, int nitems, int nlong,
                     hipStream_t st) {
    if (nitems > 0) k_cg_dxrhs<<<nitems + (nlong + 15) / 16, kBlock, 0, st>>>(insts, C, ncols, nitems);
}
void launch_cg_residual(const InstDev* insts, const Calls& C, const WorkItem* ncols, int nn, const WorkItem* mrows,
                        int nm, int ninst, hipStream_t st) {
    if (nn > 0) k_cg_res_n<<<nn * kRowSplit, kBlock, 0, st>>>(insts, C, ncols);
    if (nm > 0) k_cg_res_m<<<nm, kBlock, 0, st>>>(insts, C, mrows);
    if (ninst > 0) k_cg_eta<<<ninst, kBlock, 0, st>>>(insts);
}

}  // namespace kkt
