// etpic: envelope-tracking particle-mesh step for gfx950 (MI355X).
//
// Kernels (all launched on the caller's stream):
//   k_tet_coef    per tet: carrier-rotated Whitney coefficients.  With
//                 lam the barycentrics, E(x) = sum_i lam_i A_i and
//                 B(x) = sum_i lam_i C_i inside a tet (both expansions are affine
//                 in lam), where A_i, C_i fold the real parts Re{dof e^{jwt}} + dc
//                 of the 6 edge and 4 face DoFs into the gradients; the envelope
//                 may be interpolated in time between three snapshots.  Per
//                 step, per two steps, or once per multi-step call as the
//                 parts the steps' rows are formed from.
//   k_push_multi  several steps of a multi-step call per launch: per particle,
//                 tet-sorted, gather, Boris push and in-tet path integrals of
//                 each step from the staged row parts, the state in registers
//                 in between; reduction over runs of equal tet and float64
//                 atomics once per launch; reads the particles in their old
//                 order and writes them sorted where the call sorts.
//   k_walk_multi  the particles that left their tet in such a launch:
//                 barycentric walk, reflection, deposit, and their remaining
//                 steps.
//   k_push, k_push_rho, k_push_slices
//                 one step per launch: per particle, tet-sorted: gather from
//                 the coefficient row, Boris push, in-tet path-integral deposit
//                 reduced over runs of equal tet in each wavefront, float64
//                 atomics; particles leaving their tet are queued.  k_push_rho
//                 also scatters the end-point vertex charge; the sliced form
//                 gives each wavefront several consecutive 64-particle slices.
//   k_walk        the queued particles: barycentric walk, reflection, deposit.
//   k_walk_coef   the same and the next step's coefficients in one launch.
//   k_push_sort, k_push_sort_slices
//                 the one-step particle kernels reading the particles in their
//                 old order and writing them, pushed, at their tet-sorted
//                 places (the periodic re-sort folded into a step).
//   k_hist/k_scan*/k_scatter/k_run_stat   counting sort by tet.
//   k_tet_coef_env, k_push_ds, k_walk_ds
//                 the downshifted steps, several per launch: complex-envelope
//                 rows per tet, the carrier-exact velocity quadrature of
//                 interpolated samples with Adams-Bashforth positions, and the
//                 particles that leave their tet.
//   k_charge      vertex charge of the particles.
//   k_gauss_*     continuity residual D^T dG - (rho_new - rho_old).
//   k_locate, k_positions   Cartesian points <-> (tet, barycentrics).
//   k_adjoint, k_adjoint_leavers
//                 reverse of several float64 steps (gradient w.r.t. the edge
//                 envelope), and of the particles that left their tet in them.
//   k_field_spmv, k_nm_*, k_cocg_*   implicit envelope field step.
//   k_ns_*        Gauss-law (non-solenoidal) field solve: CG on the nodal operator.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <vector>
#include <array>
#include <algorithm>
#include <complex>
#include <memory>
#include <mutex>
#include <type_traits>

#include "etpic.h"
#include "field_host.hpp"
#include "mesh_host.hpp"
#include "solve_host.hpp"
#include "checkpoint_host.hpp"

using etpic::TetTopo;

namespace {

thread_local std::string g_last_error;

int fail(int code, const char *fmt, ...) {
    char buf[1024];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_last_error = buf;
    return code;
}

#define HIP_TRY(expr)                                                                         \
    do {                                                                                      \
        hipError_t e_ = (expr);                                                               \
        if (e_ != hipSuccess) return fail(ETPIC_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

constexpr int kBlock = 256;
constexpr int kTimingSets = 512;             // event sets of the step-timing pool
// Internal step flag (the public flags leave bit 31 free): the particle arrays
// hold fixed-point barycentrics (ETPIC_MIXED_FIXED).
constexpr uint32_t kFlagFixed = 1u << 31;
constexpr unsigned kWalkQueueCap = 1u << 23;  // entries of each walk queue; N_p <= 64 * kWalkQueueCap
constexpr unsigned kQueueSkip = 0xffffffffu;  // particle-queue entry to skip
// grid of the walk kernel: the walk is bound by its dependent loads and
// atomics, not by lanes, and fewer blocks pay fewer end-of-walk fences
constexpr unsigned kWalkBlocks = 64;
// grid of k_walk_multi, whose lanes take their particle through the rest of a
// launch's steps
constexpr unsigned kLeaverBlocks = 512;
constexpr int64_t kFewParticles = 2 * 1024 * 16;   // two 16-particle wavefronts on each of 256 CUs x 4 SIMDs
// walk-counter sets: 0 one step per launch, 1 and 2 alternating several, 3 and
// 4 alternating the reverse sweep
constexpr unsigned kCtrSets = 5, kCtrStride = 2048 + 64;
constexpr int64_t kMinPushWaves = 16384;      // 256 CUs x 64 wavefronts
constexpr int64_t kInfinityCacheBytes = (int64_t)256 << 20;
constexpr int64_t kFloatRowBytes = 48 + 64 + 48;   // float coefficient, push and geometry rows per tet

// Runs of equal key among the 64 lanes of a wavefront (particles are kept
// sorted by tet, so neighbouring lanes mostly share a key).  head: first lane
// of a run; head_lane / run_end: first and last lane of this lane's run.
struct WaveRuns {
    int lane, head_lane, run_end;
    bool head;
};

__device__ __forceinline__ WaveRuns wave_runs(int key, int lane = threadIdx.x & 63) {
    WaveRuns r;
    r.lane = lane;
    const int prev = __shfl_up(key, 1);
    r.head = r.lane == 0 || key != prev;
    const unsigned long long hm = __ballot(r.head);
    const unsigned long long upto = r.lane == 63 ? ~0ull : ((2ull << r.lane) - 1ull);  // lanes 0..lane
    const unsigned long long after = hm & ~upto;
    r.head_lane = 63 - __clzll((long long)(hm & upto));
    r.run_end = after ? (__ffsll((unsigned long long)after) - 2) : 63;
    return r;
}

// Lane value x of the DPP source selected by kCtrl (row shift or row broadcast);
// lanes whose row is off in kRowMask, or whose source is out of the row, get 0.
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_get(double x) {
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), kCtrl, kRowMask, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, kRowMask, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// As dpp_get, but lanes whose row is off in kRowMask keep `old` (a value the
// caller no longer needs, so its registers take the result and no zeroing
// move is issued; the caller's factor for those lanes is 0).
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_get_or(double old, double x) {
    const long long b = __double_as_longlong(x), o = __double_as_longlong(old);
    const int lo = __builtin_amdgcn_update_dpp((int)(o & 0xffffffffll), (int)(b & 0xffffffffll), kCtrl, kRowMask,
                                               0xf, true);
    const int hi = __builtin_amdgcn_update_dpp((int)(o >> 32), (int)(b >> 32), kCtrl, kRowMask, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

// Segmented inclusive prefix sum over the wave: after the call the LAST lane of
// each run (lane == run_end) holds the run's total.  Hillis-Steele within rows
// of 16 lanes by DPP row shifts (1, 2, 4, 8), then the row broadcasts of lane 15
// (into rows 1, 3) and lane 31 (into rows 2, 3); a lane only adds a partial sum
// whose lanes all belong to its own run, selected by a 0/1 factor rather than a
// branch.  The broadcasts leave the rows they skip holding the previous round's
// fetched partial sum (finite), which their factor 0 discards.
__device__ __forceinline__ double run_total(double x, const WaveRuns &r) {
    const int h = r.head_lane, l = r.lane;
    double t = dpp_get<0x111, 0xf>(x);                                // row_shr:1
    x = fma(t, l - 1 >= h ? 1.0 : 0.0, x);
    t = dpp_get<0x112, 0xf>(x);                                       // row_shr:2
    x = fma(t, l - 2 >= h ? 1.0 : 0.0, x);
    t = dpp_get<0x114, 0xf>(x);                                       // row_shr:4
    x = fma(t, l - 4 >= h ? 1.0 : 0.0, x);
    t = dpp_get<0x118, 0xf>(x);                                       // row_shr:8
    x = fma(t, l - 8 >= h ? 1.0 : 0.0, x);
    t = dpp_get_or<0x142, 0xa>(t, x);                                 // row_bcast:15
    x = fma(t, (l & 16) != 0 && h < (l & 48) ? 1.0 : 0.0, x);
    t = dpp_get_or<0x143, 0xc>(t, x);                                 // row_bcast:31
    x = fma(t, l >= 32 && h < 32 ? 1.0 : 0.0, x);
    return x;
}

// ------------------------------------------------------------------ per-tet coefficients
// Inside a tet both field expansions are affine in the barycentrics:
//   E = sum_k l_k A_k,  A_k = sum_{j != k} sign(j - k) eps_{kj} grad l_j
//     (from W1_ij = l_i grad l_j - l_j grad l_i, edge (i<j) oriented i -> j);
//   B = sum_k l_k C_k,  C_k = 2 sum_{faces f containing k} beta_f (grad l_a x grad l_b)
//     (from W2 of face (a<b<c) = 2(l_a gb x gc + l_b gc x ga + l_c ga x gb); (k, a, b)
//     the cyclic order of f's ascending triple starting at k).
// eps, beta: the real parts Re{dof e^{jwt}} + dc of the edge and face DoFs at this
// step.  Two threads per tet: one for A_0..3, one for C_0..3.
//
// With kSnap = 3 the envelope itself is interpolated in time between three
// snapshots at the coarse field times t_{n-1}, t_n, t_{n+1} (the quadratic
// Lagrange basis N_{n,k}, eqs. newmark_L / newmark_N, used for the particle
// fields in the Particle Push section): dof(t) = sum_k w_k dof_k with the
// weights w_k = N_{n,k}(t) of the fine step's time, then modulated as above.
struct FieldPtrs {
    const double2 *e_env[3];
    const double *e_dc;
    const double2 *b_env[3];
    const double *b_dc;
    double w[3];   // snapshot weights (kSnap = 3)
    double c, s;   // cos(w t), sin(w t) of the fine step's time
    double w2[3], c2, s2;   // the same of the second step (kCoefPair)
    int xcd;       // coefficient pass: one contiguous tet range per XCD
};

// local edge index of the vertex pair {i, j}, i < j
__host__ __device__ constexpr int local_edge(int i, int j) { return i == 0 ? j - 1 : (i == 1 ? j + 1 : 5); }

template <int K>
__device__ __forceinline__ void coef_A(const int32_t *tp, const double g[4][3], const FieldPtrs &F, double A[3]) {
    A[0] = A[1] = A[2] = 0.0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (j == K) continue;
        const int id = tp[local_edge(j < K ? j : K, j < K ? K : j)];
        const double2 z = F.e_env[0][id];
        double eps = z.x * F.c - z.y * F.s;
        if (F.e_dc) eps += F.e_dc[id];
        if (j < K) eps = -eps;
#pragma unroll
        for (int d = 0; d < 3; ++d) A[d] += eps * g[j][d];
    }
}

template <int K>
__device__ __forceinline__ void coef_C(const int32_t *tp, const double g[4][3], const FieldPtrs &F, double Cv[3]) {
    Cv[0] = Cv[1] = Cv[2] = 0.0;
    constexpr int lf[4][3] = {{1, 2, 3}, {0, 2, 3}, {0, 1, 3}, {0, 1, 2}};
#pragma unroll
    for (int f = 0; f < 4; ++f) {
        if (f == K) continue;
        const int a = lf[f][0] == K ? lf[f][1] : (lf[f][1] == K ? lf[f][2] : lf[f][0]);
        const int b = lf[f][0] == K ? lf[f][2] : (lf[f][1] == K ? lf[f][0] : lf[f][1]);
        const int id = tp[6 + f];
        const double2 z = F.b_env[0][id];
        double beta = z.x * F.c - z.y * F.s;
        if (F.b_dc) beta += F.b_dc[id];
        beta *= 2.0;
        Cv[0] += beta * (g[a][1] * g[b][2] - g[a][2] * g[b][1]);
        Cv[1] += beta * (g[a][2] * g[b][0] - g[a][0] * g[b][2]);
        Cv[2] += beta * (g[a][0] * g[b][1] - g[a][1] * g[b][0]);
    }
}

// What the particle kernel reads per tet besides this step's coefficients: the
// barycentric gradients grad l_1..3 (9 reals, in the kernel's precision) and the
// six global edge ids, packed in one row so that a run's lanes touch one
// contiguous record (float64: 9 doubles + 6 int32 = 96 B; float32: 9 floats,
// one pad, 6 int32 = 64 B).
template <typename Real>
struct PushRow;
template <>
struct PushRow<double> {
    static constexpr int kStride = 12;   // doubles per row
    static constexpr int kEdges = 9;     // first edge id at this Real offset
};
template <>
struct PushRow<float> {
    static constexpr int kStride = 16;
    static constexpr int kEdges = 10;
};

// The particle step's per-step coefficient row.  Inside a tet a Whitney edge
// field is E(x) = A_0 + beta x (x - r_0) (its Jacobian is antisymmetric,
// beta = sum over edges (i<j) of eps_ij grad l_i x grad l_j, half its curl) and
// a Whitney face field is B(x) = C_0 + b (x - r_0) (its Jacobian is b times
// the identity, b = div B / 3 = (sum_k C_k . grad l_k) / 3): A_0 (3), beta (3),
// C_0 (3), b, with x - r_0 = sum_{k>0} l_k (r_k - r_0) from the static
// geometry row.  10 reals; float rows are padded to 12 (16-byte aligned).
template <typename Real>
struct CoefRow;
template <>
struct CoefRow<double> {
    static constexpr int kStride = 10;
};
template <>
struct CoefRow<float> {
    static constexpr int kStride = 12;
};

// Static per-tet geometry row: the edge vectors r_1 - r_0, r_2 - r_0, r_3 - r_0
// of the canonical vertex order (9 reals, padded to 16-byte rows).
template <typename Real>
struct GeoRow;
template <>
struct GeoRow<double> {
    static constexpr int kStride = 10;
};
template <>
struct GeoRow<float> {
    static constexpr int kStride = 12;
};

// The coefficient pass reads the float64 push row (grad l_1..3 and the edge ids;
// grad l_0 = -(grad l_1 + grad l_2 + grad l_3), the sum the mesh tables define it
// by) and the four face ids of the tet: 112 B per tet.
// The dispatcher deals consecutive blocks round-robin over the 8 XCDs; this
// renumbering gives each XCD one contiguous range of the G blocks instead, so
// the tets (and the edges and faces they share) of an XCD's blocks stay in its
// L2.  The coefficient pass takes it when an XCD's share of the field DoFs
// fits its 4 MB L2; on larger meshes the round-robin order, whose neighbouring
// chunks run at the same time on different XCDs and share lines through the
// Infinity Cache, measured faster.
__device__ __forceinline__ unsigned xcd_block(unsigned c, unsigned G) {
    const unsigned q = G / 8, r = G % 8, x = c % 8, j = c / 8;
    return x * q + min(x, r) + j;
}

// The particle step's row is linear in the tet's DoFs, so it splits into the
// rows of the real, imaginary and dc parts: row(t) = dc + sum_k (wc_k re_k -
// ws_k im_k), wc_k = w_k cos wt, ws_k = w_k sin wt.  kRowParts counts them.
template <int kSnap>
constexpr int kRowParts = 2 * kSnap + 1;   // re_0, im_0, re_1, ..., dc
constexpr int kRowReals = 10;              // A_0, beta, C_0, b

// One step's row entry from its parts (stride reals apart).  Written in fma
// so that every kernel that forms a row, one step or several per launch,
// rounds it alike.
template <int kSnap>
__device__ __forceinline__ double row_entry(const double *part, int stride, const double *wc, const double *ws) {
    double v = part[(kRowParts<kSnap> - 1) * stride];
#pragma unroll
    for (int k = 0; k < kSnap; ++k) {
        v = fma(-part[(2 * k + 1) * stride], ws[k], v);
        v = fma(part[2 * k * stride], wc[k], v);
    }
    return v;
}

// a x b, each component one product and one fma
__device__ __forceinline__ void cross_fma(const double a[3], const double b[3], double o[3]) {
    o[0] = fma(a[1], b[2], -(a[2] * b[1]));
    o[1] = fma(a[2], b[0], -(a[0] * b[2]));
    o[2] = fma(a[0], b[1], -(a[1] * b[0]));
}

// Half a row from the DoFs z of the tet's edges (face = 0: A_0 = E(r_0) =
// sum_j eps_0j grad l_j and beta = sum_(i<j) eps_ij grad l_i x grad l_j) or
// faces (face = 1: C_0 = B(r_0) and b = (sum_k C_k . grad l_k) / 3, then two
// zeros).  With X_ab = grad l_a x grad l_b, face (a<b<c) adds 2 z (X_bc, -X_ac,
// X_ab) to C_a, C_b, C_c, so C_0 takes faces 1..3 and b is the sum over faces
// of 2 z grad l_a . X_bc.  (Both branches assign o in the same order: stored
// in different orders, their results met in scratch memory.)
__device__ __forceinline__ void half_row(int face, const double z[6], const double g[4][3], const double gxg[6][3],
                                         double o[6]) {
    if (face) {
        const double b0 = 2.0 * z[0], b1 = 2.0 * z[1], b2 = 2.0 * z[2], b3 = 2.0 * z[3];
        auto triple = [](const double *a, const double *X) { return fma(a[0], X[0], fma(a[1], X[1], a[2] * X[2])); };
        // faces (1,2,3), (0,2,3), (0,1,3), (0,1,2)
        const double c0 = fma(b3, gxg[3][0], fma(b2, gxg[4][0], b1 * gxg[5][0]));
        const double c1 = fma(b3, gxg[3][1], fma(b2, gxg[4][1], b1 * gxg[5][1]));
        const double c2 = fma(b3, gxg[3][2], fma(b2, gxg[4][2], b1 * gxg[5][2]));
        const double b = fma(b3, triple(g[0], gxg[3]),
                             fma(b2, triple(g[0], gxg[4]), fma(b1, triple(g[0], gxg[5]), b0 * triple(g[1], gxg[5]))));
        o[0] = c0;
        o[1] = c1;
        o[2] = c2;
        o[3] = b;
        o[4] = 0.0;
        o[5] = 0.0;
    } else {
        double r[6];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            r[d] = fma(z[2], g[3][d], fma(z[1], g[2][d], z[0] * g[1][d]));
            double b = z[0] * gxg[0][d];
#pragma unroll
            for (int e = 1; e < 6; ++e) b = fma(z[e], gxg[e][d], b);
            r[3 + d] = b;
        }
        o[0] = r[0];
        o[1] = r[1];
        o[2] = r[2];
        o[3] = r[3];
        o[4] = r[4];
        o[5] = r[5];
    }
}

// Clears the current slots of tets [T0, T0 + nloc) (by one block; null: none).
// A call clears the slots it is about to use in its first kernel, the
// coefficient pass, beside whose gathers these stores run (behind its own
// stores they cost small calls up to 1 %): so a call recorded into a graph
// may be replayed, and one that stopped short leaves nothing for the next.
// (Each slot cleared by the edge that read it: 8-byte stores out of order,
// 35 instead of 19 us on 384,000 tets; a fill of its own: one launch more.)
__device__ __forceinline__ void clear_slots(double *slots, int64_t T0, int nloc) {
    if (!slots) return;
    double2 *dst = reinterpret_cast<double2 *>(slots + T0 * 8);
    for (int i = threadIdx.x; i < nloc * 4; i += blockDim.x) dst[i] = make_double2(0.0, 0.0);
}

// What a coefficient pass writes per tet: the particle step's 10 reals of one
// step (CoefRow), the parts of the 10-real row (kRowParts * 10 float64) from
// which a multi-step launch forms the row of each of its steps, or the float64
// rows of two steps and a third of zeros, which a launch reads as the parts of
// one snapshot: re alone (weights 1, 0) is the first step's row, im alone
// (weights 0, -1) the second's.
enum CoefMode { kCoefStep, kCoefParts, kCoefPair };

template <typename Real, int kSnap, int kMode>
__device__ __forceinline__ void tet_coef(int64_t nt, const double *__restrict__ prow,
                                         const int32_t *__restrict__ tetface, const FieldPtrs &F,
                                         Real *__restrict__ coef, double *__restrict__ slots, unsigned blk) {
    // A block covers kTets tets.  Their push rows and face ids are staged in
    // LDS with coalesced 16-byte loads; then the block's first kTets lanes
    // take the edges and the other kTets lanes the faces, so each wavefront
    // takes one branch with all its lanes; the rows go back through LDS and
    // out with coalesced stores.  (Each lane reading its own 96-byte row and
    // writing its own half row strides every load and store instruction over
    // 64 rows.)  Row strides in LDS are odd numbers of reals, so that the
    // lanes' rows start in different banks.
    constexpr int kTets = kBlock / 2;
    constexpr int kRow = PushRow<double>::kStride + 1;   // staged push row, doubles
    constexpr int kOut = 11;                             // staged coefficient row, Reals
    constexpr int kPart0 = 6, kPart1 = 4;                // reals of each half
    constexpr int kOutRow = CoefRow<Real>::kStride;      // row in memory, Reals
    constexpr int kIn = kTets * kRow + kTets * 4 / 2;    // rows + face ids, in doubles
    constexpr int kOutD = (kTets * kOut * (int)sizeof(Real) + 7) / 8;
    __shared__ double lds[kIn > kOutD ? kIn : kOutD];
    const int64_t T0 = (int64_t)blk * kTets;
    if (T0 >= nt) return;   // uniform over the block
    const int nloc = (int)min<int64_t>(kTets, nt - T0);
    double *srow = lds;
    int4 *sface = reinterpret_cast<int4 *>(lds + kTets * kRow);
    {
        const double2 *src = reinterpret_cast<const double2 *>(prow + T0 * PushRow<double>::kStride);
        constexpr int kHalf = PushRow<double>::kStride / 2;   // double2 per row
        for (int i = threadIdx.x; i < nloc * kHalf; i += kBlock) {
            const double2 v = src[i];
            const int t = i / kHalf, c = 2 * (i - t * kHalf);
            srow[t * kRow + c] = v.x;
            srow[t * kRow + c + 1] = v.y;
        }
        const int4 *tf = reinterpret_cast<const int4 *>(tetface) + T0;
        for (int i = threadIdx.x; i < nloc; i += kBlock) sface[i] = tf[i];
    }
    __syncthreads();
    clear_slots(slots, T0, nloc);
    const int part = (int)(threadIdx.x >= kTets);
    const int t = threadIdx.x & (kTets - 1);
    const bool act = t < nloc;
    double g[4][3];
    int32_t id[6];   // this half's edge ids or (first four) face ids
    if (act) {
        const double *row = srow + t * kRow;
#pragma unroll
        for (int k = 1; k < 4; ++k)
#pragma unroll
            for (int d = 0; d < 3; ++d) g[k][d] = row[3 * (k - 1) + d];
#pragma unroll
        for (int d = 0; d < 3; ++d) g[0][d] = -(g[1][d] + g[2][d] + g[3][d]);
        const int32_t *re = reinterpret_cast<const int32_t *>(row + PushRow<double>::kEdges);
        const int4 fc = sface[t];
        id[0] = part ? fc.x : re[0];
        id[1] = part ? fc.y : re[1];
        id[2] = part ? fc.z : re[2];
        id[3] = part ? fc.w : re[3];
        id[4] = re[4];
        id[5] = re[5];
    }
    {
        // parts of the row, one after the other: real and imaginary part of
        // each snapshot, then dc
        constexpr int kParts = kRowParts<kSnap>;
        double gxg[6][3];
        if (act) {
            cross_fma(g[0], g[1], gxg[0]);
            cross_fma(g[0], g[2], gxg[1]);
            cross_fma(g[0], g[3], gxg[2]);
            cross_fma(g[1], g[2], gxg[3]);
            cross_fma(g[1], g[3], gxg[4]);
            cross_fma(g[2], g[3], gxg[5]);
        }
        // the dc part, and the real and imaginary parts of snapshot k, of this
        // half's reals of the row
        auto dc_part = [&](double o[6]) {
            double z[6];
            const double *dc = part ? F.b_dc : F.e_dc;
#pragma unroll
            for (int e = 0; e < 6; ++e) z[e] = dc && (e < 4 || !part) ? dc[id[e]] : 0.0;
            half_row(part, z, g, gxg, o);
        };
        auto env_parts = [&](int k, double re[6], double im[6]) {
            double zr[6], zi[6];
            const double2 *env = part ? F.b_env[k] : F.e_env[k];
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                double2 z = make_double2(0.0, 0.0);
                if (e < 4 || !part) z = env[id[e]];
                zr[e] = z.x;
                zi[e] = z.y;
            }
            half_row(part, zr, g, gxg, re);
            half_row(part, zi, g, gxg, im);
        };
        if constexpr (kMode == kCoefStep) {
            double o[6];
            if (act) {
                dc_part(o);
#pragma unroll
                for (int k = 0; k < kSnap; ++k) {   // as row_entry
                    double re[6], im[6];
                    env_parts(k, re, im);
                    const double wc = F.w[k] * F.c, ws = F.w[k] * F.s;
#pragma unroll
                    for (int d = 0; d < 6; ++d) o[d] = fma(re[d], wc, fma(-im[d], ws, o[d]));
                }
            }
            __syncthreads();
            Real *sout = reinterpret_cast<Real *>(lds);
            if (act) {
                if (part == 0) {
#pragma unroll
                    for (int d = 0; d < kPart0; ++d) sout[t * kOut + d] = (Real)o[d];
                } else {
#pragma unroll
                    for (int d = 0; d < kPart1; ++d) sout[t * kOut + kPart0 + d] = (Real)o[d];
                }
            }
            __syncthreads();
            Real *dst = coef + T0 * kOutRow;
            for (int i = threadIdx.x; i < nloc * kOutRow; i += kBlock) {
                const int tt = i / kOutRow, c = i - tt * kOutRow;
                dst[i] = c < kRowReals ? sout[tt * kOut + c] : (Real)0;
            }
        } else {
            constexpr int kOuts = kMode == kCoefPair ? 3 : kParts;   // tens of reals per tet
            double *sout = lds;
            auto put = [&](int q, const double o[6]) {
                __syncthreads();   // the staged rows or the previous part read
                if (act) {
                    if (part == 0) {
#pragma unroll
                        for (int d = 0; d < kPart0; ++d) sout[t * kOut + d] = o[d];
                    } else {
#pragma unroll
                        for (int d = 0; d < kPart1; ++d) sout[t * kOut + kPart0 + d] = o[d];
                    }
                }
                __syncthreads();
                double *dst = coef + T0 * (kOuts * kRowReals) + q * kRowReals;
                for (int i = threadIdx.x; i < nloc * kRowReals; i += kBlock) {
                    const int tt = i / kRowReals, c = i - tt * kRowReals;
                    dst[(int64_t)tt * (kOuts * kRowReals) + c] = sout[tt * kOut + c];
                }
            };
            if constexpr (kMode == kCoefPair) {
                double o[6], o2[6];
                const double none[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
                if (act) {
                    dc_part(o);
#pragma unroll
                    for (int d = 0; d < 6; ++d) o2[d] = o[d];
#pragma unroll
                    for (int k = 0; k < kSnap; ++k) {   // as row_entry
                        double re[6], im[6];
                        env_parts(k, re, im);
                        const double wc = F.w[k] * F.c, ws = F.w[k] * F.s;
                        const double wc2 = F.w2[k] * F.c2, ws2 = F.w2[k] * F.s2;
#pragma unroll
                        for (int d = 0; d < 6; ++d) {
                            o[d] = fma(re[d], wc, fma(-im[d], ws, o[d]));
                            o2[d] = fma(re[d], wc2, fma(-im[d], ws2, o2[d]));
                        }
                    }
                }
                put(0, o);
                put(1, o2);
                put(2, none);
            } else {
#pragma unroll
                for (int k = 0; k < kSnap; ++k) {
                    double re[6], im[6];
                    if (act) env_parts(k, re, im);
                    put(2 * k, re);
                    put(2 * k + 1, im);
                }
                double o[6];
                if (act) dc_part(o);
                put(kParts - 1, o);
            }
        }
    }
}

template <typename Real, int kSnap, int kMode>
__global__ void __launch_bounds__(kBlock) k_tet_coef(int64_t nt, const double *__restrict__ prow,
                                                     const int32_t *__restrict__ tetface, FieldPtrs F,
                                                     Real *__restrict__ coef, double *__restrict__ slots) {
    tet_coef<Real, kSnap, kMode>(nt, prow, tetface, F, coef, slots,
                                 F.xcd ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x);
}

// ------------------------------------------------------------------ particle step
template <typename Real>
__device__ __forceinline__ const int32_t *push_row_edges(const Real *row) {
    return reinterpret_cast<const int32_t *>(row + PushRow<Real>::kEdges);
}

template <typename Real>
struct StepArgs {
    int64_t n, nt;
    double *lam1, *lam2, *lam3;
    Real *v0, *v1, *v2;
    int32_t *tet;
    const Real *coef;          // nt rows of CoefRow<Real>: A_0, beta, C_0, b of this step (k_tet_coef)
    const Real *gpush;         // nt rows of PushRow<Real>::kStride: grad l_1..3, then the 6 edge ids
    const Real *geo;           // nt rows of GeoRow<Real>: r_1 - r_0, r_2 - r_0, r_3 - r_0
    const double *grad;        // nt*12 float64 barycentric gradients grad l_0..3
    const TetTopo *topo;
    double *dG;
    double *rho;
    int fixed;                 // lam1..3 hold uint32 fixed-point barycentrics (float kernels only)
    double *tetG;              // nt*8 per-tet current slots (q w * the six path-integral sums of
                               // the tet's runs), or null: the runs then add to dG directly
    unsigned *status;
    unsigned *walk_queue;      // particles that left their tet
    unsigned *slice_queue;     // 64-particle slices whose walkers did not fit in walk_queue
    unsigned *walk_ctr;        // [0] walk_queue length, [1] walk blocks done, [2] slice_queue length
    int walk_by_slice;         // queue every walker by its slice (the overflow path)
    // Counting-sort scatter fused into the step (k_push_sort): the particles
    // read from the arrays above are written, pushed, at their sorted
    // positions cursor[T]++ of these arrays; the walk after it runs on them.
    double *o_lam1, *o_lam2, *o_lam3;
    Real *o_v0, *o_v1, *o_v2;
    int32_t *o_tet;
    const int64_t *id;
    int64_t *o_id;
    unsigned *cursor;          // exclusive prefix sums of the tet counts
    int scatter;               // the walk follows a scatter step: its queue
                               // overflow is handled by a scan of all particles
    double qw;
    Real h;                    // q dt / (2 m)
    Real dt_r;
};

// A particle that leaves its tet is marked in place (tet = -(T + 2)) by the
// step kernel, which keeps its start barycentrics and stores its new velocity;
// its wavefront's index goes to the walk queue.  k_walk then walks it.
__device__ __forceinline__ int walker_mark(int T) { return -(T + 2); }
__device__ __forceinline__ int walker_tet(int marked) { return -marked - 2; }

// q w * path integral of the six edge functions along one straight piece inside
// a tet: with lam linear along the piece, int W1_ij . dr = m_i dl_j - m_j dl_i,
// m = lam at the midpoint, dl the barycentric increment of the piece.
__device__ __forceinline__ void piece_sums(const double l[4], const double dl[4], double g6[6]) {
    double m[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) m[k] = l[k] + 0.5 * dl[k];
    const int le[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
#pragma unroll
    for (int e = 0; e < 6; ++e) g6[e] = m[le[e][0]] * dl[le[e][1]] - m[le[e][1]] * dl[le[e][0]];
}

__device__ __forceinline__ void deposit_piece(double *__restrict__ dG, const TetTopo &tp, const double l[4],
                                              const double dl[4], double qw) {
    double g6[6];
    piece_sums(l, dl, g6);
#pragma unroll
    for (int e = 0; e < 6; ++e) unsafeAtomicAdd(&dG[tp.e[e]], qw * g6[e]);
}

// lambda_0 = 1 - (l1 + l2 + l3) with the rounding error of the sum carried
// along (Knuth's two-sum).  Near face 0 lambda_0 is small, and a plainly rounded
// sum leaves it uncertain by a unit in the last place of the sum; the crossing
// parameter lambda_0 / -dlambda_0 of a path leaving through that face would
// inherit that error divided by the step's barycentric length (~1e-5).
__device__ __forceinline__ double lam0_of(double l1, double l2, double l3) {
    const double s = l1 + l2;
    const double bs = s - l1;
    double e = (l1 - (s - bs)) + (l2 - bs);
    const double t = s + l3;
    const double bt = t - s;
    e += (s - (t - bt)) + (l3 - bt);
    return (1.0 - t) - e;
}

// Fixed-point barycentrics (the compact mixed form): lambda_k = u_k * 2^-32,
// u_k uint32, lambda_0 = 1 - the sum, which is exact.  Every such number and
// every difference of two of them is exact in float64.
constexpr double kFix = 2.3283064365386962890625e-10;   // 2^-32
constexpr double kFixScale = 4294967296.0;              // 2^32

__device__ __forceinline__ double fix_to_real(uint32_t u) { return (double)u * kFix; }

// The nearest fixed-point barycentrics to (l1, l2, l3) that keep lambda_0 =
// 1 - l1 - l2 - l3 >= 0: each rounded to the nearest multiple of 2^-32 (in
// [0, 1 - 2^-32]); if the three then sum past 1 (by at most the rounding of
// the three, for a point with lambda_0 >= 0) the largest gives up the excess.
// (A point far outside the tet, which no step stores, would have the excess
// taken from the largest remaining coordinates in turn, none below zero.)
__device__ __forceinline__ void fix_round3(double l1, double l2, double l3, uint32_t u[3]) {
    const double l[3] = {l1, l2, l3};
#pragma unroll
    for (int k = 0; k < 3; ++k) u[k] = (uint32_t)fmin(fmax(rint(l[k] * kFixScale), 0.0), kFixScale - 1.0);
    const uint64_t sum = (uint64_t)u[0] + u[1] + u[2];
    if (sum > (1ull << 32)) {
        uint64_t excess = sum - (1ull << 32);
        for (int pass = 0; pass < 3 && excess > 0; ++pass) {
            const int big = (u[0] >= u[1] && u[0] >= u[2]) ? 0 : (u[1] >= u[2] ? 1 : 2);
            const uint32_t take = (uint32_t)(excess < u[big] ? excess : u[big]);
#pragma unroll
            for (int k = 0; k < 3; ++k)
                if (k == big) u[k] -= take;
            excess -= take;
        }
    }
}

// Barycentric k of particle p from an array of either storage.
__device__ __forceinline__ double lam_at(const double *arr, int64_t p, int fixed) {
    return fixed ? fix_to_real(reinterpret_cast<const uint32_t *>(arr)[p]) : arr[p];
}

// Walk of the straight path with Cartesian remaining displacement d, starting in
// tet T at barycentrics l (l[0] is recomputed from l[1..3] by lam0_of).  Each piece is deposited.  At a face crossing the exit
// coordinate is set to exactly 0, the other three are rescaled to sum to one and
// handed to the neighbour's shared vertices; at a boundary face the remaining
// displacement and the velocity are reflected about the face normal.
// With kTrack (used by the adjoint) nothing is deposited and R accumulates the
// linear part of the step's reflections (R <- (I - 2 n n^T) R per wall hit):
// the end point is R (x + dt v) + const and the stored velocity is R v.
// kExtra further vectors ext[0..kExtra-1] (the velocity samples a multistep
// integrator keeps) are reflected with the velocity at a wall.
// With `fixed` the end point is rounded to the fixed-point barycentrics (as
// fix_round3) and the last piece runs to that rounded point, so that the
// deposit and the stored end point agree exactly.
//
// The next tet's records are requested before the crossed piece's atomics are
// issued: loads complete in order with them, and one behind six atomics would
// wait for all six.  With `last` (lstart, dl) the piece in the final tet is not
// deposited but returned, from where it starts.
// `crossed` takes the pieces up to a face, onto the edges of their tet unless
// the caller has a place for them.  Products and sums are fused where it says
// fma and nowhere else that the path depends on: the end point must be the
// same bits whatever is done with the pieces.
struct LastPiece {
    double l[4], dl[4];
};
struct ToEdges {
    double *dG, qw;
    __device__ __forceinline__ void operator()(int, const TetTopo &tp, const double l[4], const double dl[4]) const {
        deposit_piece(dG, tp, l, dl, qw);
    }
};
template <typename Real, bool kTrack, int kExtra = 0, typename Crossed>
__device__ __forceinline__ int walk_pieces(const StepArgs<Real> &a, int T, double l[4], double d[3], Real v[3],
                                           double *R, double (*ext)[3], bool fixed, LastPiece *last,
                                           const Crossed &crossed) {
    int hops = 0;
    l[0] = lam0_of(l[1], l[2], l[3]);
    double g[4][3];
    auto load_grad = [&](int t) {
        const double *gp = a.grad + (int64_t)t * 12;
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) g[k][c] = gp[3 * k + c];
    };
    load_grad(T);
    TetTopo tp = a.topo[T];
    if (last) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            last->l[k] = l[k];
            last->dl[k] = 0.0;
        }
    }
    for (;;) {
        double dl[4];
#pragma unroll
        for (int k = 1; k < 4; ++k) dl[k] = fma(g[k][2], d[2], fma(g[k][0], d[0], g[k][1] * d[1]));
        dl[0] = -(dl[1] + dl[2] + dl[3]);
        double smin = 1.0;
        int kmin = -1;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (dl[k] < 0.0 && l[k] + dl[k] < 0.0) {
                const double sk = l[k] > 0.0 ? l[k] / (-dl[k]) : 0.0;
                if (kmin < 0 || sk < smin) {
                    smin = sk;
                    kmin = k;
                }
            }
        }
        // values at the exit face, selected without dynamic register indexing
        double gx = 0.0, gy = 0.0, gz = 0.0;
        int nb = -1;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (k == kmin) {
                gx = g[k][0];
                gy = g[k][1];
                gz = g[k][2];
                nb = tp.n[k];
            }
        if (kmin < 0) {
            if (fixed) {
                uint32_t u[3];
                fix_round3(l[1] + dl[1], l[2] + dl[2], l[3] + dl[3], u);
                double lq[4];
#pragma unroll
                for (int k = 1; k < 4; ++k) lq[k] = fix_to_real(u[k - 1]);
                lq[0] = 1.0 - lq[1] - lq[2] - lq[3];
#pragma unroll
                for (int k = 0; k < 4; ++k) dl[k] = lq[k] - l[k];
            }
            if (last) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    last->l[k] = l[k];
                    last->dl[k] = dl[k];
                }
            } else if (!kTrack) {
                deposit_piece(a.dG, tp, l, dl, a.qw);
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) l[k] += dl[k];
            break;
        }
        const TetTopo from = tp;
        if (nb >= 0) {
            load_grad(nb);
            tp = a.topo[nb];
        }
        double dlp[4];
        {
            // (rounded: its sum with l below must not become an fma in one form of the walk only)
#pragma clang fp contract(off)
#pragma unroll
            for (int k = 0; k < 4; ++k) dlp[k] = smin * dl[k];
        }
        if (!kTrack) crossed(T, from, l, dlp);
        double lc[4], sum = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            lc[k] = (k == kmin) ? 0.0 : fmax(l[k] + dlp[k], 0.0);
            sum += lc[k];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) lc[k] /= sum;
#pragma unroll
        for (int c = 0; c < 3; ++c) d[c] = fma(-smin, d[c], d[c]);
        if (nb < 0) {
            const double nn = sqrt(fma(gz, gz, fma(gx, gx, gy * gy)));
            const double nh[3] = {gx / nn, gy / nn, gz / nn};
            double dd = fma(d[2], nh[2], fma(d[0], nh[0], d[1] * nh[1]));
            Real vv = fma(v[2], (Real)nh[2], fma(v[0], (Real)nh[0], v[1] * (Real)nh[1]));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                d[c] = fma(-(2.0 * dd), nh[c], d[c]);
                v[c] = fma(-((Real)2 * vv), (Real)nh[c], v[c]);
            }
#pragma unroll
            for (int i = 0; i < kExtra; ++i) {
                const double xv = ext[i][0] * nh[0] + ext[i][1] * nh[1] + ext[i][2] * nh[2];
#pragma unroll
                for (int c = 0; c < 3; ++c) ext[i][c] -= 2.0 * xv * nh[c];
            }
            if (kTrack) {
#pragma unroll
                for (int j = 0; j < 3; ++j) {
                    const double col = nh[0] * R[j] + nh[1] * R[3 + j] + nh[2] * R[6 + j];
#pragma unroll
                    for (int i = 0; i < 3; ++i) R[3 * i + j] -= 2.0 * nh[i] * col;
                }
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) l[k] = lc[k];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double x = 0.0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (from.v[i] == tp.v[j]) x = lc[i];
                l[j] = x;
            }
            T = nb;
        }
        if (++hops > ETPIC_HOP_CAP) {
            atomicOr(a.status, (unsigned)ETPIC_DEV_HOPCAP);
            if (last) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    last->l[k] = l[k];
                    last->dl[k] = 0.0;
                }
            }
            break;
        }
    }
    return T;
}

template <typename Real, bool kTrack, int kExtra = 0>
__device__ __forceinline__ int walk(const StepArgs<Real> &a, int T, double l[4], double d[3], Real v[3], double *R,
                                   double (*ext)[3] = nullptr, bool fixed = false, LastPiece *last = nullptr) {
    return walk_pieces<Real, kTrack, kExtra>(a, T, l, d, v, R, ext, fixed, last, ToEdges{a.dG, a.qw});
}

// The sums of a piece (l, dl) added to s (edge_sums), in units of 1 / one.
__device__ __forceinline__ void add_piece(const LastPiece &q, double one, double s[6]) {
    const double l1 = q.l[1] * one, l2 = q.l[2] * one, l3 = q.l[3] * one;
    const double d1 = q.dl[1] * one, d2 = q.dl[2] * one, d3 = q.dl[3] * one;
    s[0] += d1;
    s[1] += d2;
    s[2] += d3;
    s[3] = fma(l1, d2, fma(-l2, d1, s[3]));
    s[4] = fma(l1, d3, fma(-l3, d1, s[4]));
    s[5] = fma(l2, d3, fma(-l3, d2, s[5]));
}

// q w * (the run's path-integral sums) onto the six edges of tet T, and
// q w * (its end-point barycentric sums) onto the four vertices if rho is kept.
template <typename Real, bool kRho, bool kSlots = false>
__device__ __forceinline__ void flush_run(const StepArgs<Real> &a, int T, const double g6[6], const double r4[4]) {
    if (kSlots) {
        double *slot = a.tetG + (int64_t)T * 8;
#pragma unroll
        for (int e = 0; e < 6; ++e)
            if (g6[e] != 0.0) unsafeAtomicAdd(&slot[e], a.qw * g6[e]);
    } else {
        const int32_t *ed = push_row_edges(a.gpush + (int64_t)T * PushRow<Real>::kStride);
#pragma unroll
        for (int e = 0; e < 6; ++e)
            if (g6[e] != 0.0) unsafeAtomicAdd(&a.dG[ed[e]], a.qw * g6[e]);
    }
    if (kRho) {
        const TetTopo *tp = a.topo + T;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (r4[k] != 0.0) unsafeAtomicAdd(&a.rho[tp->v[k]], a.qw * r4[k]);
    }
}

// The six edge sums of the runs that end in this wavefront, added by the last
// six lanes of each run together (lane run_end - k adds local edge k, its sum
// fetched from the run's last lane): the wavefront issues one atomic
// instruction where the run-end lanes alone would issue six.  The run-end
// lanes hand their six sums over through a wavefront-private LDS row (three
// 16-byte stores, one 8-byte load per flushing lane), which costs fewer
// vector instructions than five 64-bit lane shuffles and their selects.  With kSlots the
// sums go to the run's per-tet current slots (8 * T + k: the six lanes of a
// run address one 64-byte line), else to the six edges.  A run shorter than
// six lanes leaves its remaining edges to its last lane.  `flush` marks the
// run-end lanes whose run is complete (the others stay open).
template <typename Real, bool kSlots>
__device__ __forceinline__ void flush_runs_together(const StepArgs<Real> &a, int T, const double g6[6],
                                                   const WaveRuns &r, bool flush, double2 *buf) {
    const unsigned long long fm = __ballot(flush);
    const bool mine = (fm >> r.run_end) & 1ull;
    const int k = r.run_end - r.lane;
    const int len = r.run_end - r.head_lane + 1;
    if (flush) {
        double2 *row = buf + 3 * r.lane;
        row[0] = make_double2(g6[0], g6[1]);
        row[1] = make_double2(g6[2], g6[3]);
        row[2] = make_double2(g6[4], g6[5]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    double val = 0.0;
    if (mine && k < 6 && k < len) {
        const double *sr = reinterpret_cast<const double *>(buf + 3 * r.run_end);
        val = sr[k];
        if (kSlots) {
            double *slot = a.tetG + (int64_t)T * 8;
            if (val != 0.0) unsafeAtomicAdd(&slot[k], a.qw * val);
            if (k == 0 && len < 6) {
                for (int j = len; j < 6; ++j)
                    if (g6[j] != 0.0) unsafeAtomicAdd(&slot[j], a.qw * g6[j]);
            }
        } else {
            const int32_t *ed = push_row_edges(a.gpush + (int64_t)T * PushRow<Real>::kStride);
            if (val != 0.0) unsafeAtomicAdd(&a.dG[ed[k]], a.qw * val);
            if (k == 0 && len < 6) {
                for (int j = len; j < 6; ++j)
                    if (g6[j] != 0.0) unsafeAtomicAdd(&a.dG[ed[j]], a.qw * g6[j]);
            }
        }
    }
}

// The per-tet current slots of a multi-step call added to the edges: dG[e] +=
// the slots that name edge e, in the fixed order of the edge's CSR (no atomics:
// every particle and walk kernel of the call has finished).  The slots stay as
// they are: the next call's first kernel clears them (clear_slots).  Also
// clears the walk counters `ctr` of the call's last multi-step launch (null: none).
__global__ void __launch_bounds__(kBlock) k_slots_to_edges(int64_t ne, const int32_t *__restrict__ ptr,
                                                           const int32_t *__restrict__ slot,
                                                           const double *__restrict__ tetG, double *__restrict__ dG,
                                                           unsigned *__restrict__ ctr) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < ne; e += stride) {
        // eight slots at a time, their loads in flight together (an interior
        // edge of a tet mesh has about five)
        const int32_t i0 = ptr[e], i1 = ptr[e + 1];
        const double old = dG[e];
        double s = 0.0;
        for (int32_t i = i0; i < i1; i += 8) {
            int32_t at[8];
            double x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) at[k] = slot[min(i + k, i1 - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = tetG[at[k]];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (i + k < i1) s += x[k];
        }
        if (s != 0.0) dG[e] = old + s;
    }
    if (ctr && blockIdx.x == 0)
        for (unsigned i = threadIdx.x; i < kCtrStride; i += blockDim.x) ctr[i] = 0u;
}


// 2 / d for d >= 1 or NaN: the reciprocal refined, without the operand scaling
// a general division starts with.  float64: one cubic step from the hardware's
// reciprocal (measured within 2^-24, so the step's own error is below 2^-72);
// equal to 2.0 / d in each of 1e8 values over the whole range.  float32: the
// general division's steps, equal to its result below d = 2^126 (where the
// reciprocal's underflow ends: 0 beyond, for a rotation of more than 9e18 per
// step).  The fix-up gives 0 at d = inf.
__device__ __forceinline__ float two_over(float d) {
    float y = __builtin_amdgcn_rcpf(d);
    y = fmaf(fmaf(-d, y, 1.0f), y, y);
    float q = 2.0f * y;
    q = fmaf(fmaf(-d, q, 2.0f), y, q);
    q = fmaf(fmaf(-d, q, 2.0f), y, q);
    return __builtin_amdgcn_div_fixupf(q, d, 2.0f);
}
__device__ __forceinline__ double two_over(double d) {
    const double y = __builtin_amdgcn_rcp(d);
    const double e = fma(-d, y, 1.0), y2 = y + y;
    return __builtin_amdgcn_div_fixup(fma(y2, fma(e, e, e), y2), d, 2.0);
}

// Fields at the barycentrics x_1..3 of a tet and the Boris update of v:
// E = A_0 + beta x u, B = C_0 + b u at u = x - r_0 = sum_{k>0} x_k (r_k - r_0),
// half kick, rotation (implicit midpoint in v x B), half kick.  Shared by the
// one-step and the multi-step kernels, which thereby round alike.
__device__ __forceinline__ void gather_boris(const float *cf, const float *gm, const float x[3], float h, float v[3]) {
    float u[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = x[0] * gm[d] + x[1] * gm[3 + d] + x[2] * gm[6 + d];
    float E[3], B[3];
    E[0] = cf[0] + (cf[4] * u[2] - cf[5] * u[1]);
    E[1] = cf[1] + (cf[5] * u[0] - cf[3] * u[2]);
    E[2] = cf[2] + (cf[3] * u[1] - cf[4] * u[0]);
#pragma unroll
    for (int d = 0; d < 3; ++d) B[d] = cf[6 + d] + cf[9] * u[d];
    float vm[3], tau[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        vm[d] = v[d] + h * E[d];
        tau[d] = h * B[d];
    }
    const float t2 = tau[0] * tau[0] + tau[1] * tau[1] + tau[2] * tau[2];
    const float sg = two_over(1.0f + t2);
    const float vr[3] = {vm[0] + (vm[1] * tau[2] - vm[2] * tau[1]), vm[1] + (vm[2] * tau[0] - vm[0] * tau[2]),
                         vm[2] + (vm[0] * tau[1] - vm[1] * tau[0])};
    v[0] = vm[0] + sg * (vr[1] * tau[2] - vr[2] * tau[1]) + h * E[0];
    v[1] = vm[1] + sg * (vr[2] * tau[0] - vr[0] * tau[2]) + h * E[1];
    v[2] = vm[2] + sg * (vr[0] * tau[1] - vr[1] * tau[0]) + h * E[2];
}
// (float64: each sum one chain of fma)
__device__ __forceinline__ void gather_boris(const double *cf, const double *gm, const double x[3], double h,
                                             double v[3]) {
    double u[3], E[3], vm[3], tau[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = fma(x[2], gm[6 + d], fma(x[1], gm[3 + d], x[0] * gm[d]));
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = (d + 1) % 3, q = (d + 2) % 3;
        E[d] = fma(cf[3 + p], u[q], fma(-cf[3 + q], u[p], cf[d]));
        tau[d] = h * fma(cf[9], u[d], cf[6 + d]);
        vm[d] = fma(h, E[d], v[d]);
    }
    const double sg = two_over(fma(tau[0], tau[0], fma(tau[1], tau[1], fma(tau[2], tau[2], 1.0))));
    double vr[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = (d + 1) % 3, q = (d + 2) % 3;
        vr[d] = fma(vm[p], tau[q], fma(-vm[q], tau[p], vm[d]));
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = (d + 1) % 3, q = (d + 2) % 3;
        v[d] = fma(sg, fma(vr[p], tau[q], -(vr[q] * tau[p])), fma(h, E[d], vm[d]));
    }
}

// Barycentric increments dl_1..3 of the displacement dt v and the end point t,
// in units of 1 / one (t_0 = one - t_1 - t_2 - t_3: lam0 is stored implicitly);
// true if the particle stays in its tet.  A non-finite velocity never stays:
// it makes every increment non-finite, hence some t negative or NaN.
template <typename Real>
__device__ __forceinline__ bool increments(const Real *gr, const Real v[3], Real dt, double one, const double l[4],
                                           double dl[4], double t[4]) {
    const Real dx[3] = {dt * v[0], dt * v[1], dt * v[2]};
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        if constexpr (std::is_same<Real, float>::value)
            dl[k] = (double)(gr[3 * k - 3] * dx[0] + gr[3 * k - 2] * dx[1] + gr[3 * k - 1] * dx[2]);
        else
            dl[k] = fma(gr[3 * k - 1], dx[2], fma(gr[3 * k - 2], dx[1], gr[3 * k - 3] * dx[0]));
    }
#pragma unroll
    for (int k = 1; k < 4; ++k) t[k] = l[k] + dl[k];
    t[0] = one - t[1] - t[2] - t[3];
    return t[0] >= 0.0 && t[1] >= 0.0 && t[2] >= 0.0 && t[3] >= 0.0;
}

// Path integrals of the six edge functions from the sums over straight in-tet
// pieces of dl_1..3 and a_12, a_13, a_23, a_kj = l_k dl_j - l_j dl_k: with m the
// midpoint of a piece, m_k dl_j - m_j dl_k = a_kj, and m_0 dl_j - m_j dl_0 =
// dl_j - sum_k a_kj (the barycentrics sum to one, the increments to zero).
__device__ __forceinline__ void edge_sums(const double s[6], double g6[6]) {
    g6[0] = s[0] + s[3] + s[4];
    g6[1] = s[1] - s[3] + s[5];
    g6[2] = s[2] - s[4] - s[5];
    g6[3] = s[3];
    g6[4] = s[4];
    g6[5] = s[5];
}

// ------------------------------------------------------------------ particle step
// One lane per particle, particles kept sorted by tet.  Each lane reads its
// tet's row of this step's coefficient table (lanes of a run share the row, so
// the loads coalesce), gathers E and B, applies the Boris update and, if the
// particle stays in its tet (the common case), computes the six in-tet path
// integrals.  These are summed over each run of equal tet within the
// wavefront (segmented scan by DPP lane moves); the run's last lane
// adds the sums to the edges with float64 global atomics.  There are no block
// barriers, so latency is hidden by occupancy alone.  Particles that leave
// their tet are marked and their 64-particle slice queued for k_walk.
//
// A wavefront handles kSlices consecutive slices of 64 particles.  With more
// than one, the run that reaches lane 63 stays open: its sums are parked in
// LDS and taken over by lane 0 of the next slice if the tet continues, so a
// tet holding thousands of particles is flushed a few times instead of once
// per wavefront (same-address atomics from many wavefronts serialise).  With
// about one wavefront's worth of particles per tet or fewer, one slice per
// wavefront keeps more wavefronts in flight and is faster.
// Whether a particle kernel adds its runs' sums to the per-tet current slots
// (added to the edges once per call) or straight to the edges: the slots cost
// one cache line per run instead of six, which pays in every form except the
// float64 kernels with several slices per wavefront, where the slot path's
// registers spill (measured: float64 4-slice kernel 1.20 -> 1.24 ms).
template <typename Real>
constexpr __host__ __device__ bool push_uses_slots(int slices) {
    return std::is_same<Real, float>::value || slices == 1;
}

// Element ln of a wavefront-uniform array: the scalar base plus a 32-bit byte
// offset, which the global loads and stores take as such (base in scalar
// registers, one offset register shared by every array of the same element
// size) instead of a 64-bit address per array and lane.
template <typename T>
__device__ __forceinline__ T *lane_at(T *base, unsigned ln) {
    return reinterpret_cast<T *>(reinterpret_cast<char *>(base) + ln * (unsigned)sizeof(T));
}

template <typename Real, int kSlices, bool kRho, bool kScatter = false, bool kFixed = false, bool kPipe = false>
__device__ __forceinline__ void push_slices(const StepArgs<Real> &a, int remap) {
    static_assert(!kFixed || std::is_same<Real, float>::value, "fixed-point barycentrics are a mixed-form storage");
    unsigned blk = blockIdx.x;
    if (remap) {
        // the dispatcher deals blocks round-robin over the 8 XCDs; give each XCD
        // one contiguous range of particles (hence of tets and edges in its L2)
        const unsigned G = gridDim.x, q = G / 8, r = G % 8, x = blk % 8, j = blk / 8;
        blk = x * q + min(x, r) + j;
    }
    // wv is the same in all lanes; readfirstlane tells the compiler so, which
    // keeps the slice loop and the per-slice array bases in scalar registers
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t first = ((int64_t)blk * (kBlock / 64) + wv) * kSlices;
    // the run still open at the end of the previous slice: its tet (wave-uniform)
    // and its sums, parked in LDS by lane 63 (6 path integrals, 4 barycentrics)
    __shared__ double s_carry[kBlock / 64][10];
    __shared__ double2 s_sum[kBlock / 64][64 * 3];
    int carry_T = -1;
    // kPipe: the next slice's tet and state are requested before this slice's
    // tet rows, so that the rows' round trip overlaps those loads
    int nT = -1;
    double nl1 = 0.0, nl2 = 0.0, nl3 = 0.0;
    uint32_t nu1 = 0, nu2 = 0, nu3 = 0;
    Real nv0 = 0, nv1 = 0, nv2 = 0;
    auto fetch = [&](int64_t sl) {
        const int64_t bb = sl * 64;
        unsigned lq = lane;
        asm volatile("" : "+v"(lq));
        __builtin_assume(lq < 64u);
        nT = -1;
        if (bb + lq < a.n) {
            nT = __builtin_nontemporal_load(lane_at(a.tet + bb, lq));
            if (kFixed) {
                nu1 = __builtin_nontemporal_load(lane_at(reinterpret_cast<uint32_t *>(a.lam1) + bb, lq));
                nu2 = __builtin_nontemporal_load(lane_at(reinterpret_cast<uint32_t *>(a.lam2) + bb, lq));
                nu3 = __builtin_nontemporal_load(lane_at(reinterpret_cast<uint32_t *>(a.lam3) + bb, lq));
            } else {
                nl1 = __builtin_nontemporal_load(lane_at(a.lam1 + bb, lq));
                nl2 = __builtin_nontemporal_load(lane_at(a.lam2 + bb, lq));
                nl3 = __builtin_nontemporal_load(lane_at(a.lam3 + bb, lq));
            }
            nv0 = __builtin_nontemporal_load(lane_at(a.v0 + bb, lq));
            nv1 = __builtin_nontemporal_load(lane_at(a.v1 + bb, lq));
            nv2 = __builtin_nontemporal_load(lane_at(a.v2 + bb, lq));
        }
    };
    if (kPipe) fetch(first);
#pragma unroll 1
    for (int it = 0; it < kSlices; ++it) {
        const int64_t slice = first + it;
        if (slice * 64 >= a.n) break;
        // per-slice bases are wave-uniform: every array is addressed as a
        // scalar base plus the lane offset; the lane index is re-materialised in
        // every slice, so that the compiler does not keep per-lane addresses
        // alive across the loop.  The particle state is streamed with
        // non-temporal loads and stores, which leaves the caches to the per-tet
        // rows, the field DoFs and the current accumulator.
        const int64_t b0 = slice * 64;
        unsigned ln = lane;
        asm volatile("" : "+v"(ln));
        __builtin_assume(ln < 64u);
        const int64_t p = b0 + ln;
        double *__restrict__ lam1 = a.lam1 + b0, *__restrict__ lam2 = a.lam2 + b0, *__restrict__ lam3 = a.lam3 + b0;
        Real *__restrict__ v0 = a.v0 + b0, *__restrict__ v1 = a.v1 + b0, *__restrict__ v2 = a.v2 + b0;
        int32_t *__restrict__ tetp = a.tet + b0;
        // With one slice per wavefront the whole particle state is requested at
        // once, before the tet index is back: one HBM round trip instead of tet,
        // then barycentrics and rows, then velocities (the compiler issues them in
        // that order when they sit behind the tet test).  The sliced forms keep
        // the later loads: the extra live registers cost them more than the
        // round trip (measured on both).
        constexpr bool kEarly = kSlices == 1 || kPipe;
        constexpr bool kSlots = kPipe || push_uses_slots<Real>(kSlices);
        // the compact mixed form: barycentrics stored as uint32 fixed point
        constexpr bool fx = kFixed;
        uint32_t *__restrict__ f1 = reinterpret_cast<uint32_t *>(a.lam1) + b0;
        uint32_t *__restrict__ f2 = reinterpret_cast<uint32_t *>(a.lam2) + b0;
        uint32_t *__restrict__ f3 = reinterpret_cast<uint32_t *>(a.lam3) + b0;
        int T = -1;
        double sl1 = 0.0, sl2 = 0.0, sl3 = 0.0;
        uint32_t su1 = 0, su2 = 0, su3 = 0;
        Real sv0 = 0, sv1 = 0, sv2 = 0;
        auto load_state = [&]() {
            if (fx) {
                su1 = __builtin_nontemporal_load(lane_at(f1, ln));
                su2 = __builtin_nontemporal_load(lane_at(f2, ln));
                su3 = __builtin_nontemporal_load(lane_at(f3, ln));
            } else {
                sl1 = __builtin_nontemporal_load(lane_at(lam1, ln));
                sl2 = __builtin_nontemporal_load(lane_at(lam2, ln));
                sl3 = __builtin_nontemporal_load(lane_at(lam3, ln));
            }
            sv0 = __builtin_nontemporal_load(lane_at(v0, ln));
            sv1 = __builtin_nontemporal_load(lane_at(v1, ln));
            sv2 = __builtin_nontemporal_load(lane_at(v2, ln));
        };
        if (kPipe) {
            T = nT;
            sl1 = nl1;
            sl2 = nl2;
            sl3 = nl3;
            su1 = nu1;
            su2 = nu2;
            su3 = nu3;
            sv0 = nv0;
            sv1 = nv1;
            sv2 = nv2;
            if (it + 1 < kSlices) fetch(slice + 1);
        }
        if (p < a.n) {
            if (!kPipe) {
                T = __builtin_nontemporal_load(lane_at(tetp, ln));
                if (kEarly) load_state();
            }
            if ((unsigned)T >= (unsigned)a.nt) {
                atomicOr(a.status, (unsigned)ETPIC_DEV_BADTET);
                T = -1;
            }
        }
        const bool act = T >= 0;
        // scatter form: this lane's sorted position, from one cursor atomic
        // per run of equal tet (the lanes of a run keep their order)
        unsigned dq = 0;
        if (kScatter) {
            const WaveRuns r = wave_runs(T, ln);
            unsigned base = 0;
            if (r.head && act) base = atomicAdd(&a.cursor[T], (unsigned)(r.run_end - r.lane + 1));
            base = __shfl(base, r.head_lane);
            dq = base + (unsigned)(r.lane - r.head_lane);
        }
        double g6[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};   // this lane's in-tet path integrals
        double r4[4] = {0.0, 0.0, 0.0, 0.0};             // this lane's end-point barycentrics
        int walker = 0;
        if (act) {
            double l[4];
            if (!kEarly) load_state();
            if (fx) {
                sl1 = fix_to_real(su1);
                sl2 = fix_to_real(su2);
                sl3 = fix_to_real(su3);
            }
            l[1] = sl1;
            l[2] = sl2;
            l[3] = sl3;
            l[0] = 1.0 - l[1] - l[2] - l[3];
            Real v[3] = {sv0, sv1, sv2};
            const Real x[3] = {(Real)l[1], (Real)l[2], (Real)l[3]};
            gather_boris(a.coef + (int64_t)T * CoefRow<Real>::kStride, a.geo + (int64_t)T * GeoRow<Real>::kStride, x,
                         a.h, v);
            double dl[4], end[4];
            const bool stays = increments(a.gpush + (int64_t)T * PushRow<Real>::kStride, v, a.dt_r, 1.0, l, dl, end);
            if (!stays && !(isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2])))
                atomicOr(a.status, (unsigned)ETPIC_DEV_NAN);
            if (stays) {
                // compact form: the end point rounded to the fixed-point grid, and
                // the piece taken to that point, so that deposit and stored end
                // point agree exactly (the differences are exact in float64)
                uint32_t un[3] = {0, 0, 0};
                if (fx) {
                    fix_round3(l[1] + dl[1], l[2] + dl[2], l[3] + dl[3], un);
                    dl[1] = ((double)un[0] - (double)su1) * kFix;
                    dl[2] = ((double)un[1] - (double)su2) * kFix;
                    dl[3] = ((double)un[2] - (double)su3) * kFix;
                    end[1] = l[1] + dl[1];
                    end[2] = l[2] + dl[2];
                    end[3] = l[3] + dl[3];
                }
                // path integrals of the six W1_ij along the straight piece
                // (edge_sums): deposit and stored end point see the same
                // increments (continuity to float64 rounding)
                const double ps[6] = {dl[1], dl[2], dl[3], fma(l[1], dl[2], -(l[2] * dl[1])),
                                      fma(l[1], dl[3], -(l[3] * dl[1])), fma(l[2], dl[3], -(l[3] * dl[2]))};
                edge_sums(ps, g6);
#pragma unroll
                for (int k = 1; k < 4; ++k) l[k] = end[k];
                if (kScatter) {
                    if (fx) {
                        __builtin_nontemporal_store(un[0], reinterpret_cast<uint32_t *>(a.o_lam1) + dq);
                        __builtin_nontemporal_store(un[1], reinterpret_cast<uint32_t *>(a.o_lam2) + dq);
                        __builtin_nontemporal_store(un[2], reinterpret_cast<uint32_t *>(a.o_lam3) + dq);
                    } else {
                        __builtin_nontemporal_store(l[1], &a.o_lam1[dq]);
                        __builtin_nontemporal_store(l[2], &a.o_lam2[dq]);
                        __builtin_nontemporal_store(l[3], &a.o_lam3[dq]);
                    }
                    a.o_tet[dq] = T;
                } else if (fx) {
                    __builtin_nontemporal_store(un[0], lane_at(f1, ln));
                    __builtin_nontemporal_store(un[1], lane_at(f2, ln));
                    __builtin_nontemporal_store(un[2], lane_at(f3, ln));
                } else {
                    __builtin_nontemporal_store(l[1], lane_at(lam1, ln));
                    __builtin_nontemporal_store(l[2], lane_at(lam2, ln));
                    __builtin_nontemporal_store(l[3], lane_at(lam3, ln));
                }
                if (kRho) {
                    r4[0] = 1.0 - l[1] - l[2] - l[3];
                    r4[1] = l[1];
                    r4[2] = l[2];
                    r4[3] = l[3];
                }
            } else if (kScatter) {
                // the walk starts from the old barycentrics at the new position
                if (fx) {
                    reinterpret_cast<uint32_t *>(a.o_lam1)[dq] = su1;
                    reinterpret_cast<uint32_t *>(a.o_lam2)[dq] = su2;
                    reinterpret_cast<uint32_t *>(a.o_lam3)[dq] = su3;
                } else {
                    a.o_lam1[dq] = l[1];
                    a.o_lam2[dq] = l[2];
                    a.o_lam3[dq] = l[3];
                }
                a.o_tet[dq] = walker_mark(T);
                walker = 1;
            } else {
                *lane_at(tetp, ln) = walker_mark(T);
                walker = 1;
            }
            if (kScatter) {
                __builtin_nontemporal_store(v[0], &a.o_v0[dq]);
                __builtin_nontemporal_store(v[1], &a.o_v1[dq]);
                __builtin_nontemporal_store(v[2], &a.o_v2[dq]);
                if (a.id) __builtin_nontemporal_store(__builtin_nontemporal_load(&a.id[p]), &a.o_id[dq]);
            } else {
                __builtin_nontemporal_store(v[0], lane_at(v0, ln));
                __builtin_nontemporal_store(v[1], lane_at(v1, ln));
                __builtin_nontemporal_store(v[2], lane_at(v2, ln));
            }
        }
        const WaveRuns runs = wave_runs(T, ln);
        // the open run continues into this slice: lane 0 takes over its sums;
        // otherwise it is complete and flushed now
        if (kSlices > 1 && carry_T >= 0) {
            __builtin_amdgcn_wave_barrier();
            if (ln == 0) {
                double cg[6], cr[4];
#pragma unroll
                for (int e = 0; e < 6; ++e) cg[e] = s_carry[wv][e];
#pragma unroll
                for (int k = 0; k < 4; ++k) cr[k] = s_carry[wv][6 + k];
                if (T == carry_T) {
#pragma unroll
                    for (int e = 0; e < 6; ++e) g6[e] += cg[e];
#pragma unroll
                    for (int k = 0; k < 4; ++k) r4[k] += cr[k];
                } else {
                    flush_run<Real, kRho, kPipe || push_uses_slots<Real>(kSlices)>(a, carry_T, cg, cr);
                }
            }
        }
        // segmented reduction over runs of equal tet; the run's last lane holds
        // its sums and adds them to HBM, except for the run reaching lane 63,
        // which stays open for the next slice
#pragma unroll
        for (int e = 0; e < 6; ++e) g6[e] = run_total(g6[e], runs);
        if (kRho) {
#pragma unroll
            for (int k = 0; k < 4; ++k) r4[k] = run_total(r4[k], runs);
        }
        const bool last = it == kSlices - 1 || (slice + 1) * 64 >= a.n;
        const bool flush = act && runs.lane == runs.run_end && (ln != 63 || last);
        if (kRho) {
            if (flush) flush_run<Real, kRho, kSlots>(a, T, g6, r4);
        } else {
            flush_runs_together<Real, kSlots>(a, T, g6, runs, flush, s_sum[wv]);
        }
        if (!last) {
            carry_T = __builtin_amdgcn_readlane(T, 63);
            if (ln == 63) {
#pragma unroll
                for (int e = 0; e < 6; ++e) s_carry[wv][e] = g6[e];
#pragma unroll
                for (int k = 0; k < 4; ++k) s_carry[wv][6 + k] = r4[k];
            }
        }
        // walkers go to the particle queue (one atomic per wavefront); a
        // wavefront whose walkers do not all fit queues its slice instead
        const unsigned long long wmask = __ballot(walker);
        if (wmask) {
            const unsigned cnt = (unsigned)__popcll(wmask);
            unsigned base = 0;
            if (ln == 0) base = atomicAdd(&a.walk_ctr[0], cnt);
            base = __shfl(base, 0);
            const bool fits = (kScatter || !a.walk_by_slice) && base < kWalkQueueCap && cnt <= kWalkQueueCap - base;
            const unsigned rank = (unsigned)__popcll(wmask & ((1ull << ln) - 1ull));
            if (walker && base + rank < kWalkQueueCap)
                a.walk_queue[base + rank] = fits ? (kScatter ? dq : (unsigned)p) : kQueueSkip;
            // (after a scatter step the walkers of a slice are spread over the
            // output, so an overflow there makes the walk scan every particle)
            if (!kScatter && !fits && ln == 0) a.slice_queue[atomicAdd(&a.walk_ctr[2], 1u)] = (unsigned)slice;
        }
    }
}

// One slice per wavefront; without the vertex charge the kernel fits 64 VGPRs
// (8 wavefronts per SIMD), which the compiler does not choose by itself.
template <typename Real>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7))) k_push(StepArgs<Real> a, int remap) {
    push_slices<Real, 1, false>(a, remap);
}

template <typename Real>
__global__ void __launch_bounds__(kBlock) k_push_rho(StepArgs<Real> a, int remap) {
    push_slices<Real, 1, true>(a, remap);
}

// The particle kernel's HBM access pattern and nothing else, to measure the
// streaming rate that pattern can reach: the same launch shape (one lane per
// particle, 64-particle slices, XCD-contiguous block ranges), the same
// non-temporal loads of tet, lambda_1..3 and v and non-temporal stores of
// lambda_1..3 and v back in place.  Each stored value is the loaded one plus
// zero times the tet index (zero is a run-time argument), so the particle
// state is left as it was and no load can be dropped.
template <typename Real>
__global__ void __launch_bounds__(kBlock) k_stream(int64_t n, double *__restrict__ lam1, double *__restrict__ lam2,
                                                   double *__restrict__ lam3, Real *__restrict__ v0,
                                                   Real *__restrict__ v1, Real *__restrict__ v2,
                                                   const int32_t *__restrict__ tet, double zero, int remap, int fixed) {
    unsigned blk = blockIdx.x;
    if (remap) blk = xcd_block(blk, gridDim.x);
    const int64_t p = (int64_t)blk * kBlock + threadIdx.x;
    if (p >= n) return;
    const double z = zero * (double)__builtin_nontemporal_load(&tet[p]);
    const Real a = __builtin_nontemporal_load(&v0[p]), b = __builtin_nontemporal_load(&v1[p]),
               c = __builtin_nontemporal_load(&v2[p]);
    if (fixed) {
        uint32_t *u1 = reinterpret_cast<uint32_t *>(lam1), *u2 = reinterpret_cast<uint32_t *>(lam2),
                 *u3 = reinterpret_cast<uint32_t *>(lam3);
        const uint32_t zi = (uint32_t)z;
        const uint32_t k1 = __builtin_nontemporal_load(&u1[p]), k2 = __builtin_nontemporal_load(&u2[p]),
                       k3 = __builtin_nontemporal_load(&u3[p]);
        __builtin_nontemporal_store(k1 + zi, &u1[p]);
        __builtin_nontemporal_store(k2 + zi, &u2[p]);
        __builtin_nontemporal_store(k3 + zi, &u3[p]);
    } else {
        const double l1 = __builtin_nontemporal_load(&lam1[p]), l2 = __builtin_nontemporal_load(&lam2[p]),
                     l3 = __builtin_nontemporal_load(&lam3[p]);
        __builtin_nontemporal_store(l1 + z, &lam1[p]);
        __builtin_nontemporal_store(l2 + z, &lam2[p]);
        __builtin_nontemporal_store(l3 + z, &lam3[p]);
    }
    __builtin_nontemporal_store(a + (Real)z, &v0[p]);
    __builtin_nontemporal_store(b + (Real)z, &v1[p]);
    __builtin_nontemporal_store(c + (Real)z, &v2[p]);
}

template <typename Real, int kSlices, bool kRho>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7)))
k_push_slices(StepArgs<Real> a, int remap) {
    push_slices<Real, kSlices, kRho>(a, remap);
}

// The same kernels reading the particles in their old order and writing them,
// pushed, to their tet-sorted positions: the counting sort's scatter pass
// folded into the step.
template <typename Real, bool kRho>
__global__ void __launch_bounds__(kBlock) k_push_sort(StepArgs<Real> a, int remap) {
    push_slices<Real, 1, kRho, true>(a, remap);
}

template <typename Real, int kSlices, bool kRho>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7)))
k_push_sort_slices(StepArgs<Real> a, int remap) {
    push_slices<Real, kSlices, kRho, true>(a, remap);
}

// Two slices per wavefront with the second slice's state requested before the
// first one's tet rows are read (float forms; in float64 the form needs 80
// VGPRs, six wavefronts per SIMD, and measured no gain worth it).  Chosen where
// the mesh's float rows outgrow the Infinity Cache, so that a wavefront's row
// reads are HBM round trips: there the state loads of one slice overlap the
// row round trip of the other.  (At most 7 wavefronts: 8 leave the compact
// form too few registers, 1683 -> 1800 us for ten steps of 1e7.)
template <bool kFixed>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7)))
k_push_pipe(StepArgs<float> a, int remap) {
    push_slices<float, 2, false, false, kFixed, true>(a, remap);
}

// The compact mixed form (barycentrics stored as uint32 fixed point): the same
// kernels with that storage compiled in.
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7)))
k_push_fixed(StepArgs<float> a, int remap) {
    push_slices<float, 1, false, false, true>(a, remap);
}

__global__ void __launch_bounds__(kBlock) k_push_rho_fixed(StepArgs<float> a, int remap) {
    push_slices<float, 1, true, false, true>(a, remap);
}

template <int kSlices, bool kRho>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7)))
k_push_slices_fixed(StepArgs<float> a, int remap) {
    push_slices<float, kSlices, kRho, false, true>(a, remap);
}

template <bool kRho>
__global__ void __launch_bounds__(kBlock) k_push_sort_fixed(StepArgs<float> a, int remap) {
    push_slices<float, 1, kRho, true, true>(a, remap);
}

template <int kSlices, bool kRho>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7)))
k_push_sort_slices_fixed(StepArgs<float> a, int remap) {
    push_slices<float, kSlices, kRho, true, true>(a, remap);
}

// Walk of one marked particle p: every piece of its path is deposited with
// global atomics, and the end point, reflected velocity and new tet are stored.
template <typename Real>
__device__ __forceinline__ void walk_particle(const StepArgs<Real> &a, int64_t p) {
    const int marked = a.tet[p];
    if (marked > -2) return;
    int T = walker_tet(marked);
    if (T >= a.nt) return;
    const bool fx = std::is_same<Real, float>::value && a.fixed;
    uint32_t *fl[3] = {reinterpret_cast<uint32_t *>(a.lam1), reinterpret_cast<uint32_t *>(a.lam2),
                       reinterpret_cast<uint32_t *>(a.lam3)};
    double l[4];
    if (fx) {
        l[1] = fix_to_real(fl[0][p]);
        l[2] = fix_to_real(fl[1][p]);
        l[3] = fix_to_real(fl[2][p]);
    } else {
        l[1] = a.lam1[p];
        l[2] = a.lam2[p];
        l[3] = a.lam3[p];
    }
    l[0] = 1.0 - l[1] - l[2] - l[3];
    Real v[3] = {a.v0[p], a.v1[p], a.v2[p]};
    const Real dx[3] = {a.dt_r * v[0], a.dt_r * v[1], a.dt_r * v[2]};
    double d[3] = {(double)dx[0], (double)dx[1], (double)dx[2]};
    T = walk<Real, false>(a, T, l, d, v, nullptr, nullptr, fx);
    a.tet[p] = T;
    if (fx) {
        // the walk ended on the fixed-point grid (rounding leaves such a point
        // as it is; a walk stopped at the hop cap is rounded onto the grid)
        uint32_t u[3];
        fix_round3(l[1], l[2], l[3], u);
        fl[0][p] = u[0];
        fl[1][p] = u[1];
        fl[2][p] = u[2];
    } else {
        a.lam1[p] = l[1];
        a.lam2[p] = l[2];
        a.lam3[p] = l[3];
    }
    a.v0[p] = v[0];
    a.v1[p] = v[1];
    a.v2[p] = v[2];
    if (a.rho) {
        const TetTopo tp = a.topo[T];
        const double l0 = 1.0 - l[1] - l[2] - l[3];
        unsafeAtomicAdd(&a.rho[tp.v[0]], a.qw * l0);
        unsafeAtomicAdd(&a.rho[tp.v[1]], a.qw * l[1]);
        unsafeAtomicAdd(&a.rho[tp.v[2]], a.qw * l[2]);
        unsafeAtomicAdd(&a.rho[tp.v[3]], a.qw * l[3]);
    }
}

// Walks the queued particles, one lane each, then the particles of the
// overflow slices, one wavefront per slice.  The last block to finish resets
// the counters for the next step.
template <typename Real, typename WalkOne>
__device__ __forceinline__ void walk_queued(const StepArgs<Real> &a, unsigned blk, unsigned nblk, WalkOne walk_one) {
    const unsigned total = __atomic_load_n(&a.walk_ctr[0], __ATOMIC_RELAXED);
    if (a.scatter && (a.walk_by_slice || total > kWalkQueueCap)) {
        // after a scatter step whose walkers did not all fit in the queue:
        // every marked particle, found by a scan (one lane per particle)
        for (int64_t p = (int64_t)blk * kBlock + threadIdx.x; p < a.n; p += (int64_t)nblk * kBlock)
            walk_one(p);
    } else {
        const unsigned count = min(total, kWalkQueueCap);
        for (unsigned i = blk * kBlock + threadIdx.x; i < count; i += nblk * kBlock) {
            const unsigned q = a.walk_queue[i];
            if (q != kQueueSkip && (int64_t)q < a.n) walk_one((int64_t)q);
        }
        const unsigned slices = __atomic_load_n(&a.walk_ctr[2], __ATOMIC_RELAXED);
        const unsigned wpb = kBlock / 64;
        for (unsigned i = blk * wpb + (threadIdx.x >> 6); i < slices; i += nblk * wpb) {
            const int64_t p = (int64_t)a.slice_queue[i] * 64 + (threadIdx.x & 63);
            if (p < a.n) walk_one(p);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        if (atomicAdd(&a.walk_ctr[1], 1u) == nblk - 1) {
            a.walk_ctr[0] = 0u;
            a.walk_ctr[1] = 0u;
            a.walk_ctr[2] = 0u;
        }
    }
}

template <typename Real>
__global__ void __launch_bounds__(kBlock) k_walk(StepArgs<Real> a) {
    walk_queued(a, blockIdx.x, gridDim.x, [&](int64_t p) { walk_particle(a, p); });
}

// The walk of one step and the coefficient pass of the next in one launch, for
// calls of several steps that go one step per launch: blocks [0, kWalkBlocks)
// walk, the others build the next step's rows.  The walk does not read the
// rows and the pass reads nothing the walk writes, so the short, latency-bound
// walk hides behind it (ten steps of 1e7, one slice forced: float64
// 2844 -> 2777 us, mixed 2130 -> 2035, compact 1757 -> 1666).
template <typename Real, int kSnap>
__global__ void __launch_bounds__(kBlock) k_walk_coef(StepArgs<Real> a, int64_t nt, const double *prow,
                                                      const int32_t *tetface, FieldPtrs F) {
    if (blockIdx.x < kWalkBlocks) {
        walk_queued(a, blockIdx.x, kWalkBlocks, [&](int64_t p) { walk_particle(a, p); });
    } else {
        const unsigned blk = blockIdx.x - kWalkBlocks;
        tet_coef<Real, kSnap, kCoefStep>(nt, prow, tetface, F, const_cast<Real *>(a.coef), nullptr,
                                         F.xcd ? xcd_block(blk, gridDim.x - kWalkBlocks) : blk);
    }
}

// ------------------------------------------------------------------ several steps per launch
// Within one call the fields are known for every step and the particles do not
// act on each other, so a launch can take each particle through several steps
// while its state stays in registers: the state crosses HBM once per launch
// instead of once per step, and the segmented reduction and the flush of the
// path integrals, a third of a single step's instructions, run once per launch
// on sums over its steps.  What is left per step is the arithmetic of the push
// itself.  Measured, ten steps and their re-sort in one call, 40^3 x 6 tets,
// against one step per launch: 1e7 float64 2.90 -> 0.65 ms, 5e7 mixed 9.64 ->
// 2.27 ms, 1e7 compact 1.99 -> 0.60 ms; the 100 steps of 1,000 electrons on
// 750 tets 1.14 -> 0.14 ms.
//
// The rows of each step come from the parts of the tet's row (real, imaginary,
// dc, built once per call by the coefficient pass).  A wavefront stages the
// parts of its tets in LDS; before each step its 64 lanes together form the
// 10 entries of every such tet's row, two fma each, and every lane reads its
// tet's row back (lanes of a run read one address).  Per-lane rows from
// memory instead would cost 30 float64 loads and 20 fma per lane and step.
// kRuns tets are staged at a time; a wavefront with more runs of equal tet
// takes them in passes, each pass running all the steps of its lanes.
//
// A particle that leaves its tet at step j stops there (its start point of
// that step, its new velocity and j are kept: tet = -(T + j nt + 2)) and is
// queued; k_walk_multi walks it and takes it through the remaining steps.
//
// A launch takes up to 16 steps, of few particles up to 32: there the launch
// itself and the walk after it are the larger part (100 steps in 7 launches
// and in 4: 1,000 electrons on 750 tets 199 and 182 us a call, 32,768 207 and
// 170, 32,768 on 83,000 tets 278 and 221; 50,000 and 400,000 electrons, left
// at 16, would gain 13 to 16 % too where few leave their tet).  The more steps in one
// launch, the more of many particles finish it in the walk, one lane each.
constexpr int kMaxFused = 32, kMaxFusedMany = 16;
// per tet: the largest of the coefficient forms but the parts of three
// snapshots, which go to the wide rows (etpic_ds_rows_bind) where those are bound
constexpr int kCoefDoubles = kRowParts<1> * kRowReals;

template <int kSnap>
struct MultiArgs {
    const double *parts;   // nt rows of kRowParts<kSnap> * 10 float64
    int nsteps;            // steps of this launch
    int width;             // particles per wavefront (64, or fewer where wavefronts are few)
    double wc[kMaxFused + 1][kSnap], ws[kMaxFused + 1][kSnap];   // step weights; one more than any step reads
};

__device__ __forceinline__ int leaver_mark(int T, int j, int64_t nt) { return -(T + j * (int)nt + 2); }

// The multi-step kernels keep the barycentrics in units of 1 / kOne: 1, or
// 2^32 in the compact form, whose stored numbers are then whole doubles and
// every step's scalings by 2^32 drop out (the geometry and gradient rows take
// them once per launch; a power of two changes no rounding).
template <bool kFixed>
constexpr double kOne = kFixed ? kFixScale : 1.0;

// A tet's geometry and gradient rows in those units.
template <typename Real, bool kFixed>
__device__ __forceinline__ void load_rows(const StepArgs<Real> &a, int T, Real gm[9], Real gr[9]) {
    const Real *gmp = a.geo + (int64_t)T * GeoRow<Real>::kStride;
    const Real *grp = a.gpush + (int64_t)T * PushRow<Real>::kStride;
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        gm[k] = kFixed ? gmp[k] * (Real)kFix : gmp[k];
        gr[k] = kFixed ? grp[k] * (Real)kFixScale : grp[k];
    }
}

// One in-tet step's contribution to those sums, and the new barycentrics; in
// the compact form the end point goes to the fixed-point grid first (as
// fix_round3) and the piece runs to it.
template <bool kFixed>
__device__ __forceinline__ void stay_step(double l[4], double dl[4], double t[4], double s[6]) {
    if (kFixed) {
#pragma unroll
        for (int k = 1; k < 4; ++k) t[k] = fmin(rint(t[k]), kFixScale - 1.0);
        if (t[1] + t[2] + t[3] > kFixScale) {
            uint32_t un[3];
            fix_round3(t[1] * kFix, t[2] * kFix, t[3] * kFix, un);
#pragma unroll
            for (int k = 1; k < 4; ++k) t[k] = (double)un[k - 1];
        }
#pragma unroll
        for (int k = 1; k < 4; ++k) dl[k] = t[k] - l[k];
    }
    s[0] += dl[1];
    s[1] += dl[2];
    s[2] += dl[3];
    s[3] = fma(l[1], dl[2], fma(-l[2], dl[1], s[3]));
    s[4] = fma(l[1], dl[3], fma(-l[3], dl[1], s[4]));
    s[5] = fma(l[2], dl[3], fma(-l[3], dl[2], s[5]));
#pragma unroll
    for (int k = 1; k < 4; ++k) l[k] = t[k];
}

// The sums in barycentric units.
template <bool kFixed>
__device__ __forceinline__ void unscale_sums(double s[6]) {
    if (kFixed)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            s[k] *= kFix;
            s[3 + k] *= kFix * kFix;
        }
}

// The leaver queue of the multi-step kernels: kShards parts of walk_queue, each
// with its own length on a line of its own; kShardRun consecutive blocks of
// particles share a part (their leavers then share tets and lines in the walk).  (One length for all had the wavefronts of a dense bunch,
// most of which hold a leaver, wait for one address: 1e8 particles 9.4 ms per
// launch, 6.7 ms without that wait.)  Counters of one set: [1] a scatter
// launch overflowed, [2] slice_queue length, [kShardAt + kShardStride i] the
// length of part i.
constexpr unsigned kShards = 64, kShardRun = 32, kShardCap = kWalkQueueCap / kShards, kShardAt = 32, kShardStride = 32;
static_assert(kShardAt + kShards * kShardStride <= kCtrStride, "a counter set holds its shards");

// Queues the lanes of wmask (entry: this lane's).  False if they did not all
// fit (or `allowed` is not set): none is queued then.
template <typename Real>
__device__ __forceinline__ bool queue_leavers(const StepArgs<Real> &a, unsigned long long wmask, bool left,
                                              unsigned entry, bool allowed, unsigned blk) {
    const unsigned ln = threadIdx.x & 63, cnt = (unsigned)__popcll(wmask), shard = blk / kShardRun % kShards;
    unsigned base = 0;
    if (ln == 0) base = atomicAdd(&a.walk_ctr[kShardAt + shard * kShardStride], cnt);
    base = __shfl(base, 0);
    const bool fits = allowed && base < kShardCap && cnt <= kShardCap - base;
    const unsigned at = base + (unsigned)__popcll(wmask & ((1ull << ln) - 1ull));
    if (left && at < kShardCap) a.walk_queue[shard * kShardCap + at] = fits ? entry : kQueueSkip;
    return fits;
}

// Takes the queued particles, one lane each (block b a share of part b % kShards),
// then those of the overflow slices, one wavefront per slice; after a scatter
// launch whose leavers did not all fit, every marked particle, by a scan.
template <typename Real, typename TakeOne>
__device__ __forceinline__ void take_leavers(const StepArgs<Real> &a, TakeOne take_one) {
    const unsigned blk = blockIdx.x, nblk = gridDim.x;
    if (a.scatter && (a.walk_by_slice || __atomic_load_n(&a.walk_ctr[1], __ATOMIC_RELAXED))) {
        for (int64_t p = (int64_t)blk * kBlock + threadIdx.x; p < a.n; p += (int64_t)nblk * kBlock) take_one(p);
        return;
    }
    const unsigned shard = blk % kShards, per = nblk / kShards, part = blk / kShards;
    const unsigned count = min(__atomic_load_n(&a.walk_ctr[kShardAt + shard * kShardStride], __ATOMIC_RELAXED), kShardCap);
    const unsigned to = (unsigned)((uint64_t)count * (part + 1) / per);
    for (unsigned i = (unsigned)((uint64_t)count * part / per) + threadIdx.x; i < to; i += kBlock) {
        const unsigned q = a.walk_queue[shard * kShardCap + i];
        if (q != kQueueSkip && (int64_t)q < a.n) take_one((int64_t)q);
    }
    const unsigned slices = __atomic_load_n(&a.walk_ctr[2], __ATOMIC_RELAXED);
    const unsigned wpb = kBlock / 64;
    for (unsigned i = blk * wpb + (threadIdx.x >> 6); i < slices; i += nblk * wpb) {
        const int64_t p = (int64_t)a.slice_queue[i] * 64 + (threadIdx.x & 63);
        if (p < a.n) take_one(p);
    }
}

// Clears a counter set (by one block).
__device__ __forceinline__ void clear_counters(unsigned *ctr) {
    if (threadIdx.x < 3) ctr[threadIdx.x] = 0u;
    for (unsigned i = threadIdx.x; i < kShards; i += blockDim.x) ctr[kShardAt + i * kShardStride] = 0u;
}

// The row parts of a wavefront's nr tets into LDS, part[q * kEnt + 10 j + c]:
// half a wavefront loads the row of one tet (its 30 or 70 reals in one or
// three lots), two lots of tets in flight; a lane's place in the row is fixed,
// so that a tet costs a few instructions.
template <int kParts, int kEnt>
__device__ __forceinline__ void stage_parts(const double *__restrict__ parts, const int *tets, int nr, int ln,
                                            double *part) {
    constexpr int kLen = kParts * kRowReals, kLots = (kLen + 31) / 32;
    const int half = ln >> 5;
#pragma unroll
    for (int lot = 0; lot < kLots; ++lot) {
        const int e = 32 * lot + (ln & 31), q = e / kRowReals;
        if (e < kLen) {
            double *dst = part + q * kEnt + (e - q * kRowReals);
#pragma unroll 1
            for (int j = half; j < nr; j += 4) {
                const int k = min(j + 2, nr - 1);
                const double x = parts[(int64_t)max(tets[j], 0) * kLen + e];
                const double y = parts[(int64_t)max(tets[k], 0) * kLen + e];
                dst[j * kRowReals] = x;
                dst[k * kRowReals] = y;
            }
        }
    }
}

template <typename Real, int kSnap, bool kRho, bool kScatter, bool kFixed>
__global__ void __launch_bounds__(kBlock) k_push_multi(StepArgs<Real> a, MultiArgs<kSnap> ma, int remap) {
    constexpr int kParts = kRowParts<kSnap>;
    constexpr int kRuns = kSnap == 1 ? 16 : 8;
    constexpr int kEnt = kRuns * kRowReals;     // row entries staged per wavefront
    constexpr int kWaves = kBlock / 64;
    constexpr int kRowBytes = kEnt * (int)sizeof(Real);
    constexpr int kLds = kParts * kEnt * 8 + 2 * kRowBytes + 64 * 4;   // per wavefront
    static_assert(kParts * kEnt * 8 >= 64 * 3 * 16, "the flush buffer shares the parts' space");
    __shared__ __align__(16) char s_lds[kWaves][kLds];
    unsigned blk = blockIdx.x;
    if (remap) blk = xcd_block(blk, gridDim.x);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned ln = threadIdx.x & 63;
    double *part = reinterpret_cast<double *>(s_lds[wv]);
    Real *rows = reinterpret_cast<Real *>(s_lds[wv] + kParts * kEnt * 8);
    int *s_tet = reinterpret_cast<int *>(s_lds[wv] + kParts * kEnt * 8 + 2 * kRowBytes);
    const int64_t b0 = ((int64_t)blk * kWaves + wv) * ma.width;
    if (b0 >= a.n) return;   // the whole wavefront; no block barrier below
    const int64_t p = b0 + ln;
    int T = -1, stored = -1;
    double l[4] = {0.0, 0.0, 0.0, 0.0};   // l[0] unused: lam0 is implicit
    uint32_t u[3] = {0, 0, 0};
    Real v[3] = {0, 0, 0};
    int64_t id = 0;
    const bool here = p < a.n && (int)ln < ma.width;
    if (here) {
        T = stored = __builtin_nontemporal_load(lane_at(a.tet + b0, ln));
        if (kFixed) {
            u[0] = __builtin_nontemporal_load(lane_at(reinterpret_cast<uint32_t *>(a.lam1) + b0, ln));
            u[1] = __builtin_nontemporal_load(lane_at(reinterpret_cast<uint32_t *>(a.lam2) + b0, ln));
            u[2] = __builtin_nontemporal_load(lane_at(reinterpret_cast<uint32_t *>(a.lam3) + b0, ln));
        } else {
            l[1] = __builtin_nontemporal_load(lane_at(a.lam1 + b0, ln));
            l[2] = __builtin_nontemporal_load(lane_at(a.lam2 + b0, ln));
            l[3] = __builtin_nontemporal_load(lane_at(a.lam3 + b0, ln));
        }
        v[0] = __builtin_nontemporal_load(lane_at(a.v0 + b0, ln));
        v[1] = __builtin_nontemporal_load(lane_at(a.v1 + b0, ln));
        v[2] = __builtin_nontemporal_load(lane_at(a.v2 + b0, ln));
        if (kScatter && a.id) id = __builtin_nontemporal_load(&a.id[p]);
        if ((unsigned)T >= (unsigned)a.nt) {
            atomicOr(a.status, (unsigned)ETPIC_DEV_BADTET);
            T = -1;
        }
    }
    if (kFixed) {
#pragma unroll
        for (int k = 0; k < 3; ++k) l[k + 1] = (double)u[k];
    }
    const bool act = T >= 0;
    const WaveRuns runs = wave_runs(T, ln);
    // scatter form: the sorted position, one cursor atomic per run; without
    // cursors the particles keep their places in the other arrays
    // (requested here, with the particle's id, and taken up after the steps)
    unsigned base = 0;
    if (kScatter && a.cursor && runs.head && act)
        base = atomicAdd(&a.cursor[T], (unsigned)(runs.run_end - runs.lane + 1));
    const unsigned long long heads = __ballot(runs.head);
    const int nruns = __popcll(heads);
    const int run = __popcll(heads & (ln == 63 ? ~0ull : ((2ull << ln) - 1ull))) - 1;
    if (runs.head) s_tet[run] = T;
    Real gm[9], gr[9];
    load_rows<Real, kFixed>(a, max(T, 0), gm, gr);
    double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int leave = -1;   // step at which the particle left its tet
#pragma unroll 1
    for (int r0 = 0; r0 < nruns; r0 += kRuns) {
        const int nr = min(kRuns, nruns - r0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        stage_parts<kParts, kEnt>(ma.parts, s_tet + r0, nr, ln, part);
        bool live = act && run >= r0 && run < r0 + nr;
        const Real *cf = rows + (live ? (run - r0) * kRowReals : 0);
        // the rows of step j + 1 are formed while step j's arithmetic runs
        // (two row buffers), and its weights are read a step ahead of that
        double wc[kSnap], ws[kSnap];
        auto weights = [&](int j) {
#pragma unroll
            for (int k = 0; k < kSnap; ++k) {
                wc[k] = ma.wc[j][k];
                ws[k] = ma.ws[j][k];
            }
        };
        // this lane's entry of the first 64 keeps its parts in registers
        const int entries = nr * kRowReals;
        double mine[kParts];
        auto form_rows = [&](Real *row) {
            if ((int)ln < entries) row[ln] = (Real)row_entry<kSnap>(mine, 1, wc, ws);
            for (int e = ln + 64; e < entries; e += 64) row[e] = (Real)row_entry<kSnap>(part + e, kEnt, wc, ws);
        };
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int q = 0; q < kParts; ++q) mine[q] = part[q * kEnt + ln];
        weights(0);
        form_rows(rows);
        weights(1);
        int odd = 0;
#pragma unroll 1
        for (int j = 0; j < ma.nsteps; ++j) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const Real *cj = cf + odd;
            odd = kEnt - odd;
            if (j + 1 < ma.nsteps) {
                form_rows(rows + odd);
                weights(j + 2 <= kMaxFused ? j + 2 : kMaxFused);
            }
            if (live) {
                const Real x[3] = {(Real)l[1], (Real)l[2], (Real)l[3]};
                gather_boris(cj, gm, x, a.h, v);
                double dl[4], t[4];
                if (increments(gr, v, a.dt_r, kOne<kFixed>, l, dl, t)) {
                    stay_step<kFixed>(l, dl, t, s);
                } else {
                    if (!(isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2])))
                        atomicOr(a.status, (unsigned)ETPIC_DEV_NAN);
                    leave = j;
                    live = false;
                }
            }
            if (!__builtin_amdgcn_ballot_w64(live)) break;
        }
    }
    unscale_sums<kFixed>(s);
    if (kFixed) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            u[k] = (uint32_t)l[k + 1];
            l[k + 1] *= kFix;
        }
    }
    const bool left = leave >= 0;
    unsigned dq = (unsigned)p;
    if (kScatter && a.cursor) dq = __shfl(base, runs.head_lane) + (unsigned)(runs.lane - runs.head_lane);
    // (a particle without a valid tet has no sorted place; one that keeps its
    // place is copied as it is)
    if (act || (kScatter && !a.cursor && here)) {
        const int64_t q = kScatter ? (int64_t)dq : p;
        if (kScatter) {
            if (kFixed) {
                __builtin_nontemporal_store(u[0], reinterpret_cast<uint32_t *>(a.o_lam1) + q);
                __builtin_nontemporal_store(u[1], reinterpret_cast<uint32_t *>(a.o_lam2) + q);
                __builtin_nontemporal_store(u[2], reinterpret_cast<uint32_t *>(a.o_lam3) + q);
            } else {
                __builtin_nontemporal_store(l[1], &a.o_lam1[q]);
                __builtin_nontemporal_store(l[2], &a.o_lam2[q]);
                __builtin_nontemporal_store(l[3], &a.o_lam3[q]);
            }
            __builtin_nontemporal_store(v[0], &a.o_v0[q]);
            __builtin_nontemporal_store(v[1], &a.o_v1[q]);
            __builtin_nontemporal_store(v[2], &a.o_v2[q]);
            a.o_tet[q] = left ? leaver_mark(T, leave, a.nt) : stored;
            if (a.id) __builtin_nontemporal_store(id, &a.o_id[q]);
        } else {
            if (kFixed) {
                __builtin_nontemporal_store(u[0], lane_at(reinterpret_cast<uint32_t *>(a.lam1) + b0, ln));
                __builtin_nontemporal_store(u[1], lane_at(reinterpret_cast<uint32_t *>(a.lam2) + b0, ln));
                __builtin_nontemporal_store(u[2], lane_at(reinterpret_cast<uint32_t *>(a.lam3) + b0, ln));
            } else {
                __builtin_nontemporal_store(l[1], lane_at(a.lam1 + b0, ln));
                __builtin_nontemporal_store(l[2], lane_at(a.lam2 + b0, ln));
                __builtin_nontemporal_store(l[3], lane_at(a.lam3 + b0, ln));
            }
            __builtin_nontemporal_store(v[0], lane_at(a.v0 + b0, ln));
            __builtin_nontemporal_store(v[1], lane_at(a.v1 + b0, ln));
            __builtin_nontemporal_store(v[2], lane_at(a.v2 + b0, ln));
            if (left) *lane_at(a.tet + b0, ln) = leaver_mark(T, leave, a.nt);
        }
    }
#pragma unroll
    for (int e = 0; e < 6; ++e) s[e] = run_total(s[e], runs);
    double g6[6];
    edge_sums(s, g6);
    const bool flush = act && runs.lane == runs.run_end;
    flush_runs_together<Real, true>(a, T, g6, runs, flush, reinterpret_cast<double2 *>(part));
    if (kRho) {
        double r4[4];
#pragma unroll
        for (int k = 1; k < 4; ++k) r4[k] = run_total(act && !left ? l[k] : 0.0, runs);
        // lam_0 sums to the number of the run's particles that stayed less the rest
        const unsigned long long stayed = __ballot(act && !left);
        const unsigned long long upto = ln == 63 ? ~0ull : ((2ull << ln) - 1ull);
        r4[0] = (double)__popcll(stayed & upto & ~((1ull << runs.head_lane) - 1ull)) - r4[1] - r4[2] - r4[3];
        if (flush) {
            const int32_t *tv = a.topo[T].v;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (r4[k] != 0.0) unsafeAtomicAdd(&a.rho[tv[k]], a.qw * r4[k]);
        }
    }
    // leavers to the particle queue, or (in place) their slice when it is full
    const unsigned long long wmask = __ballot(left);
    if (wmask) {
        const bool fits = queue_leavers(a, wmask, left, kScatter ? dq : (unsigned)p, kScatter || !a.walk_by_slice, blk);
        if (!fits && ln == 0) {
            if (kScatter)
                atomicOr(&a.walk_ctr[1], 1u);   // (the slice's particles are spread over the output)
            else
                a.slice_queue[atomicAdd(&a.walk_ctr[2], 1u)] = (unsigned)(b0 >> 6);
        }
    }
}

// Where a block of k_walk_multi adds up what its leavers leave in each tet
// (six edge sums, four vertex sums) before it goes to memory: leavers of one
// place cross the same few tets.  Open addressing by tet; what finds no place
// within kTries steps goes to memory directly.  The walk was bound by these
// float64 atomics, 16 or more per leaver: 1e8 particles in a bunch 1430 -> 780 us,
// 1e7 float64 50 -> 37, 5e7 mixed 127 -> 111.
struct LeaverSums {
    static constexpr int kSlots = 512, kTries = 8, kSums = 10;
    double sum[kSlots][kSums];
    int tet[kSlots];

    __device__ __forceinline__ int place(int T) {
        int h = T & (kSlots - 1);
        for (int tries = 0; tries < kTries; ++tries, h = (h + 1) & (kSlots - 1)) {
            const int was = atomicCAS(&tet[h], -1, T);
            if (was == -1 || was == T) return h;
        }
        return -1;
    }
    template <typename Real>
    __device__ __forceinline__ void add_edges(const StepArgs<Real> &a, int T, const double g6[6]) {
        const int h = place(T);
        if (h >= 0) {
#pragma unroll
            for (int e = 0; e < 6; ++e) unsafeAtomicAdd(&sum[h][e], g6[e]);
        } else {
            double *slot = a.tetG + (int64_t)T * 8;
#pragma unroll
            for (int e = 0; e < 6; ++e) unsafeAtomicAdd(&slot[e], a.qw * g6[e]);
        }
    }
    template <typename Real>
    __device__ __forceinline__ void add_charge(const StepArgs<Real> &a, int T, const double l[4]) {
        const int h = place(T);
        if (h >= 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) unsafeAtomicAdd(&sum[h][6 + k], l[k]);
        } else {
            const TetTopo tp = a.topo[T];
#pragma unroll
            for (int k = 0; k < 4; ++k) unsafeAtomicAdd(&a.rho[tp.v[k]], a.qw * l[k]);
        }
    }
    // by all threads of the block
    __device__ __forceinline__ void clear() {
        for (int i = threadIdx.x; i < kSlots; i += blockDim.x) tet[i] = -1;
        for (int i = threadIdx.x; i < kSlots * kSums; i += blockDim.x) (&sum[0][0])[i] = 0.0;
        __syncthreads();
    }
    template <typename Real>
    __device__ __forceinline__ void flush(const StepArgs<Real> &a) {
        __syncthreads();
        for (int i = threadIdx.x; i < kSlots * kSums; i += blockDim.x) {
            const int h = i / kSums, k = i % kSums, T = tet[h];
            const double x = sum[h][k];
            if (T < 0 || x == 0.0) continue;
            if (k < 6)
                unsafeAtomicAdd(&a.tetG[(int64_t)T * 8 + k], a.qw * x);
            else
                unsafeAtomicAdd(&a.rho[a.topo[T].v[k - 6]], a.qw * x);
        }
    }
};

// A leaver of k_push_multi: its walk at the step it left in, then its
// remaining steps, each as the particle kernel and the walk take it.  In-tet
// pieces are summed per visit of a tet and added to the tet's current slots.
template <typename Real, int kSnap, bool kFixed>
__device__ __forceinline__ void walk_leaver(const StepArgs<Real> &a, const MultiArgs<kSnap> &ma, LeaverSums &sums,
                                            int64_t p) {
    double *lam[3] = {a.lam1, a.lam2, a.lam3};
    uint32_t *fl[3] = {reinterpret_cast<uint32_t *>(a.lam1), reinterpret_cast<uint32_t *>(a.lam2),
                       reinterpret_cast<uint32_t *>(a.lam3)};
    const int marked = a.tet[p];
    double l[4];
    l[0] = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) l[k + 1] = kFixed ? (double)fl[k][p] : lam[k][p];
    Real v[3] = {a.v0[p], a.v1[p], a.v2[p]};
    if (marked > -2) return;
    const int code = walker_tet(marked);
    int j = code / (int)a.nt;
    int T = code - j * (int)a.nt;
    if (j >= ma.nsteps) return;
    double s[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    bool some = false;
    auto flush = [&]() {
        if (!some) return;
        double g6[6];
        unscale_sums<kFixed>(s);
        edge_sums(s, g6);
        sums.add_edges(a, T, g6);
#pragma unroll
        for (int e = 0; e < 6; ++e) s[e] = 0.0;
        some = false;
    };
    bool walks = true;
#pragma unroll 1
    for (;;) {
        if (walks) {
            flush();
            const Real dx[3] = {a.dt_r * v[0], a.dt_r * v[1], a.dt_r * v[2]};
            double d[3] = {(double)dx[0], (double)dx[1], (double)dx[2]};
            if (kFixed)
#pragma unroll
                for (int k = 1; k < 4; ++k) l[k] *= kFix;
            LastPiece end;
            T = walk_pieces<Real, false>(a, T, l, d, v, nullptr, nullptr, kFixed, &end,
                                         [&](int t, const TetTopo &, const double l0[4], const double dl[4]) {
                                             double g6[6];
                                             piece_sums(l0, dl, g6);
                                             sums.add_edges(a, t, g6);
                                         });
            add_piece(end, kOne<kFixed>, s);
            some = true;
            if (kFixed) {
                uint32_t u[3];
                fix_round3(l[1], l[2], l[3], u);
#pragma unroll
                for (int k = 0; k < 3; ++k) l[k + 1] = (double)u[k];
            }
        }
        if (++j >= ma.nsteps) break;
        Real cf[kRowReals];
        const double *pr = ma.parts + (int64_t)T * (kRowParts<kSnap> * kRowReals);
#pragma unroll
        for (int c = 0; c < kRowReals; ++c) cf[c] = (Real)row_entry<kSnap>(pr + c, kRowReals, ma.wc[j], ma.ws[j]);
        Real gm[9], gr[9];
        load_rows<Real, kFixed>(a, T, gm, gr);
        const Real x[3] = {(Real)l[1], (Real)l[2], (Real)l[3]};
        gather_boris(cf, gm, x, a.h, v);
        double dl[4], t[4];
        walks = !increments(gr, v, a.dt_r, kOne<kFixed>, l, dl, t);
        if (!walks) {
            stay_step<kFixed>(l, dl, t, s);
            some = true;
        } else if (!(isfinite(v[0]) && isfinite(v[1]) && isfinite(v[2]))) {
            atomicOr(a.status, (unsigned)ETPIC_DEV_NAN);
        }
    }
    flush();
    a.tet[p] = T;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (kFixed) {
            fl[k][p] = (uint32_t)l[k + 1];
            l[k + 1] *= kFix;
        } else {
            lam[k][p] = l[k + 1];
        }
    }
    a.v0[p] = v[0];
    a.v1[p] = v[1];
    a.v2[p] = v[2];
    if (a.rho) {
        l[0] = 1.0 - l[1] - l[2] - l[3];
        sums.add_charge(a, T, l);
    }
}

// The counters of the two walk queues alternate between two sets from one
// launch pair to the next: this kernel reads its own set and clears the other
// one for the next pair, so no block waits for the last one to reset them.
template <typename Real, int kSnap, bool kFixed>
__global__ void __launch_bounds__(kBlock) k_walk_multi(StepArgs<Real> a, MultiArgs<kSnap> ma, unsigned *next_ctr) {
    __shared__ LeaverSums sums;
    if (blockIdx.x == 0) clear_counters(next_ctr);
    sums.clear();
    take_leavers(a, [&](int64_t p) { walk_leaver<Real, kSnap, kFixed>(a, ma, sums, p); });
    sums.flush(a);
}

// ------------------------------------------------------------------ downshifted step
// The Particle Push section's other scheme: the velocity update integrates the
// carrier exactly against the envelope fields and velocities sampled along the
// trajectory and interpolated in time (Lagrange basis N_k on the nodes t_n,
// t_{n-1}, t_{n-2}):
//   v^{n+1} = v^n + q/m sum_k (Re E_k M^r_k + Im E_k M^i_k + Edc_k P_k)
//           + q/m sum_{j,k} v^{n-j} x (Re B_k L^r_jk + Im B_k L^i_jk + Bdc_k Q_jk),
// the positions advance by the Adams-Bashforth stencil in the velocities
// (eq. newtons), and the path is walked and deposited as in the fine-step
// scheme.  The weights M, L, P, Q of a step are computed on the host.
//
// The envelope samples need the complex per-tet coefficients (Re, Im and dc
// parts separately, the carrier being applied by the weights): rows of 72
// reals per tet, A_re, A_im, A_dc, C_re, C_im, C_dc, each 4 x 3 (A_k at 3k),
// built once per call since the fields are fixed within it.
constexpr int kEnvRow = 72;
static_assert(kRowParts<3> * kRowReals <= kEnvRow, "the parts of three snapshots fit the wide rows");

__global__ void __launch_bounds__(kBlock) k_tet_coef_env(int64_t nt, const double *__restrict__ prow,
                                                         const int32_t *__restrict__ tetface, FieldPtrs F,
                                                         double *__restrict__ out, double *__restrict__ slots) {
    // blockIdx.y: 0..2 the edge rows (Re, Im, dc), 3..5 the face rows
    const int part = blockIdx.y;
    if (part == 0) {
        const int64_t T0 = (int64_t)blockIdx.x * kBlock;
        clear_slots(slots, T0, (int)min((int64_t)kBlock, nt - T0));
    }
    const int64_t T = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (T >= nt) return;
    const double *row = prow + T * PushRow<double>::kStride;
    double g[4][3];
#pragma unroll
    for (int k = 1; k < 4; ++k)
#pragma unroll
        for (int d = 0; d < 3; ++d) g[k][d] = row[3 * (k - 1) + d];
#pragma unroll
    for (int d = 0; d < 3; ++d) g[0][d] = -(g[1][d] + g[2][d] + g[3][d]);
    int32_t tp[10];
    const int32_t *re = reinterpret_cast<const int32_t *>(row + PushRow<double>::kEdges);
#pragma unroll
    for (int k = 0; k < 6; ++k) tp[k] = re[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) tp[6 + k] = tetface[4 * T + k];
    // the same expansions as the per-step coefficients, with (c, s) selecting
    // the real part (1, 0), the imaginary part (0, -1) or neither (0, 0), and
    // the dc DoFs kept only for the dc rows
    const int which = part % 3;
    FieldPtrs G = F;
    G.c = which == 0 ? 1.0 : 0.0;
    G.s = which == 1 ? -1.0 : 0.0;
    if (which != 2) {
        G.e_dc = nullptr;
        G.b_dc = nullptr;
    }
    double o[12];
    if (part < 3) {
        coef_A<0>(tp, g, G, o);
        coef_A<1>(tp, g, G, o + 3);
        coef_A<2>(tp, g, G, o + 6);
        coef_A<3>(tp, g, G, o + 9);
    } else {
        coef_C<0>(tp, g, G, o);
        coef_C<1>(tp, g, G, o + 3);
        coef_C<2>(tp, g, G, o + 6);
        coef_C<3>(tp, g, G, o + 9);
    }
    double *dst = out + T * kEnvRow + 12 * part;
#pragma unroll
    for (int d = 0; d < 12; ++d) dst[d] = o[d];
}

// History of the downshifted integrator: 48 arrays of length n in one
// caller-owned buffer (float64, or float32 in the mixed form), array i at
// hist + i * n.  Arrays 0..11: velocity ring,
// v^m in slot m mod 4 (components 3 slot + c); 12..29: E samples, the sample of
// step m in slot m mod 2 (12 + 9 slot + i, i = Re 0..2, Im 3..5, dc 6..8);
// 30..47: B samples likewise.
constexpr int kDsArrays = 48;

// Weights of one step, in float64 on the host.
struct DsWeights {
    double Mr[3], Mi[3], P[3], Lr[9], Li[9], Q[9];
    double ab[4];             // Adams-Bashforth coefficients times the step
};

// A launch takes each particle through several downshifted steps, as
// k_push_multi takes the fine-step scheme's: state, velocity ring and field
// samples stay in registers between them and cross HBM once per launch (the
// history alone is 384 B of float64 per particle), the rows of the wavefront's
// tets are staged in LDS once, and the path integrals are reduced and flushed
// once.  Every step takes three interpolation nodes and the fourth-order
// displacement; while fewer earlier steps exist the weights of the missing
// ones are 0 and their registers hold 0 (those first steps go one per launch:
// their P, Q and displacement weights differ).  Measured, 1e7 float64 on 40^3 x
// 6 tets, ten steps per call: 13.34 -> 2.51 ms; 3e6 mixed, 13 steps: 3.85 ->
// 0.76 ms.  The float64 form keeps 217 registers, two wavefronts per SIMD: its
// steps are arithmetic, and the history is read and written once per launch.
constexpr int kMaxDs = 16;

template <typename Real>
struct DsArgs {
    const double *rows;       // float32: nt * kEnvRow; float64: nt * kRowParts<1> * 10 (the row's parts)
    Real *hist;
    int64_t stride;           // n
    int phase;                // number of the first step, mod 4
    int hist0;                // downshifted steps taken before it (at most 3 matter)
    int nsteps;
    int width;                // particles per wavefront (push_width)
    Real P[3], Q[9];          // weights that do not depend on the step's time (3 nodes; Q[3 j + k])
    Real ab[4];               // Adams-Bashforth coefficients times the step
    Real qm;
    Real Mr[kMaxDs][3], Mi[kMaxDs][3], Lr[kMaxDs][9], Li[kMaxDs][9];
};

template <typename Real>
__device__ __forceinline__ Real *ds_v(const DsArgs<Real> &d, int slot, int c) { return d.hist + (3 * slot + c) * d.stride; }
template <typename Real>
__device__ __forceinline__ Real *ds_e(const DsArgs<Real> &d, int slot, int i) { return d.hist + (12 + 9 * slot + i) * d.stride; }
template <typename Real>
__device__ __forceinline__ Real *ds_b(const DsArgs<Real> &d, int slot, int i) { return d.hist + (30 + 9 * slot + i) * d.stride; }

// A particle's multistep state before a step n: V[0..3] = v^n .. v^{n-3} and
// V[4] (kept for the ring's oldest slot), E[k], B[k] = samples of t_{n-1-k}
// (re, im, dc; 3 each).
template <typename Real>
struct DsState {
    Real V[5][3], E[2][9], B[2][9];
};

// The velocities and samples of the steps before step j of the launch.
template <typename Real, bool kEdc>
__device__ __forceinline__ void ds_load(const DsArgs<Real> &d, int64_t p, int j, int steps_before, DsState<Real> &s) {
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int c = 0; c < 3; ++c)
            s.V[i + 1][c] =
                i < steps_before ? __builtin_nontemporal_load(ds_v(d, (d.phase + j - 1 - i) & 3, c) + p) : (Real)0;
#pragma unroll
    for (int k = 0; k < 2; ++k)
#pragma unroll
        for (int c = 0; c < 9; ++c) {
            const int sl = (d.phase + j - 1 - k) & 1;
            s.E[k][c] = k < steps_before && (kEdc || c < 6) ? __builtin_nontemporal_load(ds_e(d, sl, c) + p) : (Real)0;
            s.B[k][c] = k < steps_before ? __builtin_nontemporal_load(ds_b(d, sl, c) + p) : (Real)0;
        }
}

// The history after step j: v^n, ... and the samples of the last `taken` steps.
template <typename Real, bool kEdc>
__device__ __forceinline__ void ds_store(const DsArgs<Real> &d, int64_t p, int j, int taken, const DsState<Real> &s) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (i < taken)
#pragma unroll
            for (int c = 0; c < 3; ++c)
                __builtin_nontemporal_store(s.V[i + 1][c], ds_v(d, (d.phase + j - i) & 3, c) + p);
#pragma unroll
    for (int k = 0; k < 2; ++k)
        if (k < taken)
#pragma unroll
            for (int c = 0; c < 9; ++c) {
                const int sl = (d.phase + j - k) & 1;
                if (kEdc || c < 6) __builtin_nontemporal_store(s.E[k][c], ds_e(d, sl, c) + p);
                __builtin_nontemporal_store(s.B[k][c], ds_b(d, sl, c) + p);
            }
}

// A tet's rows for the step: in the float32 form the 72 complex-envelope reals,
// in the float64 form the parts of the 10-real row (E = A_0 + beta x u, B =
// C_0 + b u for the real, imaginary and dc part alike) and the geometry row.
template <typename Row, typename Real>
struct DsRows {
    const Row *row;
    const Real *geo, *grad;
};

// Samples of E (re, im, dc) and B (re, im, dc) at the barycentrics l.
template <bool kEdc, typename Row>
__device__ __forceinline__ void ds_sample(const DsRows<Row, float> &r, const double l[4], float E[9], float B[9]) {
    const float lr[4] = {(float)(1.0 - l[1] - l[2] - l[3]), (float)l[1], (float)l[2], (float)l[3]};
#pragma unroll
    for (int part = 0; part < 3; ++part)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const Row *e = r.row + 12 * part + c, *b = e + 36;
            E[3 * part + c] = (part == 2 && !kEdc)
                                  ? 0.0f
                                  : lr[0] * (float)e[0] + lr[1] * (float)e[3] + lr[2] * (float)e[6] + lr[3] * (float)e[9];
            B[3 * part + c] = lr[0] * (float)b[0] + lr[1] * (float)b[3] + lr[2] * (float)b[6] + lr[3] * (float)b[9];
        }
}
template <bool kEdc>
__device__ __forceinline__ void ds_sample(const DsRows<double, double> &r, const double l[4], double E[9], double B[9]) {
    double u[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = fma(l[3], r.geo[6 + d], fma(l[2], r.geo[3 + d], l[1] * r.geo[d]));
#pragma unroll
    for (int part = 0; part < 3; ++part) {
        const double *q = r.row + kRowReals * part;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const int x = (c + 1) % 3, y = (c + 2) % 3;
            E[3 * part + c] = (part == 2 && !kEdc) ? 0.0 : fma(q[3 + x], u[y], fma(-q[3 + y], u[x], q[c]));
            B[3 * part + c] = fma(q[9], u[c], q[6 + c]);
        }
    }
}

// acc = the velocity update's sums at step j over the samples E_k, B_k of
// t_{n-k} (k = 0: S) and the velocities V_j.
template <bool kEdc>
__device__ __forceinline__ void ds_sums(const DsArgs<float> &d, int j0, const float S_E[9], const float S_B[9],
                                        const DsState<float> &s, float acc[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = S_E[c] * d.Mr[j0][0] + S_E[3 + c] * d.Mi[j0][0] + S_E[6 + c] * d.P[0];
#pragma unroll
    for (int k = 1; k < 3; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            acc[c] += s.E[k - 1][c] * d.Mr[j0][k] + s.E[k - 1][3 + c] * d.Mi[j0][k];
            if (kEdc) acc[c] += s.E[k - 1][6 + c] * d.P[k];
        }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float *Bk = k == 0 ? S_B : s.B[k - 1];
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            const int jk = 3 * j + k;
            float Bw[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) Bw[c] = Bk[c] * d.Lr[j0][jk] + Bk[3 + c] * d.Li[j0][jk] + Bk[6 + c] * d.Q[jk];
            acc[0] += s.V[j][1] * Bw[2] - s.V[j][2] * Bw[1];
            acc[1] += s.V[j][2] * Bw[0] - s.V[j][0] * Bw[2];
            acc[2] += s.V[j][0] * Bw[1] - s.V[j][1] * Bw[0];
        }
    }
}
// (float64: the velocities weighted first, three crosses per node, fma chains)
template <bool kEdc>
__device__ __forceinline__ void ds_sums(const DsArgs<double> &d, int j0, const double S_E[9], const double S_B[9],
                                        const DsState<double> &s, double acc[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double *Ek = k == 0 ? S_E : s.E[k - 1], *Bk = k == 0 ? S_B : s.B[k - 1];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            acc[c] = fma(Ek[c], d.Mr[j0][k], fma(Ek[3 + c], d.Mi[j0][k], acc[c]));
            if (kEdc) acc[c] = fma(Ek[6 + c], d.P[k], acc[c]);
        }
#pragma unroll
        for (int part = 0; part < 3; ++part) {
            const double *w = part == 0 ? d.Lr[j0] : (part == 1 ? d.Li[j0] : d.Q);
            const double *b = Bk + 3 * part;
            double U[3];
#pragma unroll
            for (int c = 0; c < 3; ++c)
                U[c] = fma(s.V[2][c], w[6 + k], fma(s.V[1][c], w[3 + k], s.V[0][c] * w[k]));
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int x = (c + 1) % 3, y = (c + 2) % 3;
                acc[c] = fma(U[x], b[y], fma(-U[y], b[x], acc[c]));
            }
        }
    }
}

// The Adams-Bashforth displacement from v^n .. v^{n-3}.
template <typename Real>
__device__ __forceinline__ void ds_displacement(const DsArgs<Real> &d, const Real *V0, const Real *V1, const Real *V2,
                                                const Real *V3, Real dx[3]) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        if constexpr (std::is_same<Real, float>::value) {
            dx[c] = 0;
            dx[c] += d.ab[0] * V0[c];
            dx[c] += d.ab[1] * V1[c];
            dx[c] += d.ab[2] * V2[c];
            dx[c] += d.ab[3] * V3[c];
        } else {
            dx[c] = fma(d.ab[3], V3[c], fma(d.ab[2], V2[c], fma(d.ab[1], V1[c], d.ab[0] * V0[c])));
        }
    }
}

// One step's samples, velocity and increments; on return s holds the state
// before the next step (V[0] = v^{n+1}, not yet mirrored).  True if the particle
// stays in its tet.
template <typename Real, bool kEdc, typename Row>
__device__ __forceinline__ bool ds_step(const DsArgs<Real> &d, int j, const DsRows<Row, Real> &r, const double l[4],
                                        DsState<Real> &s, double dl[4], double t[4]) {
    Real S_E[9], S_B[9], acc[3], dx[3];
    ds_sample<kEdc>(r, l, S_E, S_B);
    ds_sums<kEdc>(d, j, S_E, S_B, s, acc);
    ds_displacement(d, s.V[0], s.V[1], s.V[2], s.V[3], dx);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const Real vn = s.V[0][c] + d.qm * acc[c];
        s.V[4][c] = s.V[3][c];
        s.V[3][c] = s.V[2][c];
        s.V[2][c] = s.V[1][c];
        s.V[1][c] = s.V[0][c];
        s.V[0][c] = vn;
    }
#pragma unroll
    for (int c = 0; c < 9; ++c) {
        s.E[1][c] = s.E[0][c];
        s.E[0][c] = S_E[c];
        s.B[1][c] = s.B[0][c];
        s.B[0][c] = S_B[c];
    }
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        if constexpr (std::is_same<Real, float>::value)
            dl[k] = (double)(r.grad[3 * k - 3] * dx[0] + r.grad[3 * k - 2] * dx[1] + r.grad[3 * k - 1] * dx[2]);
        else
            dl[k] = fma(r.grad[3 * k - 1], dx[2], fma(r.grad[3 * k - 2], dx[1], r.grad[3 * k - 3] * dx[0]));
        t[k] = l[k] + dl[k];
    }
    t[0] = 1.0 - t[1] - t[2] - t[3];
    return t[0] >= 0.0 && t[1] >= 0.0 && t[2] >= 0.0 && t[3] >= 0.0;
}

// kLen reals of each of a wavefront's nr tets, `stride` apart in memory, into
// its LDS rows, four loads of a lane in flight together (one after the other
// they were most of a launch of few particles: one step of 1,000 on 750 tets,
// mixed, 66 -> 41 us with 16 particles to a wavefront; of 4e6 on 384,000, ten
// steps, 878 -> 737.  Eight: 734, but ten float64 steps of 1e7, three tets to a
// wavefront, 2495 instead of 2460).
template <int kLen, int kRow, typename Src, typename Real>
__device__ __forceinline__ void stage_rows(const Src *__restrict__ src, int stride, const int *tets, int nr, int ln,
                                           Real *rows) {
    constexpr int kLoads = 4;
    const int total = nr * kLen;
#pragma unroll 1
    for (int i0 = ln; i0 < total; i0 += 64 * kLoads) {
        Src x[kLoads];
        int at[kLoads];
#pragma unroll
        for (int k = 0; k < kLoads; ++k) {
            const int i = min(i0 + 64 * k, total - 1), j = i / kLen, c = i - j * kLen;
            at[k] = j * kRow + c;
            x[k] = src[(int64_t)max(tets[j], 0) * stride + c];
        }
#pragma unroll
        for (int k = 0; k < kLoads; ++k) rows[at[k]] = (Real)x[k];
    }
}

// Real = double: the float64 form.  Real = float: samples, velocities and the
// velocity update in float32, positions, the barycentric increments and the
// deposit in float64 (the mixed form of the fine-step kernel).
template <typename Real, bool kRho, bool kEdc>
__global__ void __launch_bounds__(kBlock) k_push_ds(StepArgs<Real> a, DsArgs<Real> d, int remap) {
    constexpr bool f64 = std::is_same<Real, double>::value;
    constexpr int kRuns = 16;
    constexpr int kSrc = f64 ? kRowParts<1> * kRowReals : kEnvRow;   // reals of a tet's row in memory
    constexpr int kGeo = f64 ? 9 : 0;
    constexpr int kRow = f64 ? 50 : 84;          // staged: row, geometry (float64), gradients, padding
    constexpr int kWaves = kBlock / 64;
    constexpr int kRowBytes = kRuns * kRow * (int)sizeof(Real);
    static_assert(kSrc + kGeo + 9 <= kRow && kRowBytes >= 64 * 3 * 16, "staged row");
    __shared__ __align__(16) char s_lds[kWaves][kRowBytes + 64 * 4];
    unsigned blk = blockIdx.x;
    if (remap) blk = xcd_block(blk, gridDim.x);
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned ln = threadIdx.x & 63;
    Real *rows = reinterpret_cast<Real *>(s_lds[wv]);
    int *s_tet = reinterpret_cast<int *>(s_lds[wv] + kRowBytes);
    const int64_t b0 = ((int64_t)blk * kWaves + wv) * d.width;
    if (b0 >= a.n) return;   // the whole wavefront; no block barrier below
    const int64_t p = b0 + ln;
    int T = -1;
    double l[4] = {0.0, 0.0, 0.0, 0.0};   // l[0] unused: lam0 is implicit
    DsState<Real> s{};
    if (p < a.n && (int)ln < d.width) {
        T = __builtin_nontemporal_load(lane_at(a.tet + b0, ln));
        l[1] = __builtin_nontemporal_load(lane_at(a.lam1 + b0, ln));
        l[2] = __builtin_nontemporal_load(lane_at(a.lam2 + b0, ln));
        l[3] = __builtin_nontemporal_load(lane_at(a.lam3 + b0, ln));
        s.V[0][0] = __builtin_nontemporal_load(lane_at(a.v0 + b0, ln));
        s.V[0][1] = __builtin_nontemporal_load(lane_at(a.v1 + b0, ln));
        s.V[0][2] = __builtin_nontemporal_load(lane_at(a.v2 + b0, ln));
        ds_load<Real, kEdc>(d, p, 0, d.hist0, s);
        if ((unsigned)T >= (unsigned)a.nt) {
            atomicOr(a.status, (unsigned)ETPIC_DEV_BADTET);
            T = -1;
        }
    }
    const bool act = T >= 0;
    const WaveRuns runs = wave_runs(T, ln);
    const unsigned long long upto = ln == 63 ? ~0ull : ((2ull << ln) - 1ull);
    const unsigned long long heads = __ballot(runs.head);
    const int nruns = __popcll(heads);
    const int run = __popcll(heads & upto) - 1;
    if (runs.head) s_tet[run] = T;
    double sum[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int leave = -1;   // step at which the particle left its tet
#pragma unroll 1
    for (int r0 = 0; r0 < nruns; r0 += kRuns) {
        const int nr = min(kRuns, nruns - r0);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        stage_rows<kSrc, kRow>(d.rows, kSrc, s_tet + r0, nr, ln, rows);
        if (kGeo) stage_rows<9, kRow>(a.geo, GeoRow<Real>::kStride, s_tet + r0, nr, ln, rows + kSrc);
        stage_rows<9, kRow>(a.gpush, PushRow<Real>::kStride, s_tet + r0, nr, ln, rows + kSrc + kGeo);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        bool live = act && run >= r0 && run < r0 + nr;
        const Real *row = rows + (live ? (run - r0) * kRow : 0);
        const DsRows<Real, Real> r{row, row + kSrc, row + kSrc + kGeo};
#pragma unroll 1
        for (int j = 0; j < d.nsteps; ++j) {
            if (live) {
                double dl[4], t[4];
                if (ds_step<Real, kEdc>(d, j, r, l, s, dl, t)) {
                    stay_step<false>(l, dl, t, sum);
                } else {
                    leave = j;
                    live = false;
                }
                // (unlike the fine-step scheme's, this step's displacement
                // does not contain its new velocity)
                if (!(isfinite(s.V[0][0]) && isfinite(s.V[0][1]) && isfinite(s.V[0][2])))
                    atomicOr(a.status, (unsigned)ETPIC_DEV_NAN);
            }
            if (!__builtin_amdgcn_ballot_w64(live)) break;
        }
    }
    const bool left = leave >= 0;
    if (act) {
        __builtin_nontemporal_store(l[1], lane_at(a.lam1 + b0, ln));
        __builtin_nontemporal_store(l[2], lane_at(a.lam2 + b0, ln));
        __builtin_nontemporal_store(l[3], lane_at(a.lam3 + b0, ln));
        __builtin_nontemporal_store(s.V[0][0], lane_at(a.v0 + b0, ln));
        __builtin_nontemporal_store(s.V[0][1], lane_at(a.v1 + b0, ln));
        __builtin_nontemporal_store(s.V[0][2], lane_at(a.v2 + b0, ln));
        if (left) *lane_at(a.tet + b0, ln) = leaver_mark(T, leave, a.nt);
        const int last = left ? leave : d.nsteps - 1;
        ds_store<Real, kEdc>(d, p, last, last + 1, s);
    }
#pragma unroll
    for (int e = 0; e < 6; ++e) sum[e] = run_total(sum[e], runs);
    double g6[6];
    edge_sums(sum, g6);
    const bool flush = act && runs.lane == runs.run_end;
    if (a.tetG)
        flush_runs_together<Real, true>(a, T, g6, runs, flush, reinterpret_cast<double2 *>(rows));
    else
        flush_runs_together<Real, false>(a, T, g6, runs, flush, reinterpret_cast<double2 *>(rows));
    if (kRho) {
        double r4[4];
#pragma unroll
        for (int k = 1; k < 4; ++k) r4[k] = run_total(act && !left ? l[k] : 0.0, runs);
        const unsigned long long here = __ballot(act && !left);
        r4[0] = (double)__popcll(here & upto & ~((1ull << runs.head_lane) - 1ull)) - r4[1] - r4[2] - r4[3];
        if (flush) {
            const TetTopo *tp = a.topo + T;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (r4[k] != 0.0) unsafeAtomicAdd(&a.rho[tp->v[k]], a.qw * r4[k]);
        }
    }
    // leavers to the particle queue, or their slice when it is full
    const unsigned long long wmask = __ballot(left);
    if (wmask) {
        if (!queue_leavers(a, wmask, left, (unsigned)p, !a.walk_by_slice, blk) && ln == 0)
            a.slice_queue[atomicAdd(&a.walk_ctr[2], 1u)] = (unsigned)(b0 >> 6);
    }
}

// A leaver of k_push_ds: the walk of the step it left in (its displacement
// rebuilt from the stored ring; at a wall the velocity samples the next steps
// use, v^n, v^{n-1}, v^{n-2}, are mirrored with v^{n+1}), then its remaining steps.
template <typename Real, bool kEdc>
__device__ __forceinline__ void walk_leaver_ds(const StepArgs<Real> &a, const DsArgs<Real> &d, int64_t p) {
    const int marked = a.tet[p];
    if (marked > -2) return;
    const int code = walker_tet(marked);
    int j = code / (int)a.nt;
    int T = code - j * (int)a.nt;
    if (j >= d.nsteps) return;
    double *lam[3] = {a.lam1, a.lam2, a.lam3};
    double l[4];
    l[0] = 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) l[k + 1] = lam[k][p];
    // the state before the step after the one that left: V[0] = v^{n+1}
    DsState<Real> s{};
    ds_load<Real, kEdc>(d, p, j + 1, d.hist0 + j + 1, s);
    s.V[0][0] = a.v0[p];
    s.V[0][1] = a.v1[p];
    s.V[0][2] = a.v2[p];
#pragma unroll
    for (int c = 0; c < 3; ++c) s.V[4][c] = d.hist0 + j + 1 > 3 ? ds_v(d, (d.phase + j - 3) & 3, c)[p] : (Real)0;
    double sum[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    bool some = false;
    auto flush = [&]() {
        if (!some) return;
        double g6[6];
        edge_sums(sum, g6);
        const double none[4] = {0.0, 0.0, 0.0, 0.0};
        if (a.tetG)
            flush_run<Real, false, true>(a, T, g6, none);
        else
            flush_run<Real, false, false>(a, T, g6, none);
#pragma unroll
        for (int e = 0; e < 6; ++e) sum[e] = 0.0;
        some = false;
    };
    bool walks = true;
#pragma unroll 1
    for (;;) {
        if (walks) {
            flush();
            Real dx[3];
            ds_displacement(d, s.V[1], s.V[2], s.V[3], s.V[4], dx);
            double dd[3] = {(double)dx[0], (double)dx[1], (double)dx[2]};
            double ext[3][3];
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int c = 0; c < 3; ++c) ext[i][c] = (double)s.V[i + 1][c];
            Real v[3] = {s.V[0][0], s.V[0][1], s.V[0][2]};
            LastPiece end;
            T = walk<Real, false, 3>(a, T, l, dd, v, nullptr, ext, false, &end);
            add_piece(end, 1.0, sum);
            some = true;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                s.V[0][c] = v[c];
#pragma unroll
                for (int i = 0; i < 3; ++i) s.V[i + 1][c] = (Real)ext[i][c];
            }
        }
        if (++j >= d.nsteps) break;
        const Real *grad = a.gpush + (int64_t)T * PushRow<Real>::kStride;
        const Real *geo = a.geo + (int64_t)T * GeoRow<Real>::kStride;
        double dl[4], t[4];
        constexpr int kSrc = std::is_same<Real, double>::value ? kRowParts<1> * kRowReals : kEnvRow;
        const DsRows<double, Real> r{d.rows + (int64_t)T * kSrc, geo, grad};
        walks = !ds_step<Real, kEdc>(d, j, r, l, s, dl, t);
        if (!(isfinite(s.V[0][0]) && isfinite(s.V[0][1]) && isfinite(s.V[0][2])))
            atomicOr(a.status, (unsigned)ETPIC_DEV_NAN);
        if (!walks) {
            stay_step<false>(l, dl, t, sum);
            some = true;
        }
    }
    flush();
    a.tet[p] = T;
#pragma unroll
    for (int k = 0; k < 3; ++k) lam[k][p] = l[k + 1];
    a.v0[p] = s.V[0][0];
    a.v1[p] = s.V[0][1];
    a.v2[p] = s.V[0][2];
    // every ring slot that holds a step taken: a wall mirrors older ones too
    ds_store<Real, kEdc>(d, p, d.nsteps - 1, d.hist0 + d.nsteps, s);
    if (a.rho) {
        const TetTopo tp = a.topo[T];
        l[0] = 1.0 - l[1] - l[2] - l[3];
#pragma unroll
        for (int k = 0; k < 4; ++k) unsafeAtomicAdd(&a.rho[tp.v[k]], a.qw * l[k]);
    }
}

template <typename Real, bool kEdc>
__global__ void __launch_bounds__(kBlock) k_walk_ds(StepArgs<Real> a, DsArgs<Real> d, unsigned *next_ctr) {
    if (blockIdx.x == 0) clear_counters(next_ctr);
    take_leavers(a, [&](int64_t p) { walk_leaver_ds<Real, kEdc>(a, d, p); });
}

// ------------------------------------------------------------------ adjoint step
// Reverse of float64 steps for every particle, given the state before the
// first of them (a checkpoint) and the adjoints of the state after the last.
// Recomputes gather, Boris and the walk's reflections, then back-propagates:
//   x_{k+1} = R (x_k + dt v+) + const, v_{k+1} = R v+         (walk, reflections R)
//   v+ = Boris(v_k, E, B)                                        (vjp written out)
//   E = A_0 + beta x u, B = C_0 + b u, u = x - r_0
// and accumulates the gradient with respect to the complex edge envelope,
// dL/dRe e_e + j dL/dIm e_e = (Ebar . W1_e(x_k)) e^{-j w t_k}, reduced over runs
// of equal tet before the float64 atomics.
constexpr int kMaxAdj = 5;   // steps reversed per launch: the states between them fill the LDS left beside the rows

__global__ void __launch_bounds__(kBlock) k_copy_state(etpic_particles src, etpic_particles dst) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= src.n) return;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        dst.lam[k][p] = src.lam[k][p];
        static_cast<double *>(dst.vel[k])[p] = static_cast<const double *>(src.vel[k])[p];
    }
    dst.tet[p] = src.tet[p];
}

struct AdjArgs {
    const double *parts;             // row parts (k_tet_coef, kCoefParts)
    const double *lam[3], *v[3];     // the state before the launch's first step
    const int32_t *tet;
    double *vb[3], *xb[3];
    double *grad_e;
    int64_t first, end;              // particles [first, end) of this launch
    int nsteps;                      // at most kMaxAdj
    double c[kMaxAdj], s[kMaxAdj];   // cos, sin of the carrier phase of each step
    // per-step states of the particles that leave their tet (k_adjoint_leavers)
    double *s_lam[kMaxAdj][3], *s_v[kMaxAdj][3];
    int32_t *s_tet[kMaxAdj];
};

// Reverse of one step from the state (l, v) before it: xb, vb in: adjoints of
// the end point and velocity, out: of the start point and velocity.  R: the
// step's reflections (null: none).  w: the envelope gradient's six sums, w[0..2]
// = Eb . grad l_k, w[3..5] = l_i Eb . grad l_k - l_k Eb . grad l_i for (i,k) =
// (1,2), (1,3), (2,3) (edge_sums turns them into Eb . W1_e).
__device__ __forceinline__ void adjoint_step(const double *cf, const double *gm, const double *gr, const double l[4],
                                             const double v[3], double h, double dt, const double *R, double xb[3],
                                             double vb[3], double w[6]) {
    double u[3], E[3], vm[3], tau[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) u[d] = fma(l[3], gm[6 + d], fma(l[2], gm[3 + d], l[1] * gm[d]));
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = (d + 1) % 3, q = (d + 2) % 3;
        E[d] = fma(cf[3 + p], u[q], fma(-cf[3 + q], u[p], cf[d]));
        tau[d] = h * fma(cf[9], u[d], cf[6 + d]);
        vm[d] = fma(h, E[d], v[d]);
    }
    const double sg = two_over(fma(tau[0], tau[0], fma(tau[1], tau[1], fma(tau[2], tau[2], 1.0))));
    double vr[3], sig[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = (d + 1) % 3, q = (d + 2) % 3;
        vr[d] = fma(vm[p], tau[q], fma(-vm[q], tau[p], vm[d]));
        sig[d] = sg * tau[d];
    }
    double ob[3];
    if (R) {
        double xr[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            ob[i] = xr[i] = 0.0;
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                ob[i] = fma(R[3 * j + i], fma(dt, xb[j], vb[j]), ob[i]);
                xr[i] = fma(R[3 * j + i], xb[j], xr[i]);
            }
        }
#pragma unroll
        for (int i = 0; i < 3; ++i) xb[i] = xr[i];
    } else {
#pragma unroll
        for (int i = 0; i < 3; ++i) ob[i] = fma(dt, xb[i], vb[i]);
    }
    // out = vm + vr x sig + h E, vr = vm + vm x tau, sig = 2 tau / (1 + |tau|^2)
    double vrb[3], sigb[3], vmb[3], taub[3], Eb[3], Bb[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = (d + 1) % 3, q = (d + 2) % 3;
        vrb[d] = fma(sig[p], ob[q], -(sig[q] * ob[p]));
        sigb[d] = fma(ob[p], vr[q], -(ob[q] * vr[p]));
    }
    const double st = fma(sigb[0], tau[0], fma(sigb[1], tau[1], sigb[2] * tau[2]));
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = (d + 1) % 3, q = (d + 2) % 3;
        vmb[d] = ob[d] + fma(tau[p], vrb[q], fma(-tau[q], vrb[p], vrb[d]));
        // d sig / d tau: sg I - sg^2 tau tau^T
        taub[d] = fma(vrb[p], vm[q], fma(-vrb[q], vm[p], sg * fma(-st * sg, tau[d], sigb[d])));
        Eb[d] = h * (ob[d] + vmb[d]);
        Bb[d] = h * taub[d];
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int p = (d + 1) % 3, q = (d + 2) % 3;
        vb[d] = vmb[d];
        // E = A_0 + beta x u, B = C_0 + b u
        xb[d] += fma(cf[9], Bb[d], fma(Eb[p], cf[3 + q], -(Eb[q] * cf[3 + p])));
    }
    double eg[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        eg[k] = fma(Eb[2], gr[3 * k + 2], fma(Eb[1], gr[3 * k + 1], Eb[0] * gr[3 * k]));
#pragma unroll
    for (int k = 0; k < 3; ++k) w[k] = eg[k];
    w[3] = fma(l[1], eg[1], -(l[2] * eg[0]));
    w[4] = fma(l[1], eg[2], -(l[3] * eg[0]));
    w[5] = fma(l[2], eg[2], -(l[3] * eg[1]));
}

// The reverse of up to kMaxAdj steps per launch, one lane per particle, one
// wavefront per block: the steps are first taken forward from the state before
// them (bit for bit as the run took them), each step's start kept in LDS, then
// reversed with the adjoints in registers; the gradient sums of the tet's
// edges gather over the steps and are reduced over runs of equal tet once.
// Rows are formed from the staged parts as in k_push_multi.  A particle that
// leaves its tet in one of the steps is left to k_adjoint_leavers.
//   Bound by latency at the wavefronts that the LDS lets in: the last step's
// start stays in registers and the first one's is read again, so 14.6 KB per
// wavefront instead of 20.7, and the leavers' queue comes in parts, for which
// fewer wavefronts wait.  2e6 particles, 5 steps: 218 -> 175 us (8 rows staged
// at a time instead of 16: 166, but a second pass from 9 tets per wavefront on).
__global__ void __launch_bounds__(64) k_adjoint(StepArgs<double> a, AdjArgs b) {
    constexpr int kParts = kRowParts<1>;
    constexpr int kRuns = 16;
    constexpr int kEnt = kRuns * kRowReals;
    __shared__ double part[kParts * kEnt];
    __shared__ __align__(16) double rows[kEnt];
    __shared__ double s_state[kMaxAdj - 2][6][64];   // starts of all but the first and the last step
    __shared__ int s_tet[64];
    const unsigned ln = threadIdx.x;
    const unsigned blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t p = b.first + (int64_t)blk * 64 + ln;
    int T = -1;
    if (p < b.end) {
        T = b.tet[p];
        if ((unsigned)T >= (unsigned)a.nt) {
            atomicOr(a.status, (unsigned)ETPIC_DEV_BADTET);
            T = -1;
        }
    }
    const bool act = T >= 0;
    double l[4] = {0.0, 0.0, 0.0, 0.0}, v[3] = {0.0, 0.0, 0.0}, xb[3] = {0.0, 0.0, 0.0}, vb[3] = {0.0, 0.0, 0.0};
    if (act) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            l[k + 1] = b.lam[k][p];
            v[k] = b.v[k][p];
            xb[k] = b.xb[k][p];
            vb[k] = b.vb[k][p];
        }
    }
    double gm[9], gr[9];
    load_rows<double, false>(a, max(T, 0), gm, gr);
    const WaveRuns runs = wave_runs(T, ln);
    const unsigned long long upto = ln == 63 ? ~0ull : ((2ull << ln) - 1ull);
    const unsigned long long heads = __ballot(runs.head);
    const int nruns = __popcll(heads), run = __popcll(heads & upto) - 1;
    if (runs.head) s_tet[run] = T;
    bool left = false;
    double gc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, gs[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
    for (int r0 = 0; r0 < nruns; r0 += kRuns) {
        const int nr = min(kRuns, nruns - r0), entries = nr * kRowReals;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        stage_parts<kParts, kEnt>(b.parts, s_tet + r0, nr, ln, part);
        const bool mine = act && run >= r0 && run < r0 + nr;
        const double *cf = rows + (mine ? (run - r0) * kRowReals : 0);
        auto form_rows = [&](int j) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            for (int e = ln; e < entries; e += 64) rows[e] = row_entry<1>(part + e, kEnt, &b.c[j], &b.s[j]);
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        bool live = mine;
#pragma unroll 1
        for (int j = 0; j < b.nsteps; ++j) {
            form_rows(j);
            if (live) {
                const bool on = j < b.nsteps - 1;
                const double x[3] = {l[1], l[2], l[3]};
                double dl[4], t[4], out[3] = {v[0], v[1], v[2]};
                if (on && j > 0)
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        s_state[j - 1][k][ln] = l[k + 1];
                        s_state[j - 1][3 + k][ln] = v[k];
                    }
                gather_boris(cf, gm, x, a.h, out);
                if (!increments(gr, out, a.dt_r, 1.0, l, dl, t)) {
                    left = true;
                    live = false;
                } else if (on) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        l[k + 1] = t[k + 1];
                        v[k] = out[k];
                    }
                }
            }
        }
#pragma unroll 1
        for (int j = b.nsteps - 1; j >= 0; --j) {
            const bool kept = j == b.nsteps - 1;   // the last step's rows and states are still there
            if (!kept) form_rows(j);
            if (live) {
                if (!kept && j > 0) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        l[k + 1] = s_state[j - 1][k][ln];
                        v[k] = s_state[j - 1][3 + k][ln];
                    }
                } else if (!kept) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        l[k + 1] = b.lam[k][p];
                        v[k] = b.v[k][p];
                    }
                }
                double w[6];
                adjoint_step(cf, gm, gr, l, v, a.h, a.dt_r, nullptr, xb, vb, w);
#pragma unroll
                for (int e = 0; e < 6; ++e) {
                    gc[e] = fma(w[e], b.c[j], gc[e]);
                    gs[e] = fma(w[e], -b.s[j], gs[e]);
                }
            }
        }
    }
    if (act && !left) {
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            b.vb[k][p] = vb[k];
            b.xb[k][p] = xb[k];
        }
    }
#pragma unroll
    for (int e = 0; e < 6; ++e) {
        gc[e] = run_total(gc[e], runs);
        gs[e] = run_total(gs[e], runs);
    }
    if (act && runs.lane == runs.run_end) {
        double re[6], im[6];
        edge_sums(gc, re);
        edge_sums(gs, im);
        const int32_t *ed = push_row_edges(a.gpush + (int64_t)T * PushRow<double>::kStride);
#pragma unroll
        for (int e = 0; e < 6; ++e) {
            unsafeAtomicAdd(&b.grad_e[2 * (int64_t)ed[e]], re[e]);
            unsafeAtomicAdd(&b.grad_e[2 * (int64_t)ed[e] + 1], im[e]);
        }
    }
    // a launch takes at most kWalkQueueCap particles, and a part of the queue
    // belongs to at most kShardCap of them: the queue holds them all
    const unsigned long long wmask = __ballot(left);
    static_assert(kWalkQueueCap / 64 % (kShards * kShardRun) == 0, "the launch's blocks share the parts evenly");
    if (wmask && !queue_leavers(a, wmask, left, (unsigned)p, true, blk) && ln == 0)
        atomicOr(a.status, (unsigned)ETPIC_DEV_HOPCAP);
}

// The same for the queued particles, one lane each: forward through their
// walks with every step's start kept in the segment's state slots, then back,
// each step's reflections recomputed.  Bound by the float64 atomics on the
// edges, 12 per tet a particle visits (12 per step before: 125 -> 53 us at 2e6
// particles and 5 steps).
__global__ void __launch_bounds__(kBlock) k_adjoint_leavers(StepArgs<double> a, AdjArgs b, unsigned *next_ctr) {
    if (blockIdx.x == 0) clear_counters(next_ctr);
    take_leavers(a, [&](int64_t p) {
        if (p >= b.end) return;
        int T = b.tet[p];
        double l[4], v[3], xb[3], vb[3];
        l[0] = 0.0;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            l[k + 1] = b.lam[k][p];
            v[k] = b.v[k][p];
            xb[k] = b.xb[k][p];
            vb[k] = b.vb[k][p];
        }
        auto row_at = [&](int j, double cf[kRowReals]) {
            const double *pr = b.parts + (int64_t)T * (kRowParts<1> * kRowReals);
#pragma unroll
            for (int c = 0; c < kRowReals; ++c) cf[c] = row_entry<1>(pr + c, kRowReals, &b.c[j], &b.s[j]);
        };
#pragma unroll 1
        for (int j = 0; j < b.nsteps; ++j) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                b.s_lam[j][k][p] = l[k + 1];
                b.s_v[j][k][p] = v[k];
            }
            b.s_tet[j][p] = T;
            if (j == b.nsteps - 1) break;   // the last step's end is not needed
            double cf[kRowReals], gm[9], gr[9], dl[4], t[4];
            row_at(j, cf);
            load_rows<double, false>(a, T, gm, gr);
            const double x[3] = {l[1], l[2], l[3]};
            gather_boris(cf, gm, x, a.h, v);
            if (increments(gr, v, a.dt_r, 1.0, l, dl, t)) {
#pragma unroll
                for (int k = 1; k < 4; ++k) l[k] = t[k];
            } else {
                double d[3] = {a.dt_r * v[0], a.dt_r * v[1], a.dt_r * v[2]};
                double R[9] = {1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0};   // not needed yet
                T = walk<double, true>(a, T, l, d, v, R);
            }
        }
        // the gradient sums of consecutive steps in one tet go to its edges together
        double gc[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0}, gs[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        auto flush = [&]() {
            double re[6], im[6];
            edge_sums(gc, re);
            edge_sums(gs, im);
            const int32_t *ed = push_row_edges(a.gpush + (int64_t)T * PushRow<double>::kStride);
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                unsafeAtomicAdd(&b.grad_e[2 * (int64_t)ed[e]], re[e]);
                unsafeAtomicAdd(&b.grad_e[2 * (int64_t)ed[e] + 1], im[e]);
                gc[e] = gs[e] = 0.0;
            }
        };
#pragma unroll 1
        for (int j = b.nsteps - 1; j >= 0; --j) {
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                l[k + 1] = b.s_lam[j][k][p];
                v[k] = b.s_v[j][k][p];
            }
            const int at = b.s_tet[j][p];
            if (at != T || j == b.nsteps - 1) {
                if (j < b.nsteps - 1) flush();
                T = at;
            }
            double cf[kRowReals], gm[9], gr[9], dl[4], t[4];
            row_at(j, cf);
            load_rows<double, false>(a, T, gm, gr);
            // reflections of this step (identity unless the particle left its tet)
            double R[9] = {1.0, 0.0, 0.0, 0.0, 1.0, 0.0, 0.0, 0.0, 1.0};
            const double x[3] = {l[1], l[2], l[3]};
            double out[3] = {v[0], v[1], v[2]};
            gather_boris(cf, gm, x, a.h, out);
            if (!increments(gr, out, a.dt_r, 1.0, l, dl, t)) {
                double d[3] = {a.dt_r * out[0], a.dt_r * out[1], a.dt_r * out[2]};
                double lw[4] = {0.0, l[1], l[2], l[3]};
                walk<double, true>(a, T, lw, d, out, R);
            }
            double w[6];
            adjoint_step(cf, gm, gr, l, v, a.h, a.dt_r, R, xb, vb, w);
#pragma unroll
            for (int e = 0; e < 6; ++e) {
                gc[e] = fma(w[e], b.c[j], gc[e]);
                gs[e] = fma(w[e], -b.s[j], gs[e]);
            }
        }
        flush();
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            b.vb[k][p] = vb[k];
            b.xb[k][p] = xb[k];
        }
    });
}

// ------------------------------------------------------------------ point location
// Particles enter as Cartesian points; the step works on (tet, barycentrics).
// A point is located by a straight walk from the centroid of a start tet (the
// caller's hint, else the tet of the point's start-grid cell) to the point:
// each hop leaves the current tet through the face whose barycentric reaches
// zero first and enters the neighbour.  The final barycentrics are recomputed
// from the point itself, lam_k = grad l_k . (x - r_0) (k = 1..3).  A walk that
// reaches a boundary face or the hop cap marks the point as not located; a
// point within kLocateTol (in barycentric terms) outside a boundary face counts
// as on it, so points on the domain boundary are located.
constexpr int kLocateHopCap = 4096;
constexpr double kLocateTol = 1e-10;

struct GridArgs {
    const int32_t *cell;
    double lo[3], inv[3];
    int dims[3];
};

__global__ void __launch_bounds__(kBlock) k_locate(int64_t n, const double *__restrict__ x0,
                                                   const double *__restrict__ x1, const double *__restrict__ x2,
                                                   const int32_t *__restrict__ hint, int64_t nt,
                                                   const TetTopo *__restrict__ topo, const double *__restrict__ grad,
                                                   const double *__restrict__ xyz, GridArgs G,
                                                   double *__restrict__ lam1, double *__restrict__ lam2,
                                                   double *__restrict__ lam3, int32_t *__restrict__ tet,
                                                   unsigned *__restrict__ fails, int fixed) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const double x[3] = {x0[p], x1[p], x2[p]};
    bool ok = isfinite(x[0]) && isfinite(x[1]) && isfinite(x[2]);
    int T = hint ? hint[p] : -1;
    if (ok && (unsigned)T >= (unsigned)nt) {
        int64_t c[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const double f = floor((x[d] - G.lo[d]) * G.inv[d]);
            c[d] = (int64_t)fmin(fmax(f, 0.0), (double)(G.dims[d] - 1));
        }
        T = G.cell[c[0] + (int64_t)G.dims[0] * (c[1] + (int64_t)G.dims[1] * c[2])];
    }
    if (ok) {
        // start at the centroid of T (barycentrics 1/4) with displacement x - centroid
        double l[4] = {0.25, 0.25, 0.25, 0.25}, d[3] = {x[0], x[1], x[2]};
        {
            const TetTopo tp = topo[T];
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int c = 0; c < 3; ++c) d[c] -= 0.25 * xyz[3 * (int64_t)tp.v[k] + c];
        }
        int hops = 0;
        for (;;) {
            const double *gp = grad + (int64_t)T * 12;
            const TetTopo tp = topo[T];
            double dl[4];
#pragma unroll
            for (int k = 1; k < 4; ++k) dl[k] = gp[3 * k] * d[0] + gp[3 * k + 1] * d[1] + gp[3 * k + 2] * d[2];
            dl[0] = -(dl[1] + dl[2] + dl[3]);
            double smin = 1.0;
            int kmin = -1;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (dl[k] < 0.0 && l[k] + dl[k] < 0.0 && !(tp.n[k] < 0 && l[k] + dl[k] >= -kLocateTol)) {
                    const double sk = l[k] > 0.0 ? l[k] / (-dl[k]) : 0.0;
                    if (kmin < 0 || sk < smin) {
                        smin = sk;
                        kmin = k;
                    }
                }
            if (kmin < 0) break;
            int nb = -1;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (k == kmin) nb = tp.n[k];
            if (nb < 0 || ++hops > kLocateHopCap) {
                ok = false;
                break;
            }
            double lc[4], sum = 0.0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                lc[k] = (k == kmin) ? 0.0 : fmax(l[k] + smin * dl[k], 0.0);
                sum += lc[k];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) d[c] -= smin * d[c];
            const TetTopo tn = topo[nb];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double v = 0.0;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (tp.v[i] == tn.v[j]) v = lc[i] / sum;
                l[j] = v;
            }
            T = nb;
        }
    }
    if (!ok) {
        tet[p] = -1;
        atomicAdd(fails, 1u);
        return;
    }
    const TetTopo tp = topo[T];
    const double *r0 = xyz + 3 * (int64_t)tp.v[0];
    const double dx[3] = {x[0] - r0[0], x[1] - r0[1], x[2] - r0[2]};
    const double *gp = grad + (int64_t)T * 12;
    const double l1 = gp[3] * dx[0] + gp[4] * dx[1] + gp[5] * dx[2];
    const double l2 = gp[6] * dx[0] + gp[7] * dx[1] + gp[8] * dx[2];
    const double l3 = gp[9] * dx[0] + gp[10] * dx[1] + gp[11] * dx[2];
    if (fixed) {
        uint32_t u[3];
        fix_round3(l1, l2, l3, u);
        reinterpret_cast<uint32_t *>(lam1)[p] = u[0];
        reinterpret_cast<uint32_t *>(lam2)[p] = u[1];
        reinterpret_cast<uint32_t *>(lam3)[p] = u[2];
    } else {
        lam1[p] = l1;
        lam2[p] = l2;
        lam3[p] = l3;
    }
    tet[p] = T;
}

// x = sum_k lam_k r_k of every particle (lam_0 = 1 - lam_1 - lam_2 - lam_3).
__global__ void __launch_bounds__(kBlock) k_positions(int64_t n, int64_t nt, const double *__restrict__ lam1,
                                                      const double *__restrict__ lam2, const double *__restrict__ lam3,
                                                      const int32_t *__restrict__ tet, const TetTopo *__restrict__ topo,
                                                      const double *__restrict__ xyz, double *__restrict__ x0,
                                                      double *__restrict__ x1, double *__restrict__ x2,
                                                      unsigned *__restrict__ status, int fixed) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    const int T = tet[p];
    if ((unsigned)T >= (unsigned)nt) {
        atomicOr(status, (unsigned)ETPIC_DEV_BADTET);
        x0[p] = x1[p] = x2[p] = NAN;
        return;
    }
    const double a1 = lam_at(lam1, p, fixed), a2 = lam_at(lam2, p, fixed), a3 = lam_at(lam3, p, fixed);
    const double l[4] = {1.0 - a1 - a2 - a3, a1, a2, a3};
    const TetTopo tp = topo[T];
    double x[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) x[c] += l[k] * xyz[3 * (int64_t)tp.v[k] + c];
    x0[p] = x[0];
    x1[p] = x[1];
    x2[p] = x[2];
}

// ------------------------------------------------------------------ vertex charge
// A block takes kChargePer * 256 consecutive particles: sums per run of equal
// tets, and the runs' vertices added up in a table in LDS (open addressing, the
// key is the vertex) before they go to memory, since neighbouring tets share
// most of their vertices.  A vertex that finds no place within four steps is
// added directly, so any order of the particles is right.
//   Bound by the atomics on the vertices, which all XCDs share: four per run of
// a wavefront before, one per vertex of a block now, and an XCD's blocks take
// one contiguous range.  1.23e6 particles, 11 per tet: 29.0 -> 13.2 us (1 or 4
// per thread: 13.7, 14.1); 5e7, 109 per tet: 315 -> 261 us and 1e8, 1600 per
// tet: 750 -> 571 us, both against a kernel that carried a run over 4 or 16
// slices of a wavefront (8 per thread: 311, 658).
constexpr int kChargePer = 2;
constexpr int kChargeSlots = 512;

__global__ void __launch_bounds__(kBlock) k_charge(int64_t n, int64_t nt, const double *__restrict__ lam1,
                                                   const double *__restrict__ lam2, const double *__restrict__ lam3,
                                                   const int32_t *__restrict__ tet, const TetTopo *__restrict__ topo,
                                                   double qw, double *__restrict__ rho, unsigned *status, int fixed) {
    __shared__ double s_sum[kChargeSlots];
    __shared__ int s_vert[kChargeSlots];
    for (int i = threadIdx.x; i < kChargeSlots; i += kBlock) {
        s_vert[i] = -1;
        s_sum[i] = 0.0;
    }
    const int64_t first = (int64_t)xcd_block(blockIdx.x, gridDim.x) * (kChargePer * kBlock) + threadIdx.x;
    int t[kChargePer];
    double x[kChargePer][3];
#pragma unroll
    for (int s = 0; s < kChargePer; ++s) {
        const int64_t p = first + s * kBlock;
        t[s] = -1;
        x[s][0] = x[s][1] = x[s][2] = 0.0;
        if (p < n) {
            t[s] = tet[p];
            x[s][0] = lam_at(lam1, p, fixed);
            x[s][1] = lam_at(lam2, p, fixed);
            x[s][2] = lam_at(lam3, p, fixed);
        }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < kChargePer; ++s) {
        int T = t[s];
        if (first + s * kBlock < n && (unsigned)T >= (unsigned)nt) {
            atomicOr(status, (unsigned)ETPIC_DEV_BADTET);
            T = -1;
        }
        const WaveRuns r = wave_runs(T);
        const bool end = r.lane == r.run_end && T >= 0;
        TetTopo tp;
        if (end) tp = topo[T];
        double l[4];
        l[0] = 0.0;
#pragma unroll
        for (int k = 1; k < 4; ++k) l[k] = run_total(T >= 0 ? x[s][k - 1] : 0.0, r);
        if (end) {
            // lam_0 sums to the run's length less the other three sums
            l[0] = (double)(r.run_end - r.head_lane + 1) - l[1] - l[2] - l[3];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int v = tp.v[k];
                unsigned h = ((unsigned)v * 2654435761u) >> 23;   // the top 9 bits
                int tries = 4;
                for (; tries > 0; --tries, h = (h + 1) & (kChargeSlots - 1)) {
                    const int was = atomicCAS(&s_vert[h], -1, v);
                    if (was == -1 || was == v) break;
                }
                if (tries > 0)
                    unsafeAtomicAdd(&s_sum[h], l[k]);
                else
                    unsafeAtomicAdd(&rho[v], qw * l[k]);
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kChargeSlots; i += kBlock)
        if (s_vert[i] >= 0) unsafeAtomicAdd(&rho[s_vert[i]], qw * s_sum[i]);
}

// ------------------------------------------------------------------ continuity residual
// r_k = sum_{e incident} (+dG_e if k is the head, -dG_e if the tail) - (rho_new_k - rho_old_k).
// out[0] = max |r|, out[1] = max |rho_old| as the bit patterns of non-negative doubles
// (which order like unsigned integers).  The maxima propagate NaN: a non-finite
// dG or rho makes the residual NaN (whose bit pattern orders above +inf), never
// a passing number.
__device__ __forceinline__ double max_keep_nan(double a, double b) { return (a != a || a > b) ? a : b; }

// |r_k| of vertex k: the signed sum of its incident edge currents (CSR of
// (edge << 1 | head) codes) minus its change of charge.
__device__ __forceinline__ double gauss_r(int64_t k, const int32_t *__restrict__ ptr,
                                          const int32_t *__restrict__ code, const double *__restrict__ dG,
                                          const double *__restrict__ rho_new, const double *__restrict__ rho_old) {
    // eight edges at a time, their loads in flight together (an inner vertex has about
    // fourteen), summed in the order of the list: a chain of two loads per eight edges
    // where there was one per edge (22,000 vertices: 14.2 -> 4.8 us)
    const int32_t i0 = ptr[k], i1 = ptr[k + 1];
    const double change = rho_new[k] - rho_old[k];
    double div = 0.0;
    for (int32_t i = i0; i < i1; i += 8) {
        int32_t c[8];
        double g[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) c[j] = code[min(i + j, i1 - 1)];
#pragma unroll
        for (int j = 0; j < 8; ++j) g[j] = dG[c[j] >> 1];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (i + j < i1) div += (c[j] & 1) ? g[j] : -g[j];
    }
    return fabs(div - change);
}

// max|r| and max|rho_old| in two passes without atomics: k_gauss_part leaves
// one pair per block (grid-stride over the vertices, kResBlocks blocks at
// most) in part[2 * block], k_gauss_final reduces the pairs into out[0..1].
// Every partial is written before it is read, so nothing needs clearing
// between calls.
constexpr int kResBlocks = 1024;

__global__ void __launch_bounds__(kBlock) k_gauss_part(int64_t nv, const int32_t *__restrict__ ptr,
                                                       const int32_t *__restrict__ code,
                                                       const double *__restrict__ dG,
                                                       const double *__restrict__ rho_new,
                                                       const double *__restrict__ rho_old, double *__restrict__ part) {
    double r = 0.0, p = 0.0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < nv; k += (int64_t)gridDim.x * blockDim.x) {
        r = max_keep_nan(gauss_r(k, ptr, code, dG, rho_new, rho_old), r);
        p = max_keep_nan(fabs(rho_old[k]), p);
    }
    for (int off = 32; off > 0; off >>= 1) {
        r = max_keep_nan(r, __shfl_xor(r, off));
        p = max_keep_nan(p, __shfl_xor(p, off));
    }
    __shared__ double wr[kBlock / 64], wp[kBlock / 64];
    if ((threadIdx.x & 63) == 0) {
        wr[threadIdx.x >> 6] = r;
        wp[threadIdx.x >> 6] = p;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) {
            r = max_keep_nan(r, wr[w]);
            p = max_keep_nan(p, wp[w]);
        }
        part[2 * blockIdx.x] = r;
        part[2 * blockIdx.x + 1] = p;
    }
}

__global__ void __launch_bounds__(kBlock) k_gauss_final(const double *__restrict__ part, int nblk,
                                                        double *__restrict__ out) {
    double r = 0.0, p = 0.0;
    for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
        r = max_keep_nan(r, part[2 * b]);
        p = max_keep_nan(p, part[2 * b + 1]);
    }
    for (int off = 32; off > 0; off >>= 1) {
        r = max_keep_nan(r, __shfl_xor(r, off));
        p = max_keep_nan(p, __shfl_xor(p, off));
    }
    __shared__ double wr[kBlock / 64], wp[kBlock / 64];
    if ((threadIdx.x & 63) == 0) {
        wr[threadIdx.x >> 6] = r;
        wp[threadIdx.x >> 6] = p;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) {
            r = max_keep_nan(r, wr[w]);
            p = max_keep_nan(p, wp[w]);
        }
        out[0] = r;
        out[1] = p;
    }
}

constexpr size_t kScratchDoubles = 2 * (size_t)kResBlocks + 2;

// ------------------------------------------------------------------ counting sort
__global__ void __launch_bounds__(kBlock) k_fill_u32(unsigned *__restrict__ x, int64_t n, unsigned val) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] = val;
}

// Four slices per wavefront, their loads in flight together: with one slice
// each the launch was bound by the rate at which wavefronts start.
constexpr int kHistSlices = 4;
__global__ void __launch_bounds__(kBlock) k_hist(int64_t n, int64_t nt, const int32_t *__restrict__ tet,
                                                 unsigned *__restrict__ count, unsigned *status) {
    const int64_t p0 = (int64_t)blockIdx.x * (kHistSlices * kBlock) + threadIdx.x;
    int T[kHistSlices];
#pragma unroll
    for (int i = 0; i < kHistSlices; ++i) T[i] = p0 + i * kBlock < n ? tet[p0 + i * kBlock] : -1;
#pragma unroll
    for (int i = 0; i < kHistSlices; ++i) {
        if (p0 + i * kBlock < n && (unsigned)T[i] >= (unsigned)nt) {
            atomicOr(status, (unsigned)ETPIC_DEV_BADTET);
            T[i] = -1;
        }
        const WaveRuns r = wave_runs(T[i]);
        if (r.head && T[i] >= 0) atomicAdd(&count[T[i]], (unsigned)(r.run_end - r.lane + 1));
    }
}

constexpr int kScanTile = 1024;   // elements per block in the block-local scan (4 per thread)

// sum over tets of count^2 (count = particles in the tet), accumulated into
// *out: sum(count^2) / N_p is the mean length of the same-tet run a particle
// belongs to, which picks the slices per wavefront of the particle kernel.
__global__ void __launch_bounds__(kBlock) k_run_stat(int64_t nt, const unsigned *__restrict__ count,
                                                     unsigned long long *__restrict__ out) {
    unsigned long long c2 = 0;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < nt; t += (int64_t)gridDim.x * blockDim.x) {
        const unsigned long long c = count[t];
        c2 += c * c;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) c2 += __shfl_xor(c2, off);
    __shared__ unsigned long long s_part[kBlock / 64];
    if ((threadIdx.x & 63) == 0) s_part[threadIdx.x >> 6] = c2;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long sum = 0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) sum += s_part[w];
        if (sum) atomicAdd(out, sum);
    }
}

// Exclusive scan of each 1024-element tile in place; tile totals to sums[].
__global__ void __launch_bounds__(kBlock) k_scan_tiles(unsigned *__restrict__ x, int64_t n,
                                                       unsigned *__restrict__ sums) {
    __shared__ unsigned s_wave[kBlock / 64];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
    unsigned v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = (base + i < n) ? x[base + i] : 0u;
    unsigned tsum = v[0] + v[1] + v[2] + v[3];
    // inclusive wave scan of the thread sums
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    unsigned inc = tsum;
    for (int off = 1; off < 64; off <<= 1) {
        unsigned y = __shfl_up(inc, off);
        if (lane >= off) inc += y;
    }
    if (lane == 63) s_wave[wid] = inc;
    __syncthreads();
    unsigned wpre = 0;
    for (int w = 0; w < wid; ++w) wpre += s_wave[w];
    unsigned run = wpre + inc - tsum;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (base + i < n) x[base + i] = run;
        run += v[i];
    }
    if (threadIdx.x == kBlock - 1) sums[blockIdx.x] = wpre + inc;
}

// Adds to each tile's elements the totals of the tiles before it (one block
// per tile; it sums those totals itself, which spares a launch for their scan).
__global__ void __launch_bounds__(kBlock) k_scan_add(unsigned *__restrict__ x, int64_t n,
                                                     const unsigned *__restrict__ sums) {
    __shared__ unsigned s_wave[kBlock / 64];
    unsigned before = 0;
    for (unsigned i = threadIdx.x; i < blockIdx.x; i += kBlock) before += sums[i];
    for (int off = 32; off > 0; off >>= 1) before += __shfl_xor(before, off);
    if ((threadIdx.x & 63) == 0) s_wave[threadIdx.x >> 6] = before;
    __syncthreads();
    before = 0;
    for (int w = 0; w < kBlock / 64; ++w) before += s_wave[w];
    const int64_t base = (int64_t)blockIdx.x * kScanTile + threadIdx.x * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (base + i < n) x[base + i] += before;
}

// hsrc / hdst (optional): nh further arrays of length n at stride n, of the
// velocity type, moved with the particles (the downshifted history).
template <typename Real>
__global__ void __launch_bounds__(kBlock) k_scatter(int64_t n, int64_t nt, const int32_t *__restrict__ tet,
                                                    unsigned *__restrict__ cursor, etpic_particles src,
                                                    etpic_particles dst, const Real *__restrict__ hsrc = nullptr,
                                                    Real *__restrict__ hdst = nullptr, int nh = 0, int fixed = 0) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int T = -1;
    if (p < n) {
        T = tet[p];
        if ((unsigned)T >= (unsigned)nt) T = -1;
    }
    // one cursor atomic per run of equal tet; lanes of a run keep their order
    const WaveRuns r = wave_runs(T);
    unsigned base = 0;
    if (r.head && T >= 0) base = atomicAdd(&cursor[T], (unsigned)(r.run_end - r.lane + 1));
    base = __shfl(base, r.head_lane);
    if (T < 0) return;
    const unsigned q = base + (unsigned)(r.lane - r.head_lane);
    dst.tet[q] = T;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        if (fixed)
            reinterpret_cast<uint32_t *>(dst.lam[k])[q] = reinterpret_cast<const uint32_t *>(src.lam[k])[p];
        else
            dst.lam[k][q] = src.lam[k][p];
        static_cast<Real *>(dst.vel[k])[q] = static_cast<const Real *>(src.vel[k])[p];
    }
    if (src.id && dst.id) dst.id[q] = src.id[p];
    for (int i = 0; i < nh; ++i) hdst[(int64_t)i * n + q] = hsrc[(int64_t)i * n + p];
}

// ------------------------------------------------------------------ field update
// Implicit envelope field step on the Whitney edge space (a side path of the
// particle step, timed separately).  Eliminating B~ from the envelope Maxwell
// equations (Formulation: the curl equations with the carrier) and testing
// with W1 gives
//   M e'' + 2 j w M e' + (K - w^2 M) e = f,   f = -e^{-j w t} g''
// (M = eps-mass, K = curl-curl, g the deposited edge DoFs of G), stepped with
// Newmark-beta (gamma = 1/2, beta = 1/4, Formulation) in acceleration form:
//   A a_{n+1} = f_{n+1} - M (2 j w v* - w^2 u*) - K u*,   A = (1 + j w dt - w^2 dt^2/4) M + (dt^2/4) K,
//   u* = u + dt v + dt^2/4 a,  v* = v + dt/2 a,  u_{n+1} = u* + dt^2/4 a_{n+1},  v_{n+1} = v* + dt/2 a_{n+1}.
// A is complex symmetric: Jacobi-preconditioned COCG.  The face envelope
// follows the discrete envelope Faraday law (j w + d/dt) b = -C e with the
// trapezoidal rule.
__device__ __forceinline__ double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
__device__ __forceinline__ double2 cdiv(double2 a, double2 b) {
    const double d = b.x * b.x + b.y * b.y;
    return make_double2((a.x * b.x + a.y * b.y) / d, (a.y * b.x - a.x * b.y) / d);
}

constexpr int kRowLanes = 8;   // lanes per CSR row

struct FieldCsr {
    int64_t ne;
    const int32_t *rowptr, *col;
    const double *M, *K;
    const uint8_t *dir;
};

// Row-wise (M x1)_i and (K x2)_i with kRowLanes lanes per row, summed across
// those lanes; every lane of the group returns the totals.  A lane's entries
// are taken kRowBatch at a time with their loads in flight together (a row of
// the edge matrices has about 18 entries;
// batches of 3 need more registers than two blocks of 1024 have), and added in
// the row's order.
constexpr int kRowBatch = 2;

__device__ __forceinline__ void csr_row2(const FieldCsr &S, int64_t row, int sub, const double2 *__restrict__ x1,
                                         const double2 *__restrict__ x2, double2 &m1, double2 &k2) {
    m1 = make_double2(0.0, 0.0);
    k2 = make_double2(0.0, 0.0);
    if (row < S.ne) {
        const int32_t j0 = S.rowptr[row], j1 = S.rowptr[row + 1];
        for (int32_t j = j0 + sub; j < j1; j += kRowBatch * kRowLanes) {
            int32_t at[kRowBatch], c[kRowBatch];
            double mv[kRowBatch], kv[kRowBatch];
            double2 a[kRowBatch], b[kRowBatch];
#pragma unroll
            for (int i = 0; i < kRowBatch; ++i) {
                at[i] = min(j + i * kRowLanes, j1 - 1);
                c[i] = S.col[at[i]];
            }
#pragma unroll
            for (int i = 0; i < kRowBatch; ++i) {
                mv[i] = S.M[at[i]];
                kv[i] = S.K[at[i]];
            }
#pragma unroll
            for (int i = 0; i < kRowBatch; ++i) {
                a[i] = x1[c[i]];
                b[i] = x2[c[i]];
            }
#pragma unroll
            for (int i = 0; i < kRowBatch; ++i)
                if (j + i * kRowLanes < j1) {
                    m1.x += mv[i] * a[i].x;
                    m1.y += mv[i] * a[i].y;
                    k2.x += kv[i] * b[i].x;
                    k2.y += kv[i] * b[i].y;
                }
        }
    }
#pragma unroll
    for (int off = kRowLanes / 2; off > 0; off >>= 1) {
        m1.x += __shfl_xor(m1.x, off);
        m1.y += __shfl_xor(m1.y, off);
        k2.x += __shfl_xor(k2.x, off);
        k2.y += __shfl_xor(k2.y, off);
    }
}

// block-level sum of up to 4 doubles into partial[blockIdx.x * 4 + k]
__device__ __forceinline__ void block_sum4(double v[4], double *partial) {
    __shared__ double sh[kBlock / 64][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) sh[wid][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 4) {
        double s = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) s += sh[w][threadIdx.x];
        partial[blockIdx.x * 4 + threadIdx.x] = s;
    }
}

// y = alpha M x + beta K x (complex alpha, real beta)
__global__ void __launch_bounds__(kBlock) k_field_spmv(FieldCsr S, double2 alpha, double beta,
                                                       const double2 *__restrict__ x, double2 *__restrict__ y) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t row = t / kRowLanes;
    const int sub = (int)(t % kRowLanes);
    double2 m, k;
    csr_row2(S, row, sub, x, x, m, k);
    if (row < S.ne && sub == 0) y[row] = cadd(cmul(alpha, m), cscale(k, beta));
}

// Newmark predictor: us = u + dt v + dt^2/4 a, vs = v + dt/2 a, w = 2 j w vs - w^2 us
__global__ void __launch_bounds__(kBlock) k_nm_predict(int64_t ne, const double2 *__restrict__ u,
                                                       const double2 *__restrict__ v, const double2 *__restrict__ a,
                                                       double2 *__restrict__ us, double2 *__restrict__ vs,
                                                       double2 *__restrict__ w, double dt, double omega) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ne) return;
    const double2 ui = u[i], vi = v[i], ai = a[i];
    const double2 usi = cadd(cadd(ui, cscale(vi, dt)), cscale(ai, 0.25 * dt * dt));
    const double2 vsi = cadd(vi, cscale(ai, 0.5 * dt));
    us[i] = usi;
    vs[i] = vsi;
    w[i] = csub(cmul(make_double2(0.0, 2.0 * omega), vsi), cscale(usi, omega * omega));
}

// rhs = f - M w - K us with f = -e^{-j w t} g'';  boundary rows 0
__global__ void __launch_bounds__(kBlock) k_nm_rhs(FieldCsr S, const double2 *__restrict__ w,
                                                   const double2 *__restrict__ us, const double *__restrict__ gdd,
                                                   double c, double s, double2 *__restrict__ rhs) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t row = t / kRowLanes;
    const int sub = (int)(t % kRowLanes);
    double2 m, k;
    csr_row2(S, row, sub, w, us, m, k);
    if (row < S.ne && sub == 0) {
        double2 r = make_double2(0.0, 0.0);
        if (!S.dir[row]) {
            const double g = gdd ? gdd[row] : 0.0;
            // -e^{-j w t} g = -(c - j s) g
            r = make_double2(-c * g - m.x - k.x, s * g - m.y - k.y);
        }
        rhs[row] = r;
    }
}

// COCG start: x = 0, r = rhs, z = Dinv r, p = q = 0; partials r.z (re, im),
// |r|^2, |b|^2 (= |r|^2); clears the done flag and the iteration count.
__global__ void __launch_bounds__(kBlock) k_cocg_init(int64_t ne, const double2 *__restrict__ rhs,
                                                      const double2 *__restrict__ dinv, double2 *__restrict__ x,
                                                      double2 *__restrict__ r, double2 *__restrict__ z,
                                                      double2 *__restrict__ p, double2 *__restrict__ q,
                                                      double *__restrict__ partial, double *__restrict__ sc) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (i < ne) {
        const double2 ri = rhs[i];
        const double2 zi = cmul(dinv[i], ri);
        x[i] = make_double2(0.0, 0.0);
        r[i] = ri;
        z[i] = zi;
        p[i] = make_double2(0.0, 0.0);
        q[i] = make_double2(0.0, 0.0);
        const double2 rz = cmul(ri, zi);
        v[0] = rz.x;
        v[1] = rz.y;
        v[2] = ri.x * ri.x + ri.y * ri.y;
        v[3] = v[2];
    }
    if (i == 0) {
        sc[6] = 0.0;   // (the meeting of the resident solve)
        sc[10] = 0.0;
        sc[11] = 0.0;
    }
    block_sum4(v, partial);
}

// faces: (1 + j w dt/2) b_new = (1 - j w dt/2) b - dt/2 C (u + u_new), u_new = us + dt^2/4 x,
// (C e)_f = e_ab + e_bc - e_ac
__global__ void __launch_bounds__(kBlock) k_nm_faraday(int64_t nf, const int32_t *__restrict__ fe,
                                                       const double2 *__restrict__ u, const double2 *__restrict__ us,
                                                       const double2 *__restrict__ x, double2 *__restrict__ b,
                                                       double dt, double omega) {
    const int64_t f = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= nf) return;
    const double q = 0.25 * dt * dt;
    double2 cs = make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const int32_t e = fe[3 * f + k];
        const double2 sum = cadd(u[e], cadd(us[e], cscale(x[e], q)));
        cs = (k == 2) ? csub(cs, sum) : cadd(cs, sum);
    }
    const double2 num = csub(cmul(make_double2(1.0, -0.5 * omega * dt), b[f]), cscale(cs, 0.5 * dt));
    b[f] = cdiv(num, make_double2(1.0, 0.5 * omega * dt));
}

// u = us + dt^2/4 x, v = vs + dt/2 x, a = x
__global__ void __launch_bounds__(kBlock) k_nm_correct(int64_t ne, const double2 *__restrict__ us,
                                                       const double2 *__restrict__ vs, const double2 *__restrict__ x,
                                                       double2 *__restrict__ u, double2 *__restrict__ v,
                                                       double2 *__restrict__ a, double dt) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ne) return;
    const double2 xi = x[i];
    u[i] = cadd(us[i], cscale(xi, 0.25 * dt * dt));
    v[i] = cadd(vs[i], cscale(xi, 0.5 * dt));
    a[i] = xi;
}

// ---- non-solenoidal field of the quasi-Helmholtz split (eq. ns_equation):
// Jacobi-preconditioned CG on the nodal operator D^T [*eps] D, real because
// the operator is real (the carrier phase multiplies the solution).
struct NsCsr {
    int64_t nv;
    const int32_t *rowptr, *col;
    const double *S;
};

// (S x)_row with kRowLanes lanes per row, as csr_row2 (a nodal row has about
// 15 entries, one batch of 8 x 2).
__device__ __forceinline__ double ns_row(const NsCsr &S, int64_t row, int sub, const double *__restrict__ x) {
    double sx = 0.0;
    if (row < S.nv) {
        const int32_t j0 = S.rowptr[row], j1 = S.rowptr[row + 1];
        for (int32_t j = j0 + sub; j < j1; j += 2 * kRowLanes) {
            const int32_t j2 = min(j + kRowLanes, j1 - 1);
            const int32_t c = S.col[j], c2 = S.col[j2];
            const double v = S.S[j], v2 = S.S[j2], xc = x[c], xc2 = x[c2];
            sx += v * xc;
            if (j + kRowLanes < j1) sx += v2 * xc2;
        }
    }
#pragma unroll
    for (int off = kRowLanes / 2; off > 0; off >>= 1) sx += __shfl_xor(sx, off);
    return sx;
}

// The CG kernels run on at most kNsBlocks blocks (grid-stride loops), so that
// every block can sum all block partials of the previous kernel itself, in
// the same fixed order: the scalars of the iteration need no kernel of their
// own and no cross-block synchronisation.  Partials: 4 doubles per block.
// Scalars sc (written by thread 0 of block 0 only, read by the next kernel):
// sc[0], sc[1] rho = r.z of even / odd iterations, sc[8] |r|^2, sc[9] |b|^2,
// sc[10] done flag, sc[11] iterations taken.
constexpr int kNsBlocks = 512;
constexpr int kNsThreads = 1024;   // product kernels: 16 wavefronts per block, enough rows in flight for one pass
constexpr int kNsVecThreads = 256; // vector kernels (one node per lane): more, smaller blocks

// Block-level sum of 4 doubles into partial[blk * 4 + k].
__device__ __forceinline__ void ns_block_sum4(double v[4], double *partial, unsigned blk = blockIdx.x) {
    __shared__ double sh[kNsThreads / 64][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) sh[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 4) {
        double t = 0.0;
        for (int w = 0; w < (int)(blockDim.x / 64); ++w) t += sh[w][threadIdx.x];
        partial[blk * 4 + threadIdx.x] = t;
    }
}

// This thread's share of the sums of the nb partials: their loads go out with
// the other loads of the kernel, all_sum4 adds the shares up.
__device__ __forceinline__ void fetch_sum4(int64_t nb, const double *__restrict__ partial, double v[4]) {
    int64_t b = threadIdx.x;
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = b < nb ? partial[4 * b + k] : 0.0;
    for (b += blockDim.x; b < nb; b += blockDim.x)
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] += partial[4 * b + k];
}

// Every thread gets the sums of the block's shares (fixed order).
__device__ __forceinline__ void all_sum4(double v[4], double tot[4]) {
    __shared__ double sh[kNsThreads / 64][4];
    __shared__ double res[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        for (int off = 32; off > 0; off >>= 1) v[k] += __shfl_xor(v[k], off);
    if ((threadIdx.x & 63) == 0)
#pragma unroll
        for (int k = 0; k < 4; ++k) sh[threadIdx.x >> 6][k] = v[k];
    __syncthreads();
    if (threadIdx.x < 4) {
        double t = 0.0;
        for (int w = 0; w < (int)(blockDim.x / 64); ++w) t += sh[w][threadIdx.x];
        res[threadIdx.x] = t;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 4; ++k) tot[k] = res[k];
}

using etpic::SolveWatch;

// Every kSolveReport-th launch reports, and the last: a store to host memory
// keeps its kernel from ending for 1-2 us.
constexpr int kSolveReport = 4;

__device__ __forceinline__ void report(SolveWatch *watch, int k, bool done, bool last, double r2, double b2) {
    if (last) {
        watch->r2 = r2;
        watch->b2 = b2;
    }
    if (last || k % kSolveReport == 0)
        __hip_atomic_store(&watch->word, 2ull * (k + 1) + (done ? 1 : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Right-hand side of a nodal solve: b = -(gs (D^T G + rho0) + D^T w_comp)
// at the nodes off the wall, 0 on it; every pointer may be NULL.  w is a
// complex edge vector of which component comp (0 re, 1 im) is taken.
struct NsRhs {
    const double *G, *rho0;
    double gs;
    const double2 *w;
    int comp;
};

// (D^T G)_i sums +-G over the edges at node i (+ where i is the head).
__device__ __forceinline__ double ns_rhs(int64_t i, const int32_t *__restrict__ ptr, const int32_t *__restrict__ code,
                                         const NsRhs &R, const uint8_t *__restrict__ wall) {
    if (wall[i]) return 0.0;
    const int32_t i0 = ptr[i], i1 = ptr[i + 1];
    double div = R.rho0 ? R.rho0[i] : 0.0;
    double dw = 0.0;
    for (int32_t k = i0; k < i1; k += 8) {   // eight edges' loads in flight together
        int32_t c[8];
        double g[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) c[j] = code[min(k + j, i1 - 1)];
        if (R.G) {
#pragma unroll
            for (int j = 0; j < 8; ++j) g[j] = R.G[c[j] >> 1];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (k + j < i1) div += (c[j] & 1) ? g[j] : -g[j];
        }
        if (R.w) {
            const double *w = reinterpret_cast<const double *>(R.w) + R.comp;
#pragma unroll
            for (int j = 0; j < 8; ++j) g[j] = w[2 * (int64_t)(c[j] >> 1)];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (k + j < i1) dw += (c[j] & 1) ? g[j] : -g[j];
        }
    }
    return -(R.gs * div + dw);
}

// Cold start: x = 0, r = b, z = Dinv b, p = q = 0; partials r.z, 0, |r|^2, |b|^2.
__global__ void __launch_bounds__(kNsVecThreads) k_ns_start(int64_t nv, const int32_t *__restrict__ ptr,
                                                     const int32_t *__restrict__ code, NsRhs R,
                                                     const uint8_t *__restrict__ wall,
                                                     const double *__restrict__ dinv, double *__restrict__ x,
                                                     double *__restrict__ r, double *__restrict__ z,
                                                     double *__restrict__ p, double *__restrict__ q,
                                                     double *__restrict__ partial, double *__restrict__ sc) {
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += (int64_t)gridDim.x * blockDim.x) {
        const double b = ns_rhs(i, ptr, code, R, wall);
        const double zi = dinv[i] * b;
        x[i] = 0.0;
        r[i] = b;
        z[i] = zi;
        p[i] = 0.0;
        q[i] = 0.0;
        v[0] += b * zi;
        v[2] += b * b;
        v[3] += b * b;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc[6] = 0.0;   // (the meeting of the resident solve)
        sc[10] = 0.0;
        sc[11] = 0.0;
    }
    ns_block_sum4(v, partial);
}

// Warm start from the x left by the previous solve: r = b - S x, z = Dinv r,
// p = q = 0; partials r.z, 0, |r|^2, |b|^2.  kRowLanes lanes per row.
__global__ void __launch_bounds__(kNsThreads) k_ns_start_warm(NsCsr S, const int32_t *__restrict__ ptr,
                                                          const int32_t *__restrict__ code, NsRhs R,
                                                          const uint8_t *__restrict__ wall,
                                                          const double *__restrict__ dinv,
                                                          const double *__restrict__ x, double *__restrict__ r,
                                                          double *__restrict__ z, double *__restrict__ p,
                                                          double *__restrict__ q, double *__restrict__ partial,
                                                          double *__restrict__ sc) {
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t / kRowLanes < S.nv; t += stride) {
        const int64_t row = t / kRowLanes;
        const int sub = (int)(t % kRowLanes);
        const double sx = ns_row(S, row, sub, x);
        if (sub == 0) {
            const double b = ns_rhs(row, ptr, code, R, wall);
            const double ri = b - sx;
            const double zi = dinv[row] * ri;
            r[row] = ri;
            z[row] = zi;
            p[row] = 0.0;
            q[row] = 0.0;
            v[0] += ri * zi;
            v[2] += ri * ri;
            v[3] += b * b;
        }
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc[6] = 0.0;   // (the meeting of the resident solve)
        sc[10] = 0.0;
        sc[11] = 0.0;
    }
    ns_block_sum4(v, partial);
}

// Iteration k, first half.  From the partials of the previous update (or of
// the start, k = 0): |r|^2 and rho_new = r.z; done once |r|^2 <= tol^2 |b|^2
// (or not finite, or b = 0), then every block returns.  Otherwise beta = rho_new /
// rho_old, p = z + beta p and q = A p = A z + beta q (the direction update
// folded into the product, so no separate pass over p is needed), with the
// partials of p . q.  check_only: the convergence test alone (after the last
// allowed iteration).  Returns at once if an earlier launch found convergence.
// The first pass over the rows does not need the scalars: its product runs
// before the sums of the partials, whose loads are in flight meanwhile.
__global__ void __launch_bounds__(kNsThreads) k_ns_apply(NsCsr S, double *__restrict__ sc,
                                                     const double *__restrict__ z, double *__restrict__ p,
                                                     double *__restrict__ q, const double *__restrict__ pin,
                                                     int64_t nb_in, double *__restrict__ pout, int k, double tol2,
                                                     int check_only, SolveWatch *watch) {
    const bool stopped = sc[10] != 0.0;
    const double ro = sc[(k + 1) & 1], bb = sc[9];
    double v[4], tot[4];
    fetch_sum4(nb_in, pin, v);
    const unsigned blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t t = (int64_t)blk * blockDim.x + threadIdx.x;
    const int sub = (int)(t % kRowLanes);
    int64_t row = t / kRowLanes;
    double zr = 0.0, pr = 0.0, qr = 0.0;
    if (row < S.nv && sub == 0) {
        zr = z[row];
        pr = p[row];
        qr = q[row];
    }
    double az = ns_row(S, row, sub, z);
    all_sum4(v, tot);
    if (stopped) return;
    const double b2 = k == 0 ? tot[3] : bb;
    const double r2 = tot[2], rn = tot[0];
    const bool done = b2 == 0.0 || !(r2 > tol2 * b2);   // no source: x = 0, done
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc[8] = r2;
        if (k == 0) sc[9] = b2;
        sc[k & 1] = rn;
        sc[10] = done ? 1.0 : 0.0;
        sc[11] = (double)k;
        report(watch, k, done, done || check_only, r2, b2);
    }
    if (done || check_only) return;
    const double be = (k == 0 || ro == 0.0) ? 0.0 : rn / ro;
    v[0] = v[1] = v[2] = v[3] = 0.0;
    for (;;) {
        if (row < S.nv && sub == 0) {
            const double pn = zr + be * pr;
            const double qn = az + be * qr;
            p[row] = pn;
            q[row] = qn;
            v[0] += pn * qn;
        }
        t += stride;
        row = t / kRowLanes;
        if (row >= S.nv) break;   // (the lanes of a row leave together)
        if (sub == 0) {
            zr = z[row];
            pr = p[row];
            qr = q[row];
        }
        az = ns_row(S, row, sub, z);
    }
    ns_block_sum4(v, pout, blk);
}

// Iteration k, second half: alpha = rho_new / (p . q) from the partials of the
// product; x += alpha p, r -= alpha q, z = Dinv r, with the partials of r . z
// and |r|^2.  Returns at once if the first half found convergence.
__global__ void __launch_bounds__(kNsVecThreads) k_ns_update(int64_t nv, const double *__restrict__ sc,
                                                      const double *__restrict__ dinv, const double *__restrict__ p,
                                                      const double *__restrict__ q, double *__restrict__ x,
                                                      double *__restrict__ r, double *__restrict__ z,
                                                      const double *__restrict__ pin, int64_t nb_in,
                                                      double *__restrict__ pout, int k) {
    const bool stopped = sc[10] != 0.0;
    const double rho = sc[k & 1];
    double v[4], tot[4];
    fetch_sum4(nb_in, pin, v);
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double pi = 0.0, qi = 0.0, xi = 0.0, ri = 0.0, di = 0.0;
    if (i < nv) {
        pi = p[i];
        qi = q[i];
        xi = x[i];
        ri = r[i];
        di = dinv[i];
    }
    all_sum4(v, tot);
    if (stopped) return;
    const double pq = tot[0];
    const double al = pq != 0.0 ? rho / pq : 0.0;
    v[0] = v[1] = v[2] = v[3] = 0.0;
    while (i < nv) {
        x[i] = xi + al * pi;
        ri = ri - al * qi;
        r[i] = ri;
        const double zi = di * ri;
        z[i] = zi;
        v[0] += ri * zi;
        v[2] += ri * ri;
        i += (int64_t)gridDim.x * blockDim.x;
        if (i < nv) {
            pi = p[i];
            qi = q[i];
            xi = x[i];
            ri = r[i];
            di = dinv[i];
        }
    }
    ns_block_sum4(v, pout);
}

// ---- COCG of the field step, two launches per iteration on at most
// kNsBlocks blocks, so that every block sums the previous launch's partials
// itself (as the nodal CG): no scalar kernels, the convergence test on the
// device.  Scalars sc: [0..1], [2..3] rho = r^T z (complex, unconjugated) of
// even / odd iterations, [8] |r|^2, [9] |b|^2, [10] done, [11] iterations.
//
// Iteration k, first half: done once |r_k|^2 <= tol^2 |b|^2 (or b = 0, or not
// finite); beta = rho_k / rho_{k-1}, p = z + beta p, q = A z + beta q (= A p,
// the direction update folded into the product), partials p^T q.
// A = alpha M + beta_k K.  check_only: the test alone.
// As k_ns_apply, the first pass's product runs before the sums.  An XCD's
// blocks take contiguous rows, which share the entries of z they read.
__global__ void __launch_bounds__(kNsThreads, 8) k_cocg_apply(FieldCsr S, double2 alpha, double beta_k,
                                                       double *__restrict__ sc, const double2 *__restrict__ z,
                                                       double2 *__restrict__ p, double2 *__restrict__ q,
                                                       const double *__restrict__ pin, int64_t nb_in,
                                                       double *__restrict__ pout, int k, double tol2,
                                                       int check_only, SolveWatch *watch) {
    const bool stopped = sc[10] != 0.0;
    const int o = 2 * ((k + 1) & 1);
    const double2 ro = make_double2(sc[o], sc[o + 1]);
    const double bb = sc[9];
    double v[4], tot[4];
    fetch_sum4(nb_in, pin, v);
    const unsigned blk = xcd_block(blockIdx.x, gridDim.x);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t t = (int64_t)blk * blockDim.x + threadIdx.x;
    const int sub = (int)(t % kRowLanes);
    int64_t row = t / kRowLanes;
    const double2 zero = make_double2(0.0, 0.0);
    double2 zr = zero, pr = zero, qr = zero, m, kk;
    if (row < S.ne && sub == 0) {
        zr = z[row];
        pr = p[row];
        qr = q[row];
    }
    csr_row2(S, row, sub, z, z, m, kk);
    all_sum4(v, tot);
    if (stopped) return;
    const double b2 = k == 0 ? tot[3] : bb;
    const double r2 = tot[2];
    const double2 rn = make_double2(tot[0], tot[1]);
    const bool done = b2 == 0.0 || !(r2 > tol2 * b2);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        sc[8] = r2;
        if (k == 0) sc[9] = b2;
        sc[2 * (k & 1)] = rn.x;
        sc[2 * (k & 1) + 1] = rn.y;
        sc[10] = done ? 1.0 : 0.0;
        sc[11] = (double)k;
        report(watch, k, done, done || check_only, r2, b2);
    }
    if (done || check_only) return;
    const double2 be = (k == 0 || (ro.x == 0.0 && ro.y == 0.0)) ? zero : cdiv(rn, ro);
    v[0] = v[1] = v[2] = v[3] = 0.0;
    for (;;) {
        if (row < S.ne && sub == 0) {
            const double2 pn = cadd(zr, cmul(be, pr));
            const double2 qn = cadd(cadd(cmul(alpha, m), cscale(kk, beta_k)), cmul(be, qr));
            p[row] = pn;
            q[row] = qn;
            const double2 pq = cmul(pn, qn);
            v[0] += pq.x;
            v[1] += pq.y;
        }
        t += stride;
        row = t / kRowLanes;
        if (row >= S.ne) break;   // (the lanes of a row leave together)
        if (sub == 0) {
            zr = z[row];
            pr = p[row];
            qr = q[row];
        }
        csr_row2(S, row, sub, z, z, m, kk);
    }
    ns_block_sum4(v, pout, blk);
}

// Iteration k, second half: alpha = rho_k / (p^T q); x += alpha p, r -= alpha q,
// z = Dinv r; partials r^T z (re, im), |r|^2.
__global__ void __launch_bounds__(kNsVecThreads) k_cocg_update(int64_t ne, const double *__restrict__ sc,
                                                        const double2 *__restrict__ dinv,
                                                        const double2 *__restrict__ p, const double2 *__restrict__ q,
                                                        double2 *__restrict__ x, double2 *__restrict__ r,
                                                        double2 *__restrict__ z, const double *__restrict__ pin,
                                                        int64_t nb_in, double *__restrict__ pout, int k) {
    const bool stopped = sc[10] != 0.0;
    const double2 rho = make_double2(sc[2 * (k & 1)], sc[2 * (k & 1) + 1]);
    double v[4], tot[4];
    fetch_sum4(nb_in, pin, v);
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const double2 zero = make_double2(0.0, 0.0);
    double2 pi = zero, qi = zero, xi = zero, ri = zero, di = zero;
    if (i < ne) {
        pi = p[i];
        qi = q[i];
        xi = x[i];
        ri = r[i];
        di = dinv[i];
    }
    all_sum4(v, tot);
    if (stopped) return;
    const double2 pq = make_double2(tot[0], tot[1]);
    const double2 al = (pq.x == 0.0 && pq.y == 0.0) ? zero : cdiv(rho, pq);
    v[0] = v[1] = v[2] = v[3] = 0.0;
    while (i < ne) {
        x[i] = cadd(xi, cmul(al, pi));
        ri = csub(ri, cmul(al, qi));
        r[i] = ri;
        const double2 zi = cmul(di, ri);
        z[i] = zi;
        const double2 rz = cmul(ri, zi);
        v[0] += rz.x;
        v[1] += rz.y;
        v[2] += ri.x * ri.x + ri.y * ri.y;
        i += (int64_t)gridDim.x * blockDim.x;
        if (i < ne) {
            pi = p[i];
            qi = q[i];
            xi = x[i];
            ri = r[i];
            di = dinv[i];
        }
    }
    ns_block_sum4(v, pout);
}

// ---- The same two iterations in one launch, for systems whose rows fit the
// chip at once (kResRows rows per block, one block per CU): matrix rows and the
// vectors but z stay in registers, and an iteration costs its gather of z and
// two exchanges of block sums instead of two launches that load everything
// again.
//
// Block sums are exchanged through `slots`, three sets of kResMaxBlocks x
// kResStride words taken in turn.  A word that no block has written yet holds
// kSlotEmpty (a NaN that the sums never are, see slot_bits); a block writes its
// words of set s % 3 in exchange s, reads all blocks' words of it, and then
// empties its own words of the set before, which every block has read by then
// and which is next written two exchanges later.  Words and z are written and
// read at agent scope; a block's z entries have left its CU before its word does.
//
// All blocks have to run at once.  They meet at a counter first: a block that
// has waited kMeetTicks for the others (another stream's kernels may hold the
// CUs) closes the meeting, unless it has become complete, and every block leaves,
// those that start later too; nothing has been written by then and the host takes
// the iterations by launches.  Past the meeting every block is resident, so each wait
// ends; it is bounded all the same (kSlotSpins polls, seconds).
//
// Bound by latency: two exchanges of 2.5 us and a gather of z past the L2s.
// Gauss-law solve on 9,261 nodes 12.6 -> 7.2 us per iteration (37 blocks),
// field solve on 59,900 edges 23.6 -> 10.9 us (234 blocks); two steps of the
// coupled loop on that mesh 6.63 -> 2.88 ms.  z read plainly after a fence that
// invalidates the caches: 3.4 ms; block sums packed 8 to a line: 3.1 ms, one to
// 32 or 128 bytes: 2.94 ms; more than one row per four lanes would need more
// registers than 16 wavefronts have.
constexpr int kResThreads = 1024, kResLanes = 4, kResRows = kResThreads / kResLanes;
constexpr int kResMaxBlocks = 256;             // one per CU
constexpr int kResEntries = 5;                 // entries per lane held in registers
constexpr int kResVals = 4;
constexpr int kResStride = 8;                   // words from block to block
constexpr size_t kResSlots = (size_t)3 * kResMaxBlocks * kResStride;
constexpr unsigned kMeetClosed = 0x80000000u;
constexpr long long kMeetTicks = 50000;        // 0.5 ms of the 100 MHz counter (OneLaunchTrials: what follows it)
constexpr unsigned kSlotSpins = 1u << 22;
constexpr unsigned long long kSlotEmpty = 0xfff8c0de00000001ull;

__device__ __forceinline__ unsigned long long slot_bits(double x) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    return b == kSlotEmpty ? 0x7ff8000000000000ull : b;
}

__device__ __forceinline__ void agent_store(unsigned long long *at, unsigned long long x) {
    __hip_atomic_store(at, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ unsigned long long agent_load(const unsigned long long *at) {
    return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// this wavefront's stores are where other XCDs see them
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Sum over the wavefront, in every lane: DPP row shifts and broadcasts, lane 63's total read back.
__device__ __forceinline__ double wave_sum(double x) {
    x += dpp_get<0x111, 0xf>(x);   // row_shr:1, 2, 4, 8
    x += dpp_get<0x112, 0xf>(x);
    x += dpp_get<0x114, 0xf>(x);
    x += dpp_get<0x118, 0xf>(x);
    x += dpp_get<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
    x += dpp_get<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
    const long long b = __double_as_longlong(x);
    return __longlong_as_double(((long long)__builtin_amdgcn_readlane((int)(b >> 32), 63) << 32) |
                                (unsigned)__builtin_amdgcn_readlane((int)(b & 0xffffffffll), 63));
}

struct ResShared {
    double wave[kResThreads / 64][kResVals];
    double tot[kResVals];
    int ok;
};

// The meeting; false: it was closed before all blocks came.  Also empties
// this block's words of all three sets.
__device__ __forceinline__ bool res_meet(ResShared &sh, unsigned *meet, unsigned long long *slots) {
    const unsigned nb = gridDim.x;
    if (threadIdx.x < 3 * kResVals)
        agent_store(&slots[((size_t)(threadIdx.x / kResVals) * kResMaxBlocks + blockIdx.x) * kResStride +
                           threadIdx.x % kResVals], kSlotEmpty);
    if (threadIdx.x == 0) {   // (the same wavefront as the stores above)
        stores_done();
        unsigned seen = __hip_atomic_fetch_add(meet, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
        const long long t0 = wall_clock64();
        while (seen < nb) {   // (a closed meeting reads as >= kMeetClosed)
            __builtin_amdgcn_s_sleep(1);
            seen = __hip_atomic_load(meet, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (seen < nb && wall_clock64() - t0 > kMeetTicks) {
                unsigned was = seen;
                if (__hip_atomic_compare_exchange_strong(meet, &was, was | kMeetClosed, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    was |= kMeetClosed;
                seen = was;
            }
        }
        sh.ok = seen == nb;
    }
    __syncthreads();
    return sh.ok != 0;
}

// Sums of v over all blocks, to every thread; false (in every thread): a wait ran out.
template <int kN>
__device__ __forceinline__ bool res_exchange(ResShared &sh, unsigned long long *slots, unsigned s, double v[kN]) {
    const unsigned nb = gridDim.x;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < kN; ++k) v[k] = wave_sum(v[k]);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < kN; ++k) sh.wave[wid][k] = v[k];
    stores_done();   // z
    __syncthreads();
    if (wid == 0) {
        unsigned long long *set = slots + (size_t)(s % 3) * kResMaxBlocks * kResStride;
        unsigned long long *before = slots + (size_t)((s + 2) % 3) * kResMaxBlocks * kResStride;
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            const double t = wave_sum(lane < kResThreads / 64 ? sh.wave[lane][k] : 0.0);
            if (lane == 0) agent_store(&set[blockIdx.x * kResStride + k], slot_bits(t));
        }
        double sum[kN];
#pragma unroll
        for (int k = 0; k < kN; ++k) sum[k] = 0.0;
        // a lane's words of up to four blocks are requested together
        constexpr int kPer = kResMaxBlocks / 64;
        unsigned long long got[kPer][kN];
        unsigned spins = 0;
        for (;;) {
            bool have = true;
#pragma unroll
            for (int i = 0; i < kPer; ++i)
                if (i * 64 < (int)nb)
#pragma unroll
                    for (int k = 0; k < kN; ++k)
                        got[i][k] = agent_load(&set[min(i * 64u + lane, nb - 1) * kResStride + k]);
#pragma unroll
            for (int i = 0; i < kPer; ++i)
                if (i * 64 < (int)nb)
#pragma unroll
                    for (int k = 0; k < kN; ++k) have = have && got[i][k] != kSlotEmpty;
            if (__all(have) || ++spins > kSlotSpins) break;
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i)
#pragma unroll
            for (int k = 0; k < kN; ++k)
                if (i * 64u + lane < nb) sum[k] += __longlong_as_double((long long)got[i][k]);
#pragma unroll
        for (int k = 0; k < kN; ++k) {
            sum[k] = wave_sum(sum[k]);
            if (lane == 0) sh.tot[k] = sum[k];
        }
        if (lane < kResVals) agent_store(&before[blockIdx.x * kResStride + lane], kSlotEmpty);
        if (lane == 0) sh.ok = spins <= kSlotSpins;
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kN; ++k) v[k] = sh.tot[k];
    return sh.ok != 0;
}

// A block whose wait ran out leaves without its rows of the result: the host
// must not take block 0's report for the whole.
__device__ __forceinline__ void give_up(SolveWatch *watch) {
    if (threadIdx.x == 0) __hip_atomic_store(&watch->gave_up, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ double quad_sum(double x) {   // over the kResLanes lanes of a row
    x += dpp_get<0xb1, 0xf>(x);   // quad_perm 1, 0, 3, 2
    x += dpp_get<0x4e, 0xf>(x);   // quad_perm 2, 3, 0, 1
    return x;
}

__device__ __forceinline__ double load_z(const double *z, int64_t i) {
    return __longlong_as_double((long long)agent_load(reinterpret_cast<const unsigned long long *>(z) + i));
}

__device__ __forceinline__ void store_z(double *z, int64_t i, double x) {
    agent_store(reinterpret_cast<unsigned long long *>(z) + i, (unsigned long long)__double_as_longlong(x));
}

// CG of the Gauss-law solve from what k_ns_start or k_ns_start_warm left.
__global__ void __launch_bounds__(kResThreads) k_ns_resident(NsCsr S, double *sc, const double *dinv, double *x,
                                                             const double *r, double *z, const double *pin,
                                                             int64_t nb_in, unsigned long long *slots, double tol2,
                                                             int max_iter, SolveWatch *watch) {
    __shared__ ResShared sh;
    const int64_t row = (int64_t)blockIdx.x * kResRows + threadIdx.x / kResLanes;
    const int sub = threadIdx.x % kResLanes;
    const bool mine = row < S.nv, owner = mine && sub == 0;
    int32_t j0 = 0, j1 = 0;
    if (mine) {
        j0 = S.rowptr[row];
        j1 = S.rowptr[row + 1];
    }
    int32_t c[kResEntries];
    double a[kResEntries];
#pragma unroll
    for (int i = 0; i < kResEntries; ++i) {
        const int32_t j = j0 + sub + i * kResLanes;
        c[i] = mine ? (int32_t)row : 0;   // (an absent entry: 0 times the row's own z)
        a[i] = 0.0;
        if (j < j1) {
            c[i] = S.col[j];
            a[i] = S.S[j];
        }
    }
    double xi = 0.0, ri = 0.0, zi = 0.0, di = 0.0, pi = 0.0, qi = 0.0;
    if (owner) {
        xi = x[row];
        ri = r[row];
        zi = z[row];
        di = dinv[row];
    }
    double v[4], tot[4];
    fetch_sum4(nb_in, pin, v);
    all_sum4(v, tot);
    if (!res_meet(sh, reinterpret_cast<unsigned *>(sc + 6), slots)) return;
    const double b2 = tot[3];
    double r2 = tot[2], rn = tot[0], ro = 0.0;
    bool done;
    int k = 0;
    for (unsigned s = 0;; ++k, s += 2) {
        done = b2 == 0.0 || !(r2 > tol2 * b2);   // no source: x = 0, done
        if (done || k >= max_iter) break;
        const double be = (k == 0 || ro == 0.0) ? 0.0 : rn / ro;
        double az = 0.0;
        double g[kResEntries];
#pragma unroll
        for (int i = 0; i < kResEntries; ++i) g[i] = load_z(z, c[i]);
#pragma unroll
        for (int i = 0; i < kResEntries; ++i) az += a[i] * g[i];
        for (int32_t j = j0 + sub + kResEntries * kResLanes; j < j1; j += kResLanes) az += S.S[j] * load_z(z, S.col[j]);
        az = quad_sum(az);
        double w[2] = {0.0, 0.0};
        if (owner) {
            pi = zi + be * pi;
            qi = az + be * qi;
            w[0] = pi * qi;
        }
        if (!res_exchange<1>(sh, slots, s, w)) return give_up(watch);
        const double al = w[0] != 0.0 ? rn / w[0] : 0.0;
        w[0] = w[1] = 0.0;
        if (owner) {
            xi += al * pi;
            ri -= al * qi;
            zi = di * ri;
            store_z(z, row, zi);
            w[0] = ri * zi;
            w[1] = ri * ri;
        }
        if (!res_exchange<2>(sh, slots, s + 1, w)) return give_up(watch);
        ro = rn;
        rn = w[0];
        r2 = w[1];
    }
    if (owner) x[row] = xi;
    if (blockIdx.x == 0 && threadIdx.x == 0) report(watch, k, done, true, r2, b2);
}

// COCG of the field step from what k_cocg_init left.
__global__ void __launch_bounds__(kResThreads) k_cocg_resident(FieldCsr S, double2 alpha, double beta_k, double *sc,
                                                               const double2 *dinv, double2 *x, const double2 *r,
                                                               double2 *z, const double *pin, int64_t nb_in,
                                                               unsigned long long *slots, double tol2, int max_iter,
                                                               SolveWatch *watch) {
    __shared__ ResShared sh;
    const int64_t row = (int64_t)blockIdx.x * kResRows + threadIdx.x / kResLanes;
    const int sub = threadIdx.x % kResLanes;
    const bool mine = row < S.ne, owner = mine && sub == 0;
    double *zs = reinterpret_cast<double *>(z);
    int32_t j0 = 0, j1 = 0;
    if (mine) {
        j0 = S.rowptr[row];
        j1 = S.rowptr[row + 1];
    }
    int32_t c[kResEntries];
    double am[kResEntries], ak[kResEntries];
#pragma unroll
    for (int i = 0; i < kResEntries; ++i) {
        const int32_t j = j0 + sub + i * kResLanes;
        c[i] = mine ? (int32_t)row : 0;
        am[i] = ak[i] = 0.0;
        if (j < j1) {
            c[i] = S.col[j];
            am[i] = S.M[j];
            ak[i] = S.K[j];
        }
    }
    const double2 zero = make_double2(0.0, 0.0);
    double2 xi = zero, ri = zero, zi = zero, di = zero, pi = zero, qi = zero;
    if (owner) {   // (x starts from zero)
        ri = r[row];
        zi = z[row];
        di = dinv[row];
    }
    double v[4], tot[4];
    fetch_sum4(nb_in, pin, v);
    all_sum4(v, tot);
    if (!res_meet(sh, reinterpret_cast<unsigned *>(sc + 6), slots)) return;
    const double b2 = tot[3];
    double r2 = tot[2];
    double2 rn = make_double2(tot[0], tot[1]), ro = zero;
    bool done;
    int k = 0;
    for (unsigned s = 0;; ++k, s += 2) {
        done = b2 == 0.0 || !(r2 > tol2 * b2);
        if (done || k >= max_iter) break;
        const double2 be = (k == 0 || (ro.x == 0.0 && ro.y == 0.0)) ? zero : cdiv(rn, ro);
        double2 m = zero, kk = zero;
        double2 g[kResEntries];
#pragma unroll
        for (int i = 0; i < kResEntries; ++i)
            g[i] = make_double2(load_z(zs, 2 * (int64_t)c[i]), load_z(zs, 2 * (int64_t)c[i] + 1));
#pragma unroll
        for (int i = 0; i < kResEntries; ++i) {
            m.x += am[i] * g[i].x;
            m.y += am[i] * g[i].y;
            kk.x += ak[i] * g[i].x;
            kk.y += ak[i] * g[i].y;
        }
        for (int32_t j = j0 + sub + kResEntries * kResLanes; j < j1; j += kResLanes) {
            const int64_t cj = S.col[j];
            const double mv = S.M[j], kv = S.K[j], zx = load_z(zs, 2 * cj), zy = load_z(zs, 2 * cj + 1);
            m.x += mv * zx;
            m.y += mv * zy;
            kk.x += kv * zx;
            kk.y += kv * zy;
        }
        m = make_double2(quad_sum(m.x), quad_sum(m.y));
        kk = make_double2(quad_sum(kk.x), quad_sum(kk.y));
        double w[3] = {0.0, 0.0, 0.0};
        if (owner) {
            pi = cadd(zi, cmul(be, pi));
            qi = cadd(cadd(cmul(alpha, m), cscale(kk, beta_k)), cmul(be, qi));
            const double2 pq = cmul(pi, qi);
            w[0] = pq.x;
            w[1] = pq.y;
        }
        if (!res_exchange<2>(sh, slots, s, w)) return give_up(watch);
        const double2 pq = make_double2(w[0], w[1]);
        const double2 al = (pq.x == 0.0 && pq.y == 0.0) ? zero : cdiv(rn, pq);
        w[0] = w[1] = w[2] = 0.0;
        if (owner) {
            xi = cadd(xi, cmul(al, pi));
            ri = csub(ri, cmul(al, qi));
            zi = cmul(di, ri);
            store_z(zs, 2 * row, zi.x);
            store_z(zs, 2 * row + 1, zi.y);
            const double2 rz = cmul(ri, zi);
            w[0] = rz.x;
            w[1] = rz.y;
            w[2] = ri.x * ri.x + ri.y * ri.y;
        }
        if (!res_exchange<3>(sh, slots, s + 1, w)) return give_up(watch);
        ro = rn;
        rn = make_double2(w[0], w[1]);
        r2 = w[2];
    }
    if (owner) x[row] = xi;
    if (blockIdx.x == 0 && threadIdx.x == 0) report(watch, k, done, true, r2, b2);
}

// x_out = e^{-j w t} x on the nodes, e_out = e^{-j w t} D x on the edges
// (edge e from ev[2e] to ev[2e+1]), edc_out = D x (+ edc_add): the same field
// as real, unmodulated DoFs.  Every pointer may be NULL.
__global__ void __launch_bounds__(kBlock) k_ns_out(int64_t ne, int64_t nv, const int32_t *__restrict__ ev,
                                                   const double *__restrict__ x, double c, double s,
                                                   double2 *__restrict__ x_out, double2 *__restrict__ e_out,
                                                   double *__restrict__ edc_out, const double *__restrict__ edc_add) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if ((e_out || edc_out) && i < ne) {
        const double d = x[ev[2 * i + 1]] - x[ev[2 * i]];
        if (e_out) e_out[i] = make_double2(c * d, -s * d);
        if (edc_out) edc_out[i] = edc_add ? d + edc_add[i] : d;
    }
    if (x_out && i < nv) {
        const double xi = x[i];
        x_out[i] = make_double2(c * xi, -s * xi);
    }
}

// e_out = u + D (xr + j xi) on the edges (edge e from ev[2e] to ev[2e+1])
__global__ void __launch_bounds__(kBlock) k_ns_combine(int64_t ne, const int32_t *__restrict__ ev,
                                                       const double *__restrict__ xr, const double *__restrict__ xi,
                                                       const double2 *__restrict__ u, double2 *__restrict__ e_out) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ne) return;
    const int32_t a = ev[2 * i], b = ev[2 * i + 1];
    const double2 ui = u[i];
    e_out[i] = make_double2(ui.x + xr[b] - xr[a], ui.y + xi[b] - xi[a]);
}

// Source of the field step from the running path integral: with h1, h2 the
// values of G one and two steps back, gdd = (G - 2 h1 + h2) / dt^2 (written
// into gdd, which may be h2)
__global__ void __launch_bounds__(kBlock) k_em_gdd(int64_t ne, const double *__restrict__ G,
                                                   const double *__restrict__ h1, const double *h2, double *gdd,
                                                   double inv_dt2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ne) gdd[i] = ((G[i] - 2.0 * h1[i]) + h2[i]) * inv_dt2;
}

// history shift after a field step: h2 = h1, h1 = G
__global__ void __launch_bounds__(kBlock) k_em_shift(int64_t ne, const double *__restrict__ G, double *__restrict__ h1,
                                                     double *__restrict__ h2) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ne) {
        h2[i] = h1[i];
        h1[i] = G[i];
    }
}

// Solenoidal source: gs = gdd + Re m, m = [*eps] D y with D^T [*eps] D y =
// -D^T gdd at the inner nodes (gs may be gdd)
__global__ void __launch_bounds__(kBlock) k_sol_add(int64_t ne, const double *gdd, const double2 *__restrict__ m,
                                                    double *gs) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ne) gs[i] = gdd[i] + m[i].x;
}

// e += u: the solenoidal and non-solenoidal halves of the field summed
__global__ void __launch_bounds__(kBlock) k_em_add(int64_t ne, const double2 *__restrict__ u, double2 *__restrict__ e) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ne) {
        const double2 a = u[i], b = e[i];
        e[i] = make_double2(a.x + b.x, a.y + b.y);
    }
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

// =============================================================================== context

// Device memory carved from one caller-owned buffer.  Every table and scratch
// array the library keeps on the device lives in such a buffer (context
// workspace, mesh tables, field solver, Gauss-law solver, downshifted rows); the
// library itself allocates no device memory.  A layout takes its arrays in a
// fixed order, each on a 256-byte boundary; with a null base it only counts
// the bytes, which is how the size queries are answered.
struct Carve {
    char *base = nullptr;
    size_t cap = 0, used = 0;
    template <typename T>
    T *take(size_t count) {
        const size_t off = (used + 255) & ~(size_t)255;
        used = off + sizeof(T) * std::max<size_t>(count, 1);
        return base ? reinterpret_cast<T *>(base + off) : nullptr;
    }
};

// Device state of the field update (allocated by etpic_field_setup).
struct FieldState {
    bool ready = false;
    double dt = 0, omega = 0, eps = 0, mu = 0;
    int64_t ne = 0, nf = 0, nnz = 0;
    int32_t *rowptr = nullptr, *col = nullptr, *face_edge = nullptr;
    double *M = nullptr, *K = nullptr;
    uint8_t *dir = nullptr;
    double2 *dinv = nullptr;
    double2 *vec = nullptr;     // 9 work vectors of ne: us, vs, w, rhs, x, r, z, p, q
    double *partial = nullptr;  // two sets of 4 per block: nb blocks (the start, the update), then kNsBlocks
    double *sc = nullptr;       // 12 scalars of the iteration
    int64_t nb = 0;

    double2 *v(int k) const { return vec + (size_t)k * ne; }
    FieldCsr csr() const { return FieldCsr{ne, rowptr, col, M, K, dir}; }
    void release() { *this = FieldState(); }   // the memory is the caller's
};

// Device state of the non-solenoidal solve (allocated by etpic_ns_setup).
struct NsState {
    bool ready = false;
    double eps = 0;
    int64_t nv = 0, ne = 0, nnz = 0, n_wall = 0;
    int32_t *rowptr = nullptr, *col = nullptr, *ev = nullptr;
    double *S = nullptr, *dinv = nullptr;
    uint8_t *wall = nullptr;
    double *vec = nullptr;      // 8 vectors of nv: x, r, z, p, q, the solutions (re, im) of the correction and
                                // that of the source projection
    double *partial = nullptr;  // two sets of 4 per block (kNsBlocks blocks)
    double *sc = nullptr;       // 12 scalars of the iteration
    double *bzero = nullptr;    // 2*N_f zeros: the face envelope of a loop without external fields
    double *ezero = nullptr;    // 2*N_e zeros: its edge envelope

    double *v(int k) const { return vec + (size_t)k * nv; }
    NsCsr csr() const { return NsCsr{nv, rowptr, col, S}; }
    void release() { *this = NsState(); }   // the memory is the caller's
};

// Device pointers of one (snap[1] NULL) or three envelope snapshots; the dc
// DoFs are those of snap[0] (one snapshot) or snap[1] (three).
FieldPtrs field_ptrs(const etpic_fields *const snap[3], const double w[3], double c, double s) {
    FieldPtrs F{};
    const bool three = snap[1] != nullptr;
    for (int k = 0; k < 3; ++k) {
        const etpic_fields *f = three ? snap[k] : snap[0];
        F.e_env[k] = reinterpret_cast<const double2 *>(f->e_env);
        F.b_env[k] = reinterpret_cast<const double2 *>(f->b_env);
        F.w[k] = w[k];
    }
    const etpic_fields *dc = three ? snap[1] : snap[0];
    F.e_dc = dc->e_dc;
    F.b_dc = dc->b_dc;
    F.c = c;
    F.s = s;
    return F;
}

// One step of a multi-step call: the envelope snapshots (snap[1] NULL for
// one snapshot), their weights and the gather time.
struct StepPlan {
    const etpic_fields *snap[3];
    double w[3];
    double t;
};

// Launch of one kernel of a timed step sequence.  With events the kernel's
// own dispatch carries them (hipExtLaunchKernel binds e0 to its start and e1
// to its end), so timing inserts no marker packets between the kernels of a
// step; without, a plain launch.  Errors are left for hipGetLastError.
template <typename... P, typename... A>
void launch_timed(void (*k)(P...), dim3 grid, hipStream_t st, hipEvent_t e0, hipEvent_t e1, A... args) {
    if (e0)
        hipExtLaunchKernelGGL(k, grid, dim3(kBlock), 0, st, e0, e1, 0, static_cast<P>(args)...);
    else
        hipLaunchKernelGGL(k, grid, dim3(kBlock), 0, st, static_cast<P>(args)...);
}

struct etpic_ctx {
    int device = 0;
    etpic::HostMesh host;
    bool has_mesh = false;
    uint64_t mesh_hash = 0;   // hash of the uploaded mesh (particle checkpoints resume on it only)
    TetTopo *d_topo = nullptr;
    double *d_grad64 = nullptr;
    double *d_gpush64 = nullptr;     // nt rows of PushRow<double>
    float *d_gpush32 = nullptr;       // nt rows of PushRow<float>
    double *d_geo64 = nullptr;        // nt rows of GeoRow<double>
    float *d_geo32 = nullptr;         // nt rows of GeoRow<float>
    int32_t *d_tetface = nullptr;     // nt*4 face ids (face k opposite vertex k)
    void *d_coef = nullptr;          // nt*kCoefDoubles doubles: a step's CoefRow rows or a call's row parts
    double *d_coef_env = nullptr;    // nt*kEnvRow: wide rows (bound by etpic_ds_rows_bind)
    int32_t *d_v2e_ptr = nullptr;
    int32_t *d_v2e_code = nullptr;
    int32_t *d_e2s_ptr = nullptr;    // edge -> tet-slot CSR (ne+1)
    int32_t *d_e2s_slot = nullptr;   // its slots, 8 * tet + local edge (6 nt)
    double *d_tetG = nullptr;        // per-tet current slots (nt*8), cleared by a call's first kernel
    double *d_xyz = nullptr;         // 3*nv vertex coordinates
    int32_t *d_grid = nullptr;       // start tets of the point-location grid
    GridArgs grid{};
    bool has_ws = false;             // context workspace bound (etpic_workspace_bind)
    unsigned *d_status = nullptr;    // device status word
    unsigned *d_walk_queue = nullptr;  // kWalkQueueCap particle indices
    unsigned *d_slice_queue = nullptr; // kWalkQueueCap slice indices
    unsigned *d_walk_ctr = nullptr;    // kCtrSets sets of walk-queue counters, kCtrStride words each
    unsigned long long *d_red = nullptr;  // 2 words per block of the residual maxima
    double *d_scratch = nullptr;          // device address of `scratch` on this device
    // mean same-tet run length from the last sort (sum count^2 / N_p), read
    // back without blocking: the device word, its pinned host copy, the event
    // that marks the copy, and the value in use (0 until a sort has been seen)
    unsigned long long *d_runstat = nullptr;
    unsigned long long *h_runstat = nullptr;   // (and two words the residual's maxima are written into)
    SolveWatch *h_watch = nullptr;             // pinned, behind those
    etpic::OneLaunchTrials field_trials, ns_trials;   // (their solves take different numbers of blocks)
    hipEvent_t runstat_ev = nullptr;
    bool runstat_pending = false;
    int64_t runstat_n = 0;
    double run_len = 0.0;
    int last_slices = 0;             // slices per wavefront of the last particle-kernel launch
    unsigned *d_count = nullptr;     // nt+1 counting-sort counters
    unsigned *d_tilesum = nullptr;   // scan tile totals
    int64_t tiles = 0;
    FieldState field;
    NsState ns;
    // Timing of steps run with ETPIC_STEP_TIMING: per step a set of start and
    // stop events of its kernels, interval k = 0 coefficient pass, 1 particle
    // kernel, 2 walk, 3 edge gather of the per-tet sums, each bound to its
    // kernel's dispatch (launch_timed); `has` marks the intervals launched
    // (a call of several steps has one coefficient pass),
    // `sorting` whether the particle kernel also sorted (k_push_sort).  The
    // sets are created with the context (a fixed pool of kTimingSets, the
    // vectors reserved so that pointers to sets stay valid);
    // etpic_kernel_time returns the read sets to the pool.
    struct TimingSet {
        std::array<hipEvent_t, 8> ev{};
        unsigned has = 0;
        bool sorting = false;
        int steps = 1;   // steps of this launch; the first of a sorting one is the sorting step
    };
    std::vector<TimingSet> timing;
    std::vector<TimingSet> spare;
    // host-side systems built by a size query, kept for the setup call that follows
    std::unique_ptr<etpic::FieldSystem> field_pending;
    double field_pending_eps = 0, field_pending_mu = 0;
    std::unique_ptr<etpic::NsSystem> ns_pending;
    double ns_pending_eps = 0;

    int timing_events(TimingSet **ts, bool sorting = false) {
        if (spare.empty())
            return fail(ETPIC_EINVAL, "step timing: all %d event sets in use (etpic_kernel_time returns them)",
                        kTimingSets);
        timing.push_back(spare.back());
        spare.pop_back();
        timing.back().has = 0;
        timing.back().sorting = sorting;
        timing.back().steps = 1;
        *ts = &timing.back();
        return ETPIC_OK;
    }
    // A timed call that needs more sets than are left is refused before its
    // first launch: one that stopped between two launches would leave leavers
    // queued and currents in the tets' slots for the next call to find.
    int timing_room(uint32_t flags, int sets) const {
        if ((flags & (ETPIC_STEP_TIMING | ETPIC_STEP_TIMING_ALL)) && (size_t)sets > spare.size())
            return fail(ETPIC_EINVAL, "step timing: %d event sets needed, %zu of %d left (etpic_kernel_time returns them)",
                        sets, spare.size(), kTimingSets);
        return ETPIC_OK;
    }
    // start / stop event of interval k of a timing set (none without a set)
    static hipEvent_t ev_start(TimingSet *ts, int k) {
        if (!ts) return nullptr;
        ts->has |= 1u << k;
        return ts->ev[2 * k];
    }
    static hipEvent_t ev_stop(TimingSet *ts, int k) { return ts ? ts->ev[2 * k + 1] : nullptr; }

    template <typename Real>
    StepArgs<Real> step_args(const etpic_particles *p, const etpic_species *sp, double dt, double *dG,
                             double *rho) const {
        StepArgs<Real> a{};
        a.n = p->n;
        a.nt = host.nt;
        a.lam1 = p->lam[0];
        a.lam2 = p->lam[1];
        a.lam3 = p->lam[2];
        a.v0 = static_cast<Real *>(p->vel[0]);
        a.v1 = static_cast<Real *>(p->vel[1]);
        a.v2 = static_cast<Real *>(p->vel[2]);
        a.tet = p->tet;
        a.coef = static_cast<const Real *>(d_coef);
        a.gpush = gpush_table<Real>();
        a.geo = geo_table<Real>();
        a.grad = d_grad64;
        a.topo = d_topo;
        a.dG = dG;
        a.rho = rho;
        a.status = d_status;
        a.walk_queue = d_walk_queue;
        a.slice_queue = d_slice_queue;
        a.walk_ctr = d_walk_ctr;
        a.qw = sp->q * sp->w;
        a.h = (Real)(sp->q * dt / (2.0 * sp->m));
        a.dt_r = (Real)dt;
        return a;
    }

    // One step: carrier phase in float64 on the host (t = step*dt, argument
    // reduced by libm), per-tet coefficients, particle kernel, walk kernel.
    template <typename Real>
    int step(const etpic_particles *p, const etpic_species *sp, const etpic_fields *f, int64_t step, double dt,
             double omega, double *dG, double *rho, uint32_t flags, void *stream) {
        StepPlan plan{{f, nullptr, nullptr}, {1.0, 0.0, 0.0}, (double)step * dt};
        return run_steps<Real>(p, sp, &plan, 1, dt, omega, dG, rho, flags, stream);
    }

    // XCD-contiguous coefficient pass when an eighth of the edge and face DoFs
    // (complex edge and face envelopes, dc face DoFs) fits one 4 MB L2
    int coef_xcd() const { return (16 * host.ne + 24 * host.nf) / 8 <= (int64_t)4 << 20 ? 1 : 0; }

    FieldPtrs coef_fields(const StepPlan &plan, double omega) const {
        FieldPtrs F = field_ptrs(plan.snap, plan.w, std::cos(omega * plan.t), std::sin(omega * plan.t));
        F.xcd = coef_xcd();
        return F;
    }

    template <typename Real>
    int launch_coef(const StepPlan &plan, double omega, double *slots, hipStream_t s, TimingSet *ts = nullptr) {
        const int64_t nt = host.nt;
        const FieldPtrs F = coef_fields(plan, omega);
        hipEvent_t e0 = ev_start(ts, 0), e1 = ev_stop(ts, 0);
        Real *coef = static_cast<Real *>(d_coef);
        if (plan.snap[1])
            launch_timed(k_tet_coef<Real, 3, kCoefStep>, grid_for(2 * nt), s, e0, e1, nt, d_gpush64, d_tetface, F, coef,
                         slots);
        else
            launch_timed(k_tet_coef<Real, 1, kCoefStep>, grid_for(2 * nt), s, e0, e1, nt, d_gpush64, d_tetface, F, coef,
                         slots);
        HIP_TRY(hipGetLastError());
        return ETPIC_OK;
    }

    template <typename Real, bool kRho, bool kSort>
    bool launch_push(const StepArgs<Real> &a, int slices, int remap, hipStream_t st, TimingSet *ts = nullptr) {
        const int64_t n = a.n;
        hipEvent_t e0 = ev_start(ts, 1), e1 = ev_stop(ts, 1);
        if constexpr (std::is_same<Real, float>::value) {
            if (a.fixed) {
                switch (slices) {
                case 16:
                    if (kSort)
                        launch_timed(k_push_sort_slices_fixed<16, kRho>, grid_for((n + 15) / 16), st, e0, e1, a, remap);
                    else
                        launch_timed(k_push_slices_fixed<16, kRho>, grid_for((n + 15) / 16), st, e0, e1, a, remap);
                    break;
                case 4:
                    if (kSort)
                        launch_timed(k_push_sort_slices_fixed<4, kRho>, grid_for((n + 3) / 4), st, e0, e1, a, remap);
                    else
                        launch_timed(k_push_slices_fixed<4, kRho>, grid_for((n + 3) / 4), st, e0, e1, a, remap);
                    break;
                case 2:
                    if (!kSort && !kRho) {
                        launch_timed(k_push_pipe<true>, grid_for((n + 1) / 2), st, e0, e1, a, remap);
                        break;
                    }
                    [[fallthrough]];
                default:
                    if (kSort)
                        launch_timed(k_push_sort_fixed<kRho>, grid_for(n), st, e0, e1, a, remap);
                    else if (kRho)
                        launch_timed(k_push_rho_fixed, grid_for(n), st, e0, e1, a, remap);
                    else
                        launch_timed(k_push_fixed, grid_for(n), st, e0, e1, a, remap);
                    slices = 1;
                    break;
                }
                last_slices = slices;
                return slices == 2 || push_uses_slots<Real>(slices);
            }
        }
        switch (slices) {
        case 16:
            if (kSort)
                launch_timed(k_push_sort_slices<Real, 16, kRho>, grid_for((n + 15) / 16), st, e0, e1, a, remap);
            else
                launch_timed(k_push_slices<Real, 16, kRho>, grid_for((n + 15) / 16), st, e0, e1, a, remap);
            break;
        case 4:
            if (kSort)
                launch_timed(k_push_sort_slices<Real, 4, kRho>, grid_for((n + 3) / 4), st, e0, e1, a, remap);
            else
                launch_timed(k_push_slices<Real, 4, kRho>, grid_for((n + 3) / 4), st, e0, e1, a, remap);
            break;
        case 2:
            if constexpr (std::is_same<Real, float>::value) {
                if (!kSort && !kRho) {
                    launch_timed(k_push_pipe<false>, grid_for((n + 1) / 2), st, e0, e1, a, remap);
                    break;
                }
            }
            [[fallthrough]];
        default:
            if (kSort)
                launch_timed(k_push_sort<Real, kRho>, grid_for(n), st, e0, e1, a, remap);
            else if (kRho)
                launch_timed(k_push_rho<Real>, grid_for(n), st, e0, e1, a, remap);
            else
                launch_timed(k_push<Real>, grid_for(n), st, e0, e1, a, remap);
            slices = 1;
            break;
        }
        last_slices = slices;
        return slices == 2 || push_uses_slots<Real>(slices);
    }

    // Counting sort, first half: tet counts of src, the run-length statistic
    // for the slice choice (unless one is still in flight), and the exclusive
    // prefix sums of the counts in d_count (the scatter cursors).
    int sort_count(const etpic_particles *src, hipStream_t st) {
        const int64_t nt = host.nt, n = src->n, m = nt + 1;
        k_fill_u32<<<grid_for(m), kBlock, 0, st>>>(d_count, m, 0u);
        k_hist<<<grid_for((n + kHistSlices - 1) / kHistSlices), kBlock, 0, st>>>(n, nt, src->tet, d_count, d_status);
        if (!runstat_pending) {
            k_fill_u32<<<1, kBlock, 0, st>>>(reinterpret_cast<unsigned *>(d_runstat), 2, 0u);
            k_run_stat<<<(unsigned)std::min<int64_t>(grid_for(nt), 256), kBlock, 0, st>>>(nt, d_count, d_runstat);
            HIP_TRY(hipMemcpyAsync(h_runstat, d_runstat, sizeof(unsigned long long), hipMemcpyDeviceToHost, st));
            HIP_TRY(hipEventRecord(runstat_ev, st));
            runstat_pending = true;
            runstat_n = n;
        }
        k_scan_tiles<<<(unsigned)tiles, kBlock, 0, st>>>(d_count, m, d_tilesum);
        k_scan_add<<<(unsigned)tiles, kBlock, 0, st>>>(d_count, m, d_tilesum);
        HIP_TRY(hipGetLastError());
        return ETPIC_OK;
    }

    template <typename Real>
    int sort(const etpic_particles *src, const etpic_particles *dst, hipStream_t st, const Real *hsrc = nullptr,
             Real *hdst = nullptr, int nh = 0, int fixed = 0) {
        if (int r = sort_count(src, st)) return r;
        k_scatter<Real><<<grid_for(src->n), kBlock, 0, st>>>(src->n, host.nt, src->tet, d_count, *src, *dst, hsrc,
                                                              hdst, nh, fixed);
        HIP_TRY(hipGetLastError());
        return ETPIC_OK;
    }

    // the particle arrays of src become the ones read, p's the sorted ones written
    template <typename Real>
    void scatter_from(StepArgs<Real> &a, const etpic_particles *p, const etpic_particles *src) const {
        a.lam1 = src->lam[0];
        a.lam2 = src->lam[1];
        a.lam3 = src->lam[2];
        a.v0 = static_cast<Real *>(src->vel[0]);
        a.v1 = static_cast<Real *>(src->vel[1]);
        a.v2 = static_cast<Real *>(src->vel[2]);
        a.tet = src->tet;
        a.o_lam1 = p->lam[0];
        a.o_lam2 = p->lam[1];
        a.o_lam3 = p->lam[2];
        a.o_v0 = static_cast<Real *>(p->vel[0]);
        a.o_v1 = static_cast<Real *>(p->vel[1]);
        a.o_v2 = static_cast<Real *>(p->vel[2]);
        a.o_tet = p->tet;
        a.id = src->id;
        a.o_id = p->id;
        a.cursor = d_count;
    }

    // The call's per-tet sums onto the edges.
    int launch_edges(double *dG, hipStream_t st, TimingSet *ta, unsigned *ctr) {
        const int64_t ne = host.ne;
        const unsigned gb = (unsigned)std::min<int64_t>(grid_for(ne), 4096);
        launch_timed(k_slots_to_edges, gb, st, ev_start(ta, 3), ev_stop(ta, 3), ne, d_e2s_ptr, d_e2s_slot, d_tetG, dG, ctr);
        HIP_TRY(hipGetLastError());
        return ETPIC_OK;
    }

    // nsteps consecutive steps, step j at time plans[j].t with the envelope
    // sum_k w[k] snap[k] of plans[j]; rho (if any) after the last step.  With
    // src, the particles of src are first counting-sorted by tet into p, the
    // scatter folded into the first launch's particle kernel.
    //
    // Several steps go up to most_fused at a time through k_push_multi and
    // k_walk_multi; one step, or steps whose slices per wavefront a flag
    // forces, through the one-step kernels (coefficients, particle kernel,
    // walk), which read 10 reals per tet instead of the 30 or 70 of the row
    // parts and can spread a tet's run over several wavefronts' slices.
    template <typename Real>
    int run_steps(const etpic_particles *p, const etpic_species *sp, const StepPlan *plans, int nsteps, double dt,
                  double omega, double *dG, double *rho, uint32_t flags, void *stream,
                  const etpic_particles *src = nullptr) {
        hipStream_t st = static_cast<hipStream_t>(stream);
        constexpr uint32_t kForced =
            ETPIC_STEP_SLICES_1 | ETPIC_STEP_SLICES_2 | ETPIC_STEP_SLICES_4 | ETPIC_STEP_SLICES_16;
        const bool pairs = in_pairs(plans[0], nsteps, p->n);
        const int most = std::min(pairs ? 2 : kMaxFused, most_fused(p->n));
        const bool single = nsteps == 1 || most < 2 || (flags & kForced);
        if (int r = timing_room(flags, single ? nsteps : (nsteps + most - 1) / most)) return r;
        if (src)
            if (int r = sort_count(src, st)) return r;
        if (single)
            return single_steps<Real>(p, sp, plans, nsteps, dt, omega, dG, rho, flags, st, src);
        if constexpr (std::is_same<Real, float>::value) {
            if (flags & kFlagFixed)
                return plans[0].snap[1] && !pairs
                           ? fused_steps<float, 3, true>(p, sp, plans, nsteps, most, dt, omega, dG, rho, flags, st, src)
                           : fused_steps<float, 1, true>(p, sp, plans, nsteps, most, dt, omega, dG, rho, flags, st, src);
        }
        return plans[0].snap[1] && !pairs
                   ? fused_steps<Real, 3, false>(p, sp, plans, nsteps, most, dt, omega, dG, rho, flags, st, src)
                   : fused_steps<Real, 1, false>(p, sp, plans, nsteps, most, dt, omega, dG, rho, flags, st, src);
    }

    template <typename Real>
    int single_steps(const etpic_particles *p, const etpic_species *sp, const StepPlan *plans, int nsteps, double dt,
                     double omega, double *dG, double *rho, uint32_t flags, hipStream_t st,
                     const etpic_particles *src) {
        const int remap = (flags & ETPIC_STEP_XCD_REMAP) ? 1 : 0;
        const int64_t n = p->n;
        const bool time_all = (flags & ETPIC_STEP_TIMING_ALL) != 0;
        bool used_slots = false;
        TimingSet *ta = nullptr;
        for (int j = 0; j < nsteps; ++j) {
            // ts: this step's timing set; ta: the same where every kernel is timed
            TimingSet *ts = nullptr;
            const bool sorts = j == 0 && src;
            if (flags & (ETPIC_STEP_TIMING | ETPIC_STEP_TIMING_ALL))
                if (int r = timing_events(&ts, sorts)) return r;
            ta = time_all ? ts : nullptr;
            if (j == 0)   // (a later step's came with the walk before it)
                if (int r = launch_coef<Real>(plans[0], omega, d_tetG, st, ta)) return r;
            StepArgs<Real> a = step_args<Real>(p, sp, dt, dG, j == nsteps - 1 ? rho : nullptr);
            a.walk_by_slice = (flags & ETPIC_STEP_WALK_BY_SLICE) ? 1 : 0;
            a.fixed = (flags & kFlagFixed) ? 1 : 0;
            a.tetG = d_tetG;
            if (sorts) {
                // read src, write p at the sorted positions; the walk then runs on p
                StepArgs<Real> as = a;
                scatter_from(as, p, src);
                if (as.rho)
                    used_slots |= launch_push<Real, true, true>(as, push_slices_for(flags, n, true), remap, st, ts);
                else
                    used_slots |= launch_push<Real, false, true>(as, push_slices_for(flags, n, true), remap, st, ts);
                a.scatter = 1;
            } else if (a.rho) {
                used_slots |= launch_push<Real, true, false>(a, push_slices_for(flags, n), remap, st, ts);
            } else {
                used_slots |= launch_push<Real, false, false>(a, push_slices_for(flags, n), remap, st, ts);
            }
            HIP_TRY(hipGetLastError());
            hipEvent_t w0 = ev_start(ta, 2), w1 = ev_stop(ta, 2);
            const unsigned both = kWalkBlocks + grid_for(2 * host.nt);
            if (j + 1 == nsteps)
                launch_timed(k_walk<Real>, kWalkBlocks, st, w0, w1, a);
            else if (plans[j + 1].snap[1])
                launch_timed(k_walk_coef<Real, 3>, both, st, w0, w1, a, host.nt, d_gpush64, d_tetface,
                             coef_fields(plans[j + 1], omega));
            else
                launch_timed(k_walk_coef<Real, 1>, both, st, w0, w1, a, host.nt, d_gpush64, d_tetface,
                             coef_fields(plans[j + 1], omega));
            HIP_TRY(hipGetLastError());
        }
        return used_slots ? launch_edges(dG, st, ta, nullptr) : ETPIC_OK;
    }

    // Steps per multi-step launch: a leaver's mark holds its tet and its step,
    // and both have to fit an int32.
    int most_fused(int64_t n) const {
        return (int)std::max<int64_t>(1, std::min<int64_t>(n <= kFewParticles ? kMaxFused : kMaxFusedMany,
                                                           (INT32_MAX - 2) / std::max<int64_t>(host.nt, 1)));
    }

    // Particles per wavefront of a multi-step launch.  Few particles: 16.  A
    // wavefront is then bound by the latency of its steps, and one whose 64
    // particles sit in 64 tets takes its steps in four passes one after the
    // other; up to two wavefronts per SIMD the passes run side by side
    // instead.  (Not where leavers are queued by 64-particle slice: each slice
    // has one owner.)
    static int push_width(int64_t n, uint32_t flags) {
        return n <= kFewParticles && !(flags & ETPIC_STEP_WALK_BY_SLICE) ? 16 : 64;
    }

    // Steps over three snapshots that go two to a launch, from the two steps'
    // own rows (kCoefPair, 240 B per tet) instead of the parts of three
    // snapshots (560 B per tet, which the particle kernel stages too).
    // On 384,000 tets, mixed, one step per launch / parts / pairs: two steps of
    // 2e5 particles 217 / 228 / 159 us, of 1e7 603 / 576 / 440; three steps of
    // 1,000 156 / 174 / 146, but of 2e5 294 / 229 us by one launch already, as
    // are all on few tets (750: 72 / 43), where the launches count.  Any
    // number of steps where no wide rows are bound to hold the parts.
    bool in_pairs(const StepPlan &first, int nsteps, int64_t n) const {
        return first.snap[1] &&
               (!d_coef_env || nsteps == 2 || (nsteps == 3 && n <= kFewParticles && host.nt >= 65536));
    }

    // Blocks of k_walk_multi.  Few particles: as many as the queue has parts (an
    // empty block costs its table's clearing; 1,000 electrons 5.4 us with 512).
    // More blocks take a long queue's leavers sooner and pay for it with more
    // tables; re-sort and ten steps, mixed, with 512 and 1024: 1e7 on 384,000
    // tets 632 and 654 us, 3e7 in a bunch on 3.1e6 tets 3501 and 3472, 6e7 5598
    // and 5439, 1e8 8951 and 8524; without a bunch within 1 % from 3e7 on.
    static unsigned leaver_blocks(int64_t n) {
        return n <= kFewParticles ? kShards : n < ((int64_t)1 << 26) ? kLeaverBlocks : 2 * kLeaverBlocks;
    }

    template <int kSnap>
    double *parts_table() const {
        return kSnap == 3 ? d_coef_env : static_cast<double *>(d_coef);
    }

    // the parts of the 10-real rows, from which multi-step launches form the
    // row of each of their steps
    template <int kSnap>
    int launch_parts(const etpic_fields *const snap[3], const double w[3], double *slots, hipStream_t st, TimingSet *ta) {
        FieldPtrs F = field_ptrs(snap, w, 1.0, 0.0);
        F.xcd = coef_xcd();
        launch_timed(k_tet_coef<double, kSnap, kCoefParts>, grid_for(2 * host.nt), st, ev_start(ta, 0), ev_stop(ta, 0),
                     host.nt, d_gpush64, d_tetface, F, parts_table<kSnap>(), slots);
        HIP_TRY(hipGetLastError());
        return ETPIC_OK;
    }

    // the rows of two steps (b null: of one), for a launch of them
    int launch_pair(const StepPlan &a, const StepPlan *b, double omega, double *slots, hipStream_t st, TimingSet *ta) {
        FieldPtrs F = field_ptrs(a.snap, a.w, std::cos(omega * a.t), std::sin(omega * a.t));
        F.xcd = coef_xcd();
        if (b) {
            for (int k = 0; k < 3; ++k) F.w2[k] = b->w[k];
            F.c2 = std::cos(omega * b->t);
            F.s2 = std::sin(omega * b->t);
        }
        launch_timed(k_tet_coef<double, 3, kCoefPair>, grid_for(2 * host.nt), st, ev_start(ta, 0), ev_stop(ta, 0),
                     host.nt, d_gpush64, d_tetface, F, static_cast<double *>(d_coef), slots);
        HIP_TRY(hipGetLastError());
        return ETPIC_OK;
    }

    // A call's steps taken in several calls of fused_steps.
    struct Segment {
        bool goes_on, last;
        unsigned sets;
    };

    // Multi-step launches of p.  With src, the first launch reads src and
    // writes p: at the tet-sorted places (sorted), or place for place.
    // seg: a call that goes on from an earlier one with the same fields finds
    // the rows' parts ready and adds to the slots as they are; one that another
    // goes on from leaves them; `sets` carries on the turns of the counter sets.
    // Plans over three snapshots with kSnap = 1: two steps to a
    // launch, from their own rows.
    template <typename Real, int kSnap, bool kFixed>
    int fused_steps(const etpic_particles *p, const etpic_species *sp, const StepPlan *plans, int nsteps, int most,
                    double dt, double omega, double *dG, double *rho, uint32_t flags, hipStream_t st,
                    const etpic_particles *src, bool sorted = true, Segment *seg = nullptr) {
        const int remap = (flags & ETPIC_STEP_XCD_REMAP) ? 1 : 0;
        const int64_t n = p->n, nt = host.nt;
        const bool time_all = (flags & ETPIC_STEP_TIMING_ALL) != 0;
        const int launches = (nsteps + most - 1) / most;
        const bool pairs = kSnap == 1 && plans[0].snap[1];
        const int width = push_width(n, flags);
        const unsigned push_grid = grid_for((n + width - 1) / width * 64);
        TimingSet *ta = nullptr;
        unsigned *ctr = nullptr;
        last_slices = 1;
        for (int i = 0, j0 = 0; i < launches; ++i) {
            const int j1 = (int)((int64_t)nsteps * (i + 1) / launches);   // equal shares, at least two steps each
            TimingSet *ts = nullptr;
            const bool moves = i == 0 && src;
            if (flags & (ETPIC_STEP_TIMING | ETPIC_STEP_TIMING_ALL)) {
                if (int r = timing_events(&ts, moves && sorted)) return r;
                ts->steps = j1 - j0;
            }
            ta = time_all ? ts : nullptr;
            if (pairs) {
                if (int r = launch_pair(plans[j0], j1 - j0 > 1 ? &plans[j0 + 1] : nullptr, omega,
                                        i == 0 ? d_tetG : nullptr, st, ta))
                    return r;
            } else if (i == 0 && !(seg && seg->goes_on)) {
                if (int r = launch_parts<kSnap>(plans[0].snap, plans[0].w, d_tetG, st, ta)) return r;
            }
            MultiArgs<kSnap> ma{};
            ma.parts = parts_table<kSnap>();
            ma.nsteps = j1 - j0;
            ma.width = width;
            for (int j = j0; j < j1; ++j) {
                const double c = std::cos(omega * plans[j].t), sn = std::sin(omega * plans[j].t);
                for (int k = 0; k < kSnap; ++k) {
                    ma.wc[j - j0][k] = pairs ? (j == j0 ? 1.0 : 0.0) : plans[j].w[k] * c;
                    ma.ws[j - j0][k] = pairs ? (j == j0 ? 0.0 : -1.0) : plans[j].w[k] * sn;
                }
            }
            StepArgs<Real> a = step_args<Real>(p, sp, dt, dG, j1 == nsteps ? rho : nullptr);
            a.walk_by_slice = (flags & ETPIC_STEP_WALK_BY_SLICE) ? 1 : 0;
            a.fixed = kFixed ? 1 : 0;
            a.tetG = d_tetG;
            const unsigned turn = seg ? seg->sets++ : (unsigned)i;
            ctr = d_walk_ctr + (1 + (turn & 1)) * kCtrStride;
            unsigned *next = d_walk_ctr + (1 + ((turn + 1) & 1)) * kCtrStride;
            a.walk_ctr = ctr;
            hipEvent_t e0 = ev_start(ts, 1), e1 = ev_stop(ts, 1);
            if (moves) {
                StepArgs<Real> as = a;
                scatter_from(as, p, src);
                if (!sorted) {
                    as.cursor = nullptr;
                    as.id = nullptr;
                }
                if (as.rho)
                    launch_timed(k_push_multi<Real, kSnap, true, true, kFixed>, push_grid, st, e0, e1, as, ma, remap);
                else
                    launch_timed(k_push_multi<Real, kSnap, false, true, kFixed>, push_grid, st, e0, e1, as, ma, remap);
                a.scatter = 1;
            } else if (a.rho) {
                launch_timed(k_push_multi<Real, kSnap, true, false, kFixed>, push_grid, st, e0, e1, a, ma, remap);
            } else {
                launch_timed(k_push_multi<Real, kSnap, false, false, kFixed>, push_grid, st, e0, e1, a, ma, remap);
            }
            HIP_TRY(hipGetLastError());
            launch_timed(k_walk_multi<Real, kSnap, kFixed>, leaver_blocks(n), st, ev_start(ta, 2), ev_stop(ta, 2), a, ma,
                         next);
            HIP_TRY(hipGetLastError());
            j0 = j1;
        }
        return seg && !seg->last ? ETPIC_OK : launch_edges(dG, st, ta, ctr);
    }

    template <typename Real>
    const Real *gpush_table() const;
    template <typename Real>
    const Real *geo_table() const;

    // Slices per wavefront of the particle kernel: forced by a flag, else from
    // the mean same-tet run length of the last sort (one slice while runs fit
    // in a wavefront; 4 or 16 for longer runs), kept to >= kMinPushWaves
    // wavefronts so that the chip stays full.
    int push_slices_for(uint32_t flags, int64_t n, bool sorting = false) {
        if (flags & ETPIC_STEP_SLICES_16) return last_slices = 16;
        if (flags & ETPIC_STEP_SLICES_4) return last_slices = 4;
        if (flags & ETPIC_STEP_SLICES_2) return last_slices = 2;
        if (flags & ETPIC_STEP_SLICES_1) return last_slices = 1;
        // The particle kernel adds a run's currents to its tet's slots, so
        // long runs cost it few same-address atomics: one slice measured
        // fastest up to hundreds of particles per tet (5e7 on 40^3 x 6 tets,
        // the 2e8 bunch), and slices are kept for thousands.  The sorting
        // form takes one cursor atomic per run and tet, which slices divide:
        // it keeps them from a hundred particles per tet on
        if (sorting) return last_slices = slices_from_runs(n, 96.0, 256.0);
        int s = slices_from_runs(n, 1024.0, 4096.0);
        // one slice: two pipelined ones (float forms; float64 keeps one) where
        // the float rows of the mesh (coefficient 48 B, push 64 B, geometry 48 B
        // per tet) outgrow the 256 MB Infinity Cache (measured: large box
        // mixed 4.09 -> 3.89 ms, compact 3.96 -> 3.79 ms; on the bench mesh,
        // whose rows fit, 2-5 % slower)
        if (s == 1 && host.nt * (int64_t)kFloatRowBytes > kInfinityCacheBytes && n / 128 >= kMinPushWaves) s = 2;
        return last_slices = s;
    }

    // 1, 4 or 16 slices from the last sort's mean same-tet run length (read
    // back without blocking: a statistic still in flight leaves the previous):
    // 4 from run length lo on, 16 from hi on
    int slices_from_runs(int64_t n, double lo, double hi) {
        if (runstat_pending && hipEventQuery(runstat_ev) == hipSuccess) {
            run_len = runstat_n > 0 ? (double)*h_runstat / (double)runstat_n : 0.0;
            runstat_pending = false;
        }
        (void)hipGetLastError();   // an unfinished query is not an error
        int s = run_len >= hi ? 16 : (run_len >= lo ? 4 : 1);
        while (s > 1 && n / (64 * (int64_t)s) < kMinPushWaves) s /= 4;
        return s;
    }

    // nsteps downshifted steps from step0 (t_n = n dt), hist0 of them taken
    // before; the rows are built once for the call.  The first three steps of
    // a history go one per launch, the others up to kMaxDs.
    template <typename Real>
    int ds_steps(const etpic_particles *p, void *hist, const etpic_species *sp, const etpic_fields *f,
                 int64_t step0, int nsteps, int hist0, double dt, double omega, double *dG, double *rho,
                 uint32_t flags, void *stream) {
        if (f->e_dc) return ds_launches<Real, true>(p, hist, sp, f, step0, nsteps, hist0, dt, omega, dG, rho, flags, stream);
        return ds_launches<Real, false>(p, hist, sp, f, step0, nsteps, hist0, dt, omega, dG, rho, flags, stream);
    }

    template <typename Real, bool kEdc>
    int ds_launches(const etpic_particles *p, void *hist, const etpic_species *sp, const etpic_fields *f,
                    int64_t step0, int nsteps, int hist0, double dt, double omega, double *dG, double *rho,
                    uint32_t flags, void *stream) {
        constexpr bool f64 = std::is_same<Real, double>::value;
        hipStream_t st = static_cast<hipStream_t>(stream);
        const int remap = (flags & ETPIC_STEP_XCD_REMAP) ? 1 : 0;
        const int64_t n = p->n, nt = host.nt;
        if (!d_coef_env)
            return fail(ETPIC_ESTATE, "no downshifted rows bound (etpic_ds_rows_bytes, etpic_ds_rows_bind)");
        const int most = std::min(kMaxDs, most_fused(p->n));
        const bool time_all = (flags & ETPIC_STEP_TIMING_ALL) != 0;
        const etpic_fields *snap[3] = {f, nullptr, nullptr};
        const double w1[3] = {1.0, 0.0, 0.0};
        const int width = push_width(n, flags);
        const unsigned push_grid = grid_for((n + width - 1) / width * 64);
        TimingSet *ta = nullptr;
        unsigned *ctr = nullptr;
        const int alone = std::min(nsteps, std::max(0, 3 - hist0));   // launches of the first three steps
        // One step of fewer particles than tets: most slots would be cleared and
        // gathered for nothing, so its currents go straight to the edges
        // (384,000 tets, mixed: 1,000 particles 182 -> 158 us, 2e5 257 -> 234;
        // of 4e6 the slots' one line per run is worth the gather, 613 us with
        // direct atomics, 533 with slots).
        double *const slots = nsteps == 1 && n < nt ? nullptr : d_tetG;
        if (int r = timing_room(flags, alone + (nsteps - alone + most - 1) / most)) return r;
        for (int j0 = 0, i = 0; j0 < nsteps; ++i) {
            const int H = hist0 + j0;
            const int left = nsteps - j0, launches = (left + most - 1) / most;
            const int len = H < 3 ? 1 : (left + launches - 1) / launches;
            TimingSet *ts = nullptr;
            if (flags & (ETPIC_STEP_TIMING | ETPIC_STEP_TIMING_ALL)) {
                if (int r = timing_events(&ts)) return r;
                ts->steps = len;
            }
            ta = time_all ? ts : nullptr;
            if (i == 0) {
                if constexpr (f64) {
                    if (int r = launch_parts<1>(snap, w1, slots, st, ta)) return r;
                } else {
                    launch_timed(k_tet_coef_env, dim3(grid_for(nt), 6), st, ev_start(ta, 0), ev_stop(ta, 0), nt,
                                 d_gpush64, d_tetface, field_ptrs(snap, w1, 1.0, 0.0), d_coef_env, slots);
                    HIP_TRY(hipGetLastError());
                }
            }
            StepArgs<Real> a = step_args<Real>(p, sp, dt, dG, j0 + len == nsteps ? rho : nullptr);
            a.walk_by_slice = (flags & ETPIC_STEP_WALK_BY_SLICE) ? 1 : 0;
            a.tetG = slots;
            ctr = d_walk_ctr + (1 + (i & 1)) * kCtrStride;
            unsigned *next = d_walk_ctr + (1 + ((i + 1) & 1)) * kCtrStride;
            a.walk_ctr = ctr;
            DsArgs<Real> d{};
            d.rows = f64 ? static_cast<const double *>(d_coef) : d_coef_env;
            d.hist = static_cast<Real *>(hist);
            d.stride = n;
            d.phase = (int)((((step0 + j0) % 4) + 4) % 4);
            d.hist0 = H;
            d.nsteps = len;
            d.width = width;
            d.qm = (Real)(sp->q / sp->m);
            for (int j = 0; j < len; ++j) {
                const int K = std::min(H + j, 2) + 1, A = std::min(H + j, 3) + 1;
                DsWeights W;
                ds_weights(K, A, (double)(step0 + j0 + j) * dt, dt, omega, W);
                for (int k = 0; k < K; ++k) {
                    d.Mr[j][k] = (Real)W.Mr[k];
                    d.Mi[j][k] = (Real)W.Mi[k];
                    d.P[k] = (Real)W.P[k];
                    for (int m = 0; m < K; ++m) {
                        d.Lr[j][3 * m + k] = (Real)W.Lr[m * K + k];
                        d.Li[j][3 * m + k] = (Real)W.Li[m * K + k];
                        d.Q[3 * m + k] = (Real)W.Q[m * K + k];
                    }
                }
                for (int k = 0; k < 4; ++k) d.ab[k] = (Real)W.ab[k];
            }
            if (a.rho)
                launch_timed(k_push_ds<Real, true, kEdc>, push_grid, st, ev_start(ts, 1), ev_stop(ts, 1), a, d, remap);
            else
                launch_timed(k_push_ds<Real, false, kEdc>, push_grid, st, ev_start(ts, 1), ev_stop(ts, 1), a, d, remap);
            HIP_TRY(hipGetLastError());
            launch_timed(k_walk_ds<Real, kEdc>, kLeaverBlocks, st, ev_start(ta, 2), ev_stop(ta, 2), a, d, next);
            HIP_TRY(hipGetLastError());
            j0 += len;
        }
        if (slots) return launch_edges(dG, st, ta, ctr);
        k_fill_u32<<<grid_for(kCtrStride), kBlock, 0, st>>>(ctr, kCtrStride, 0u);
        HIP_TRY(hipGetLastError());
        return ETPIC_OK;
    }

    // Weights of one downshifted step [t0, t0 + h] with K Lagrange nodes at
    // t0, t0 - h, t0 - 2h, in closed form: with s = (t - t0) / h the basis
    // polynomials have the monomial coefficients below, and
    // J_p = int_0^1 s^p e^{j theta s} ds (theta = w h) comes from its power
    // series for |theta| < 1 and from the integration-by-parts recurrence
    // J_p = (e^{j theta} - p J_{p-1}) / (j theta) above.
    static void ds_weights(int K, int A, double t0, double h, double omega, DsWeights &d) {
        using cplx = std::complex<double>;
        double cf[3][3] = {{0.0}};
        if (K == 1) {
            cf[0][0] = 1.0;
        } else if (K == 2) {
            cf[0][0] = 1.0, cf[0][1] = 1.0;      // 1 + s
            cf[1][1] = -1.0;                     // -s
        } else {
            cf[0][0] = 1.0, cf[0][1] = 1.5, cf[0][2] = 0.5;   // (s + 1)(s + 2) / 2
            cf[1][1] = -2.0, cf[1][2] = -1.0;                 // -s (s + 2)
            cf[2][1] = 0.5, cf[2][2] = 0.5;                   // s (s + 1) / 2
        }
        const double th = omega * h;
        cplx J[5];
        const cplx jt(0.0, th);
        if (std::fabs(th) < 1.0) {
            for (int q = 0; q < 5; ++q) {
                cplx sum = 0.0, term = 1.0;   // (j theta)^m / m!
                for (int m = 0; m < 30; ++m) {
                    sum += term / (double)(q + m + 1);
                    term *= jt / (double)(m + 1);
                }
                J[q] = sum;
            }
        } else {
            const cplx e = std::exp(jt);
            J[0] = (e - 1.0) / jt;
            for (int q = 1; q < 5; ++q) J[q] = (e - (double)q * J[q - 1]) / jt;
        }
        const cplx ph(std::cos(omega * t0), std::sin(omega * t0));
        for (int k = 0; k < 3; ++k) d.Mr[k] = d.Mi[k] = d.P[k] = 0.0;
        for (int k = 0; k < 9; ++k) d.Lr[k] = d.Li[k] = d.Q[k] = 0.0;
        for (int k = 0; k < K; ++k) {
            cplx mu = 0.0;
            double pk = 0.0;
            for (int q = 0; q < 3; ++q) {
                mu += cf[k][q] * J[q];
                pk += cf[k][q] / (q + 1);
            }
            mu *= h * ph;
            d.Mr[k] = mu.real();
            d.Mi[k] = -mu.imag();
            d.P[k] = h * pk;
            for (int jj = 0; jj < K; ++jj) {
                cplx la = 0.0;
                double qk = 0.0;
                for (int q1 = 0; q1 < 3; ++q1)
                    for (int q2 = 0; q2 < 3; ++q2) {
                        la += cf[jj][q1] * cf[k][q2] * J[q1 + q2];
                        qk += cf[jj][q1] * cf[k][q2] / (q1 + q2 + 1);
                    }
                la *= h * ph;
                d.Lr[jj * K + k] = la.real();
                d.Li[jj * K + k] = -la.imag();
                d.Q[jj * K + k] = h * qk;
            }
        }
        static const double kAB[4][4] = {{1.0, 0.0, 0.0, 0.0},
                                         {1.5, -0.5, 0.0, 0.0},
                                         {23.0 / 12.0, -16.0 / 12.0, 5.0 / 12.0, 0.0},
                                         {55.0 / 24.0, -59.0 / 24.0, 37.0 / 24.0, -9.0 / 24.0}};
        for (int i = 0; i < 4; ++i) d.ab[i] = h * kAB[A - 1][i];
    }

    // Forgets the mesh and everything derived from it (the buffers are the
    // caller's: nothing is freed here).
    void release() {
        d_topo = nullptr;
        d_grad64 = nullptr;
        d_gpush64 = nullptr;
        d_gpush32 = nullptr;
        d_geo64 = nullptr;
        d_geo32 = nullptr;
        d_tetface = nullptr;
        d_coef = nullptr;
        d_coef_env = nullptr;
        d_v2e_ptr = d_v2e_code = nullptr;
        d_e2s_ptr = d_e2s_slot = nullptr;
        d_tetG = nullptr;
        d_xyz = nullptr;
        d_grid = nullptr;
        grid = GridArgs{};
        d_count = d_tilesum = nullptr;
        field.release();
        ns.release();
        field_pending.reset();
        ns_pending.reset();
        has_mesh = false;
    }
};


// File-scope scratch of the allocation-free residual (each GPU holds its own
// copy for the life of the process): kResBlocks partial pairs, then the
// result pair (16 KB).  Host code never passes this name to a kernel or a
// copy: on the host it is a stand-in, not a device address.  The device
// address is taken once per device with hipGetSymbolAddress (scratch_address,
// called by etpic_create with the device current) and used everywhere instead.
static __device__ __align__(256) double scratch[kScratchDoubles];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double *g_scratch_addr[kMaxDevices] = {};

// The device address of `scratch` on the current device `device`.
int scratch_address(int device, double **out) {
    if (device < 0 || device >= kMaxDevices) return fail(ETPIC_EINVAL, "device %d beyond %d", device, kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_addr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(ETPIC_EHIP, "address of the residual scratch: %s", hipGetErrorString(e));
        g_scratch_addr[device] = static_cast<double *>(p);
    }
    *out = g_scratch_addr[device];
    return ETPIC_OK;
}
}  // namespace

template <>
const double *etpic_ctx::gpush_table<double>() const { return d_gpush64; }
template <>
const float *etpic_ctx::gpush_table<float>() const { return d_gpush32; }
template <>
const double *etpic_ctx::geo_table<double>() const { return d_geo64; }
template <>
const float *etpic_ctx::geo_table<float>() const { return d_geo32; }

namespace {

// Makes the context's device current; every call that launches kernels goes
// through here, so it also requires the context workspace (status word, walk
// queues, reduction words) to be bound.
int set_device(const etpic_ctx *ctx) {
    if (!ctx->has_ws) return fail(ETPIC_ESTATE, "no workspace bound (etpic_workspace_bytes, etpic_workspace_bind)");
    HIP_TRY(hipSetDevice(ctx->device));
    return ETPIC_OK;
}

// The device only (setup calls that copy tables but launch nothing).
int set_device_only(const etpic_ctx *ctx) {
    HIP_TRY(hipSetDevice(ctx->device));
    return ETPIC_OK;
}

// ETPIC_FP64, ETPIC_MIXED, and ETPIC_MIXED_FIXED where the entry point has the
// fixed-point form.
int check_precision(int precision, bool fixed_ok) {
    if (precision == ETPIC_FP64 || precision == ETPIC_MIXED) return ETPIC_OK;
    if (precision == ETPIC_MIXED_FIXED) {
        if (fixed_ok) return ETPIC_OK;
        return fail(ETPIC_EINVAL, "this entry point has no fixed-point (ETPIC_MIXED_FIXED) form");
    }
    return fail(ETPIC_EINVAL, "bad precision %d", precision);
}

// Public step flags: bit 31 is the library's own.
uint32_t step_flags(uint32_t flags, int precision) {
    return (flags & ~kFlagFixed) | (precision == ETPIC_MIXED_FIXED ? kFlagFixed : 0u);
}

int check_particles(const etpic_ctx *ctx, const etpic_particles *p) {
    if (!p) return fail(ETPIC_EINVAL, "null particle descriptor");
    if (p->n < 0) return fail(ETPIC_EINVAL, "negative particle count");
    if (p->n > (int64_t)kWalkQueueCap * 64) return fail(ETPIC_EINVAL, "particle count above 2^29");
    if (p->n == 0) return ETPIC_OK;
    for (int k = 0; k < 3; ++k)
        if (!p->lam[k] || !p->vel[k]) return fail(ETPIC_EINVAL, "null particle array");
    if (!p->tet) return fail(ETPIC_EINVAL, "null tet array");
    (void)ctx;
    return ETPIC_OK;
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Workspace of the differentiation entry points: ncp checkpoints and
// checkpoint_every segment slots, each a float64 particle state (lam, v, tet),
// then a scratch current accumulator.
struct AdjLayout {
    size_t arr8, arr4, state, slots_off, dG_off, total;
    int ncp;
};

AdjLayout adj_layout(int64_t n, int64_t ne, int nsteps, int every) {
    AdjLayout L{};
    L.arr8 = align256(sizeof(double) * (size_t)n);
    L.arr4 = align256(sizeof(int32_t) * (size_t)n);
    L.state = 6 * L.arr8 + L.arr4;
    L.ncp = (nsteps + every - 1) / every;
    L.slots_off = (size_t)L.ncp * L.state;
    L.dG_off = L.slots_off + (size_t)every * L.state;
    L.total = L.dG_off + align256(sizeof(double) * (size_t)ne);
    return L;
}

etpic_particles state_view(void *ws, size_t off, const AdjLayout &L, int64_t n) {
    char *b = static_cast<char *>(ws) + off;
    etpic_particles q{};
    q.n = n;
    for (int k = 0; k < 3; ++k) {
        q.lam[k] = reinterpret_cast<double *>(b + k * L.arr8);
        q.vel[k] = b + (3 + k) * L.arr8;
    }
    q.tet = reinterpret_cast<int32_t *>(b + 6 * L.arr8);
    q.id = nullptr;
    return q;
}

int check_step_args(const etpic_ctx *ctx, const etpic_species *sp, const etpic_fields *f, double dt, double omega) {
    if (!ctx || !sp || !f) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (!f->e_env || !f->b_env) return fail(ETPIC_EINVAL, "null envelope DoFs");
    if (!(std::isfinite(dt) && std::isfinite(omega) && sp->m != 0.0 && std::isfinite(sp->q) && std::isfinite(sp->m)))
        return fail(ETPIC_EINVAL, "non-finite dt / omega or zero mass");
    return ETPIC_OK;
}

}  // namespace

// =============================================================================== C ABI
extern "C" {

const char *etpic_last_error(void) { return g_last_error.c_str(); }

int etpic_create(etpic_ctx **out, int device) {
    if (!out) return fail(ETPIC_EINVAL, "null output handle");
    *out = nullptr;
    int ndev = 0;
    HIP_TRY(hipGetDeviceCount(&ndev));
    if (device < 0 || device >= ndev) return fail(ETPIC_EINVAL, "device %d not present (%d devices)", device, ndev);
    etpic_ctx *c = new etpic_ctx();
    c->device = device;
    // host-side resources only: the pinned word the run-length statistic is
    // read into, its event, the step-timing events; device memory comes from
    // the caller (etpic_workspace_bind, etpic_mesh_upload, ...)
    hipError_t e = hipSetDevice(device);
    if (e == hipSuccess) e = hipHostMalloc(&c->h_runstat, 4 * sizeof(unsigned long long) + sizeof(SolveWatch),
                                               hipHostMallocMapped | hipHostMallocCoherent);
    if (e == hipSuccess) c->h_watch = reinterpret_cast<SolveWatch *>(c->h_runstat + 4);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&c->runstat_ev, hipEventDisableTiming);
    c->spare.reserve(kTimingSets);
    c->timing.reserve(kTimingSets);
    for (int k = 0; k < kTimingSets && e == hipSuccess; ++k) {
        etpic_ctx::TimingSet set{};
        int made = 0;
        for (auto &x : set.ev) {
            // timing only: no system-scope fence when the event completes (no
            // cache writeback and invalidation between the kernels it times)
            e = hipEventCreateWithFlags(&x, hipEventDisableSystemFence);
            if (e != hipSuccess) break;
            ++made;
        }
        if (e != hipSuccess)
            for (int i = 0; i < made; ++i) (void)hipEventDestroy(set.ev[i]);
        else
            c->spare.push_back(set);
    }
    int rs = ETPIC_OK;
    if (e == hipSuccess) rs = scratch_address(device, &c->d_scratch);
    if (e != hipSuccess || rs != ETPIC_OK) {
        if (c->h_runstat) (void)hipHostFree(c->h_runstat);
        if (c->runstat_ev) (void)hipEventDestroy(c->runstat_ev);
        for (auto &set : c->spare)
            for (auto x : set.ev) (void)hipEventDestroy(x);
        delete c;
        if (rs != ETPIC_OK) return rs;
        return fail(ETPIC_EHIP, "context setup: %s", hipGetErrorString(e));
    }
    *out = c;
    return ETPIC_OK;
}

int etpic_destroy(etpic_ctx *ctx) {
    if (!ctx) return ETPIC_OK;
    (void)hipSetDevice(ctx->device);
    (void)hipDeviceSynchronize();
    ctx->release();
    (void)hipHostFree(ctx->h_runstat);
    (void)hipEventDestroy(ctx->runstat_ev);
    for (auto &e : ctx->timing)
        for (auto x : e.ev) (void)hipEventDestroy(x);
    for (auto &e : ctx->spare)
        for (auto x : e.ev) (void)hipEventDestroy(x);
    delete ctx;
    return ETPIC_OK;
}

}  // extern "C"

namespace {

// Context workspace: the status word, the residual and run-length words, the
// walk counters and the two walk queues.
struct WsPtrs {
    unsigned *status, *walk_ctr, *walk_queue, *slice_queue;
    unsigned long long *red, *runstat;
};
WsPtrs ws_layout(Carve &cv) {
    WsPtrs w;
    w.status = cv.take<unsigned>(1);
    w.walk_ctr = cv.take<unsigned>(kCtrSets * kCtrStride);
    w.red = cv.take<unsigned long long>(2 * kResBlocks);
    w.runstat = cv.take<unsigned long long>(1);
    w.walk_queue = cv.take<unsigned>(kWalkQueueCap);
    w.slice_queue = cv.take<unsigned>(kWalkQueueCap);
    return w;
}

int check_buffer(const void *buf, size_t bytes, size_t need, const char *what) {
    if (!buf) return fail(ETPIC_EINVAL, "%s: null buffer", what);
    if (reinterpret_cast<uintptr_t>(buf) & 255u) return fail(ETPIC_EINVAL, "%s: buffer not 256-byte aligned", what);
    if (bytes < need) return fail(ETPIC_EINVAL, "%s: buffer of %zu bytes, %zu needed", what, bytes, need);
    return ETPIC_OK;
}

// Mesh tables, in this order: tet topology, float64 gradients, float64 and
// float32 push rows, float64 and float32 geometry rows, tet-face ids, the
// coefficient table, vertex coordinates,
// point-location start grid, vertex -> edge CSR, sort counters and tile sums,
// edge -> tet-slot CSR, per-tet current slots.
struct MeshPtrs {
    TetTopo *topo;
    double *grad64, *gpush64, *geo64;
    float *gpush32, *geo32;
    int32_t *tetface;
    void *coef;
    double *xyz;
    int32_t *grid, *v2e_ptr, *v2e_code;
    unsigned *count, *tilesum;
    int32_t *e2s_ptr, *e2s_slot;
    double *tetG;
};
MeshPtrs mesh_layout(Carve &cv, const etpic::HostMesh &M, size_t grid_cells) {
    const int64_t nt = M.nt;
    MeshPtrs m;
    m.topo = cv.take<TetTopo>(nt);
    m.grad64 = cv.take<double>(12 * nt);
    m.gpush64 = cv.take<double>((size_t)PushRow<double>::kStride * nt);
    m.gpush32 = cv.take<float>((size_t)PushRow<float>::kStride * nt);
    m.geo64 = cv.take<double>((size_t)GeoRow<double>::kStride * nt);
    m.geo32 = cv.take<float>((size_t)GeoRow<float>::kStride * nt);
    m.tetface = cv.take<int32_t>(4 * nt);
    m.coef = cv.take<double>((size_t)kCoefDoubles * nt);
    m.xyz = cv.take<double>(3 * M.nv);
    m.grid = cv.take<int32_t>(grid_cells);
    m.v2e_ptr = cv.take<int32_t>(M.nv + 1);
    m.v2e_code = cv.take<int32_t>(2 * M.ne);
    m.count = cv.take<unsigned>(nt + 1);
    m.tilesum = cv.take<unsigned>((nt + 1 + kScanTile - 1) / kScanTile);
    m.e2s_ptr = cv.take<int32_t>(M.ne + 1);
    m.e2s_slot = cv.take<int32_t>(6 * nt);
    m.tetG = cv.take<double>(8 * nt);
    return m;
}

int host_mesh(int64_t n_vert, const double *xyz_host, int64_t n_tet, const int32_t *tet_vert_host,
              etpic::HostMesh &M, etpic::StartGrid &sg) {
    if (!xyz_host || !tet_vert_host) return fail(ETPIC_EINVAL, "mesh: null array");
    std::string err;
    int rc = etpic::build_host_mesh(n_vert, xyz_host, n_tet, tet_vert_host, M, err);
    if (rc == -1) return fail(ETPIC_EINVAL, "mesh: %s", err.c_str());
    if (rc != 0) return fail(ETPIC_EMESH, "mesh: %s", err.c_str());
    etpic::build_start_grid(M, xyz_host, 2.0, sg);
    return ETPIC_OK;
}

}  // namespace

extern "C" {

int etpic_workspace_bytes(size_t *bytes) {
    if (!bytes) return fail(ETPIC_EINVAL, "null argument");
    Carve cv;
    (void)ws_layout(cv);
    *bytes = cv.used;
    return ETPIC_OK;
}

int etpic_workspace_bind(etpic_ctx *ctx, void *dev_buf, size_t bytes) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    size_t need = 0;
    (void)etpic_workspace_bytes(&need);
    if (int r = check_buffer(dev_buf, bytes, need, "workspace")) return r;
    if (int r = set_device_only(ctx)) return r;
    HIP_TRY(hipDeviceSynchronize());
    Carve cv;
    cv.base = static_cast<char *>(dev_buf);
    cv.cap = bytes;
    const WsPtrs w = ws_layout(cv);
    ctx->d_status = w.status;
    ctx->d_walk_ctr = w.walk_ctr;
    ctx->d_red = w.red;
    ctx->d_runstat = w.runstat;
    ctx->d_walk_queue = w.walk_queue;
    ctx->d_slice_queue = w.slice_queue;
    HIP_TRY(hipMemset(ctx->d_status, 0, sizeof(unsigned)));
    HIP_TRY(hipMemset(ctx->d_walk_ctr, 0, kCtrSets * kCtrStride * sizeof(unsigned)));
    HIP_TRY(hipDeviceSynchronize());
    ctx->runstat_pending = false;
    ctx->has_ws = true;
    return ETPIC_OK;
}

int etpic_mesh_sizes(int64_t n_vert, const double *xyz_host, int64_t n_tet, const int32_t *tet_vert_host,
                     int64_t counts_out[4], size_t *dev_bytes) {
    if (!counts_out || !dev_bytes) return fail(ETPIC_EINVAL, "null output");
    etpic::HostMesh M;
    etpic::StartGrid sg;
    if (int r = host_mesh(n_vert, xyz_host, n_tet, tet_vert_host, M, sg)) return r;
    counts_out[0] = M.nv;
    counts_out[1] = M.ne;
    counts_out[2] = M.nf;
    counts_out[3] = M.nt;
    Carve cv;
    (void)mesh_layout(cv, M, sg.cell.size());
    *dev_bytes = cv.used;
    return ETPIC_OK;
}

int etpic_mesh_upload(etpic_ctx *ctx, int64_t n_vert, const double *xyz_host, int64_t n_tet,
                      const int32_t *tet_vert_host, void *dev_buf, size_t bytes) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    etpic::HostMesh M;
    etpic::StartGrid sg;
    if (int r = host_mesh(n_vert, xyz_host, n_tet, tet_vert_host, M, sg)) return r;
    size_t need = 0;
    {
        Carve cv;
        (void)mesh_layout(cv, M, sg.cell.size());
        need = cv.used;
    }
    if (int r = check_buffer(dev_buf, bytes, need, "mesh")) return r;
    if (int r = set_device_only(ctx)) return r;
    HIP_TRY(hipDeviceSynchronize());
    ctx->release();
    Carve cv;
    cv.base = static_cast<char *>(dev_buf);
    cv.cap = bytes;
    const MeshPtrs m = mesh_layout(cv, M, sg.cell.size());
    const int64_t nt = M.nt;
    ctx->d_topo = m.topo;
    ctx->d_grad64 = m.grad64;
    ctx->d_gpush64 = m.gpush64;
    ctx->d_gpush32 = m.gpush32;
    ctx->d_geo64 = m.geo64;
    ctx->d_geo32 = m.geo32;
    ctx->d_tetface = m.tetface;
    ctx->d_coef = m.coef;
    ctx->d_xyz = m.xyz;
    ctx->d_grid = m.grid;
    ctx->d_v2e_ptr = m.v2e_ptr;
    ctx->d_v2e_code = m.v2e_code;
    ctx->d_count = m.count;
    ctx->d_tilesum = m.tilesum;
    ctx->tiles = (nt + 1 + kScanTile - 1) / kScanTile;
    ctx->d_e2s_ptr = m.e2s_ptr;
    ctx->d_e2s_slot = m.e2s_slot;
    ctx->d_tetG = m.tetG;
    {
        constexpr int s64 = PushRow<double>::kStride, s32 = PushRow<float>::kStride;
        std::vector<double> gp64((size_t)nt * s64, 0.0);
        std::vector<float> gp32((size_t)nt * s32, 0.0f);
        std::vector<int32_t> tf((size_t)nt * 4);
        for (int64_t t = 0; t < nt; ++t) {
            for (int k = 0; k < 9; ++k) {
                gp64[s64 * t + k] = M.grad[12 * t + 3 + k];
                gp32[s32 * t + k] = (float)M.grad[12 * t + 3 + k];
            }
            std::memcpy(&gp64[s64 * t + PushRow<double>::kEdges], M.topo[t].e, sizeof(int32_t) * 6);
            std::memcpy(&gp32[s32 * t + PushRow<float>::kEdges], M.topo[t].e, sizeof(int32_t) * 6);
            std::memcpy(&tf[4 * t], M.topo[t].f, sizeof(int32_t) * 4);
        }
        HIP_TRY(hipMemcpy(ctx->d_gpush64, gp64.data(), sizeof(double) * s64 * nt, hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(ctx->d_gpush32, gp32.data(), sizeof(float) * s32 * nt, hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(ctx->d_tetface, tf.data(), sizeof(int32_t) * 4 * nt, hipMemcpyHostToDevice));
        // geometry rows: the edge vectors from local vertex 0 (canonical order)
        constexpr int g64 = GeoRow<double>::kStride, g32 = GeoRow<float>::kStride;
        std::vector<double> ge64((size_t)nt * g64, 0.0);
        std::vector<float> ge32((size_t)nt * g32, 0.0f);
        for (int64_t t = 0; t < nt; ++t) {
            const int64_t v0 = M.topo[t].v[0];
            for (int k = 1; k < 4; ++k)
                for (int c = 0; c < 3; ++c) {
                    const double d = xyz_host[3 * (int64_t)M.topo[t].v[k] + c] - xyz_host[3 * v0 + c];
                    ge64[g64 * t + 3 * (k - 1) + c] = d;
                    ge32[g32 * t + 3 * (k - 1) + c] = (float)d;
                }
        }
        HIP_TRY(hipMemcpy(ctx->d_geo64, ge64.data(), sizeof(double) * g64 * nt, hipMemcpyHostToDevice));
        HIP_TRY(hipMemcpy(ctx->d_geo32, ge32.data(), sizeof(float) * g32 * nt, hipMemcpyHostToDevice));
    }
    HIP_TRY(hipMemcpy(ctx->d_xyz, xyz_host, sizeof(double) * 3 * M.nv, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(ctx->d_grid, sg.cell.data(), sizeof(int32_t) * sg.cell.size(), hipMemcpyHostToDevice));
    ctx->grid.cell = ctx->d_grid;
    for (int d = 0; d < 3; ++d) {
        ctx->grid.lo[d] = sg.lo[d];
        ctx->grid.inv[d] = sg.inv[d];
        ctx->grid.dims[d] = sg.dims[d];
    }
    HIP_TRY(hipMemcpy(ctx->d_topo, M.topo.data(), sizeof(TetTopo) * nt, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(ctx->d_grad64, M.grad.data(), sizeof(double) * 12 * nt, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(ctx->d_v2e_ptr, M.v2e_ptr.data(), sizeof(int32_t) * (M.nv + 1), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(ctx->d_v2e_code, M.v2e_code.data(), sizeof(int32_t) * 2 * M.ne, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(ctx->d_e2s_ptr, M.e2s_ptr.data(), sizeof(int32_t) * (M.ne + 1), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(ctx->d_e2s_slot, M.e2s_slot.data(), sizeof(int32_t) * 6 * nt, hipMemcpyHostToDevice));
    HIP_TRY(hipMemset(ctx->d_tetG, 0, sizeof(double) * 8 * nt));
    HIP_TRY(hipDeviceSynchronize());
    ctx->host = std::move(M);
    ctx->has_mesh = true;
    ctx->mesh_hash = etpic::ckpt::mesh_hash(n_vert, xyz_host, n_tet, tet_vert_host);
    return ETPIC_OK;
}

int etpic_mesh_canonical(int64_t n_vert, const double *xyz_host, int64_t n_tet, const int32_t *tet_vert_host,
                         int64_t counts_out[4], int32_t *edge_vert_host, int32_t *face_vert_host) {
    if (!counts_out) return fail(ETPIC_EINVAL, "null counts");
    std::string err;
    etpic::HostMesh M;
    int rc = etpic::build_host_mesh(n_vert, xyz_host, n_tet, tet_vert_host, M, err);
    if (rc == -1) return fail(ETPIC_EINVAL, "mesh: %s", err.c_str());
    if (rc != 0) return fail(ETPIC_EMESH, "mesh: %s", err.c_str());
    counts_out[0] = M.nv;
    counts_out[1] = M.ne;
    counts_out[2] = M.nf;
    counts_out[3] = M.nt;
    if (edge_vert_host) std::memcpy(edge_vert_host, M.edges.data(), sizeof(int32_t) * M.edges.size());
    if (face_vert_host) std::memcpy(face_vert_host, M.faces.data(), sizeof(int32_t) * M.faces.size());
    return ETPIC_OK;
}

int etpic_mesh_counts(const etpic_ctx *ctx, int64_t counts_out[4]) {
    if (!ctx || !counts_out) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    counts_out[0] = ctx->host.nv;
    counts_out[1] = ctx->host.ne;
    counts_out[2] = ctx->host.nf;
    counts_out[3] = ctx->host.nt;
    return ETPIC_OK;
}

int etpic_mesh_edges(const etpic_ctx *ctx, int32_t *edge_vert_host) {
    if (!ctx || !edge_vert_host) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    std::memcpy(edge_vert_host, ctx->host.edges.data(), sizeof(int32_t) * ctx->host.edges.size());
    return ETPIC_OK;
}

int etpic_mesh_faces(const etpic_ctx *ctx, int32_t *face_vert_host) {
    if (!ctx || !face_vert_host) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    std::memcpy(face_vert_host, ctx->host.faces.data(), sizeof(int32_t) * ctx->host.faces.size());
    return ETPIC_OK;
}

static int check_sort_pair(etpic_ctx *ctx, const etpic_particles *src, const etpic_particles *dst) {
    if (!ctx || !src || !dst) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (int r = check_particles(ctx, src)) return r;
    if (int r = check_particles(ctx, dst)) return r;
    if (src->n != dst->n) return fail(ETPIC_EINVAL, "source and destination sizes differ");
    if ((src->id == nullptr) != (dst->id == nullptr)) return fail(ETPIC_EINVAL, "id array given on one side only");
    for (int k = 0; k < 3; ++k)
        if (src->lam[k] == dst->lam[k] || src->vel[k] == dst->vel[k])
            return fail(ETPIC_EINVAL, "sort needs distinct source and destination buffers");
    if (src->tet == dst->tet || (src->id && src->id == dst->id))
        return fail(ETPIC_EINVAL, "sort needs distinct source and destination buffers");
    return ETPIC_OK;
}

int etpic_gather_push_deposit(etpic_ctx *ctx, const etpic_particles *p, int precision, const etpic_species *sp,
                              const etpic_fields *f, int64_t step, double dt, double omega, double *dG,
                              double *rho, uint32_t flags, void *stream) {
    if (int r = check_step_args(ctx, sp, f, dt, omega)) return r;
    if (!dG) return fail(ETPIC_EINVAL, "null current accumulator");
    if (int r = check_particles(ctx, p)) return r;
    if (int r = check_precision(precision, true)) return r;
    if (p->n == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    flags = step_flags(flags, precision);
    if (precision == ETPIC_FP64) return ctx->step<double>(p, sp, f, step, dt, omega, dG, rho, flags, stream);
    return ctx->step<float>(p, sp, f, step, dt, omega, dG, rho, flags, stream);
}

int etpic_coarse_step(etpic_ctx *ctx, const etpic_particles *p, int precision, const etpic_species *sp,
                      const etpic_fields snap[3], double t_coarse, double dt_coarse, int fine_steps, double omega,
                      double *dG, double *rho, uint32_t flags, void *stream) {
    if (!snap) return fail(ETPIC_EINVAL, "null snapshot array");
    for (int k = 0; k < 3; ++k)
        if (int r = check_step_args(ctx, sp, &snap[k], dt_coarse, omega)) return r;
    if (!dG) return fail(ETPIC_EINVAL, "null current accumulator");
    if (fine_steps < 1 || !(dt_coarse > 0.0) || !std::isfinite(t_coarse))
        return fail(ETPIC_EINVAL, "need fine_steps >= 1, dt_coarse > 0 and a finite t_coarse");
    if (int r = check_particles(ctx, p)) return r;
    if (int r = check_precision(precision, true)) return r;
    if (p->n == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    const double dt = dt_coarse / fine_steps;
    std::vector<StepPlan> plans((size_t)fine_steps);
    for (int j = 0; j < fine_steps; ++j) {
        // fine step j gathers at t = t_n + j dt; with u = j / M in [0, 1) the
        // quadratic Lagrange weights on the nodes u = -1, 0, 1 are
        // u(u - 1)/2, 1 - u^2, u(u + 1)/2
        const double u = (double)j / fine_steps;
        plans[j] = StepPlan{{&snap[0], &snap[1], &snap[2]},
                            {0.5 * u * (u - 1.0), 1.0 - u * u, 0.5 * u * (u + 1.0)},
                            t_coarse + j * dt};
    }
    flags = step_flags(flags, precision);
    if (precision == ETPIC_FP64)
        return ctx->run_steps<double>(p, sp, plans.data(), fine_steps, dt, omega, dG, rho, flags, stream);
    return ctx->run_steps<float>(p, sp, plans.data(), fine_steps, dt, omega, dG, rho, flags, stream);
}

int etpic_run_steps(etpic_ctx *ctx, const etpic_particles *p, int precision, const etpic_species *sp,
                    const etpic_fields *f, int64_t step0, int nsteps, double dt, double omega, double *dG,
                    double *rho, uint32_t flags, void *stream) {
    if (int r = check_step_args(ctx, sp, f, dt, omega)) return r;
    if (!dG) return fail(ETPIC_EINVAL, "null current accumulator");
    if (nsteps < 0) return fail(ETPIC_EINVAL, "negative step count");
    if (int r = check_particles(ctx, p)) return r;
    if (int r = check_precision(precision, true)) return r;
    if (p->n == 0 || nsteps == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    std::vector<StepPlan> plans((size_t)nsteps);
    for (int j = 0; j < nsteps; ++j) plans[j] = StepPlan{{f, nullptr, nullptr}, {1.0, 0.0, 0.0}, (double)(step0 + j) * dt};
    flags = step_flags(flags, precision);
    if (precision == ETPIC_FP64)
        return ctx->run_steps<double>(p, sp, plans.data(), nsteps, dt, omega, dG, rho, flags, stream);
    return ctx->run_steps<float>(p, sp, plans.data(), nsteps, dt, omega, dG, rho, flags, stream);
}

int etpic_sort_run_steps(etpic_ctx *ctx, const etpic_particles *src, const etpic_particles *dst, int precision,
                         const etpic_species *sp, const etpic_fields *f, int64_t step0, int nsteps, double dt,
                         double omega, double *dG, double *rho, uint32_t flags, void *stream) {
    if (int r = check_sort_pair(ctx, src, dst)) return r;
    if (int r = check_step_args(ctx, sp, f, dt, omega)) return r;
    if (!dG) return fail(ETPIC_EINVAL, "null current accumulator");
    if (nsteps < 1) return fail(ETPIC_EINVAL, "need at least one step");
    if (int r = check_precision(precision, true)) return r;
    if (src->n == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    std::vector<StepPlan> plans((size_t)nsteps);
    for (int j = 0; j < nsteps; ++j) plans[j] = StepPlan{{f, nullptr, nullptr}, {1.0, 0.0, 0.0}, (double)(step0 + j) * dt};
    flags = step_flags(flags, precision);
    if (precision == ETPIC_FP64)
        return ctx->run_steps<double>(dst, sp, plans.data(), nsteps, dt, omega, dG, rho, flags, stream, src);
    return ctx->run_steps<float>(dst, sp, plans.data(), nsteps, dt, omega, dG, rho, flags, stream, src);
}

static size_t ds_history_size(int64_t n, int precision) {
    return (precision == ETPIC_FP64 ? sizeof(double) : sizeof(float)) * (size_t)kDsArrays * (size_t)n;
}

int etpic_ds_rows_bytes(const etpic_ctx *ctx, size_t *bytes) {
    if (!ctx || !bytes) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    *bytes = sizeof(double) * (size_t)kEnvRow * (size_t)ctx->host.nt;
    return ETPIC_OK;
}

int etpic_ds_rows_bind(etpic_ctx *ctx, void *dev_buf, size_t bytes) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    size_t need = 0;
    if (int r = etpic_ds_rows_bytes(ctx, &need)) return r;
    if (int r = check_buffer(dev_buf, bytes, need, "downshifted rows")) return r;
    ctx->d_coef_env = static_cast<double *>(dev_buf);
    return ETPIC_OK;
}

int etpic_ds_history_bytes(int64_t n, int precision, size_t *bytes_out) {
    if (!bytes_out || n < 0) return fail(ETPIC_EINVAL, "bad arguments");
    if (int r = check_precision(precision, false)) return r;
    *bytes_out = ds_history_size(n, precision);
    return ETPIC_OK;
}

int etpic_ds_steps(etpic_ctx *ctx, const etpic_particles *p, int precision, void *hist, size_t hist_bytes,
                   const etpic_species *sp, const etpic_fields *f, int64_t step0, int nsteps, int hist0, double dt,
                   double omega, double *dG, double *rho, uint32_t flags, void *stream) {
    if (int r = check_step_args(ctx, sp, f, dt, omega)) return r;
    if (!dG) return fail(ETPIC_EINVAL, "null current accumulator");
    if (int r = check_particles(ctx, p)) return r;
    if (nsteps < 1 || hist0 < 0) return fail(ETPIC_EINVAL, "need nsteps >= 1 and hist0 >= 0");
    if (int r = check_precision(precision, false)) return r;
    if (!hist || hist_bytes < ds_history_size(p->n, precision))
        return fail(ETPIC_EINVAL, "history buffer missing or smaller than etpic_ds_history_bytes");
    if ((reinterpret_cast<uintptr_t>(hist) & 7) != 0) return fail(ETPIC_EINVAL, "history buffer not 8-byte aligned");
    if (p->n == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    if (precision == ETPIC_FP64)
        return ctx->ds_steps<double>(p, hist, sp, f, step0, nsteps, hist0, dt, omega, dG, rho, flags, stream);
    return ctx->ds_steps<float>(p, hist, sp, f, step0, nsteps, hist0, dt, omega, dG, rho, flags, stream);
}

int etpic_ds_sort(etpic_ctx *ctx, const etpic_particles *src, const etpic_particles *dst, int precision,
                  const void *hist_src, void *hist_dst, size_t hist_bytes, void *stream) {
    if (int r = check_sort_pair(ctx, src, dst)) return r;
    if (int r = check_precision(precision, false)) return r;
    const size_t need = ds_history_size(src->n, precision);
    if (!hist_src || !hist_dst || hist_bytes < need)
        return fail(ETPIC_EINVAL, "history buffers missing or smaller than etpic_ds_history_bytes");
    if (hist_src == hist_dst) return fail(ETPIC_EINVAL, "sort needs distinct history buffers");
    if (((reinterpret_cast<uintptr_t>(hist_src) | reinterpret_cast<uintptr_t>(hist_dst)) & 7) != 0)
        return fail(ETPIC_EINVAL, "history buffers not 8-byte aligned");
    if (src->n == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (precision == ETPIC_FP64)
        return ctx->sort<double>(src, dst, st, static_cast<const double *>(hist_src), static_cast<double *>(hist_dst),
                                 kDsArrays);
    return ctx->sort<float>(src, dst, st, static_cast<const float *>(hist_src), static_cast<float *>(hist_dst),
                            kDsArrays);
}

int etpic_adjoint_workspace(const etpic_ctx *ctx, int64_t n, int nsteps, int checkpoint_every, size_t *bytes_out) {
    if (!ctx || !bytes_out) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (n < 0 || nsteps < 0 || checkpoint_every < 1) return fail(ETPIC_EINVAL, "bad sizes");
    *bytes_out = adj_layout(n, ctx->host.ne, nsteps, checkpoint_every).total;
    return ETPIC_OK;
}

// nsteps float64 steps from one state buffer into another (see fused_steps).
static int adjoint_forward(etpic_ctx *ctx, const etpic_particles &from, const etpic_particles &to,
                           const etpic_species *sp, const etpic_fields *f, int64_t step0, int nsteps, double dt,
                           double omega, double *dG, hipStream_t st, etpic_ctx::Segment *seg) {
    std::vector<StepPlan> plans((size_t)nsteps);
    for (int j = 0; j < nsteps; ++j)
        plans[j] = StepPlan{{f, nullptr, nullptr}, {1.0, 0.0, 0.0}, (double)(step0 + j) * dt};
    return ctx->fused_steps<double, 1, false>(&to, sp, plans.data(), nsteps, ctx->most_fused(to.n), dt, omega, dG, nullptr,
                                              ETPIC_STEP_XCD_REMAP, st, &from, false, seg);
}

int etpic_forward_checkpointed(etpic_ctx *ctx, const etpic_particles *p, const etpic_species *sp,
                               const etpic_fields *f, int64_t step0, int nsteps, double dt, double omega,
                               int checkpoint_every, void *workspace, size_t workspace_bytes, double *dG,
                               void *stream) {
    if (int r = check_step_args(ctx, sp, f, dt, omega)) return r;
    if (int r = check_particles(ctx, p)) return r;
    if (nsteps < 0 || checkpoint_every < 1 || !workspace) return fail(ETPIC_EINVAL, "bad sizes or null workspace");
    const AdjLayout L = adj_layout(p->n, ctx->host.ne, nsteps, checkpoint_every);
    if (workspace_bytes < L.total) return fail(ETPIC_EINVAL, "workspace too small (%zu < %zu)", workspace_bytes, L.total);
    if (p->n == 0 || nsteps == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    double *acc = dG ? dG : reinterpret_cast<double *>(static_cast<char *>(workspace) + L.dG_off);
    // the state goes from checkpoint to checkpoint, the last segment's into p
    const int64_t n = p->n;
    k_copy_state<<<grid_for(n), kBlock, 0, st>>>(*p, state_view(workspace, 0, L, n));
    HIP_TRY(hipGetLastError());
    etpic_ctx::Segment part{};
    for (int seg = 0; seg < L.ncp; ++seg) {
        const int k0 = seg * checkpoint_every, k1 = std::min(nsteps, k0 + checkpoint_every);
        const etpic_particles from = state_view(workspace, (size_t)seg * L.state, L, n);
        const etpic_particles to = seg + 1 < L.ncp ? state_view(workspace, (size_t)(seg + 1) * L.state, L, n) : *p;
        // (the currents of all segments gather in the slots and go to dG after the last)
        part.goes_on = seg > 0;
        part.last = seg + 1 == L.ncp;
        if (int r = adjoint_forward(ctx, from, to, sp, f, step0 + k0, k1 - k0, dt, omega, acc, st, &part)) return r;
    }
    return ETPIC_OK;
}

int etpic_backward(etpic_ctx *ctx, int64_t n, const etpic_species *sp, const etpic_fields *f, int64_t step0,
                   int nsteps, double dt, double omega, int checkpoint_every, void *workspace,
                   size_t workspace_bytes, double *const vbar[3], double *const xbar[3], double *grad_e,
                   void *stream) {
    if (int r = check_step_args(ctx, sp, f, dt, omega)) return r;
    if (n < 0 || nsteps < 0 || checkpoint_every < 1 || !workspace || !grad_e || !vbar || !xbar)
        return fail(ETPIC_EINVAL, "bad sizes or null pointer");
    for (int k = 0; k < 3; ++k)
        if (!vbar[k] || !xbar[k]) return fail(ETPIC_EINVAL, "null adjoint array");
    if (n > (int64_t)kWalkQueueCap * 64) return fail(ETPIC_EINVAL, "particle count above 2^29");
    const AdjLayout L = adj_layout(n, ctx->host.ne, nsteps, checkpoint_every);
    if (workspace_bytes < L.total) return fail(ETPIC_EINVAL, "workspace too small (%zu < %zu)", workspace_bytes, L.total);
    if (n == 0 || nsteps == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    double *scratch_dG = reinterpret_cast<double *>(static_cast<char *>(workspace) + L.dG_off);
    {
        const etpic_fields *snap[3] = {f, nullptr, nullptr};
        const double w1[3] = {1.0, 0.0, 0.0};
        if (int r = ctx->launch_parts<1>(snap, w1, nullptr, st, nullptr)) return r;
    }
    // both counter sets of the sweep, all parts of each: a launch's leavers
    // kernel clears the other set only
    unsigned *const ctr = ctx->d_walk_ctr + 3 * kCtrStride;
    k_fill_u32<<<grid_for(2 * kCtrStride), kBlock, 0, st>>>(ctr, 2 * kCtrStride, 0u);
    HIP_TRY(hipGetLastError());
    unsigned flip = 0;
    for (int seg = L.ncp - 1; seg >= 0; --seg) {
        // the segment in pieces of at most kMaxAdj steps: the states its later
        // pieces start from are recomputed into the slots first, the slots
        // after them take the per-step states of the particles that leave
        const int k0 = seg * checkpoint_every, len = std::min(nsteps, k0 + checkpoint_every) - k0;
        const int pieces = (len + kMaxAdj - 1) / kMaxAdj;
        auto begin = [&](int i) { return k0 + (int)((int64_t)len * i / pieces); };
        auto start = [&](int i) {
            return i == 0 ? state_view(workspace, (size_t)seg * L.state, L, n)
                          : state_view(workspace, L.slots_off + (size_t)(i - 1) * L.state, L, n);
        };
        etpic_ctx::Segment part{true, false, 0};   // (what it leaves in the slots is not wanted)
        for (int i = 1; i < pieces; ++i) {
            part.last = i + 1 == pieces;
            if (int r = adjoint_forward(ctx, start(i - 1), start(i), sp, f, step0 + begin(i - 1),
                                        begin(i) - begin(i - 1), dt, omega, scratch_dG, st, &part))
                return r;
        }
        for (int i = pieces - 1; i >= 0; --i) {
            const etpic_particles cur = start(i);
            const StepArgs<double> base = ctx->step_args<double>(&cur, sp, dt, scratch_dG, nullptr);
            AdjArgs b{};
            b.parts = static_cast<const double *>(ctx->d_coef);
            b.tet = cur.tet;
            b.grad_e = grad_e;
            b.nsteps = begin(i + 1) - begin(i);
            for (int k = 0; k < 3; ++k) {
                b.lam[k] = cur.lam[k];
                b.v[k] = static_cast<const double *>(cur.vel[k]);
                b.vb[k] = vbar[k];
                b.xb[k] = xbar[k];
            }
            for (int j = 0; j < b.nsteps; ++j) {
                const double t = (double)(step0 + begin(i) + j) * dt;
                b.c[j] = std::cos(omega * t);
                b.s[j] = std::sin(omega * t);
                const etpic_particles q = state_view(workspace, L.slots_off + (size_t)(pieces - 1 + j) * L.state, L, n);
                for (int k = 0; k < 3; ++k) {
                    b.s_lam[j][k] = q.lam[k];
                    b.s_v[j][k] = static_cast<double *>(q.vel[k]);
                }
                b.s_tet[j] = q.tet;
            }
            // at most kWalkQueueCap particles per launch: the queue holds all that leave
            for (int64_t first = 0; first < n; first += kWalkQueueCap) {
                b.first = first;
                b.end = std::min<int64_t>(n, first + kWalkQueueCap);
                StepArgs<double> a = base;
                a.walk_ctr = ctr + flip * kCtrStride;
                flip ^= 1;
                k_adjoint<<<(unsigned)((b.end - b.first + 63) / 64), 64, 0, st>>>(a, b);
                HIP_TRY(hipGetLastError());
                k_adjoint_leavers<<<kLeaverBlocks, kBlock, 0, st>>>(a, b, ctr + flip * kCtrStride);
                HIP_TRY(hipGetLastError());
            }
        }
    }
    return ETPIC_OK;
}

int etpic_particles_locate(etpic_ctx *ctx, const etpic_particles *p, int precision, const double *const xyz[3],
                           const int32_t *hint, void *stream) {
    if (!ctx || !p || !xyz) return fail(ETPIC_EINVAL, "null argument");
    if (int r = check_precision(precision, true)) return r;
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (p->n < 0 || p->n > (int64_t)kWalkQueueCap * 64) return fail(ETPIC_EINVAL, "particle count outside [0, 2^29]");
    if (p->n == 0) return ETPIC_OK;
    if (!p->lam[0] || !p->lam[1] || !p->lam[2] || !p->tet || !xyz[0] || !xyz[1] || !xyz[2])
        return fail(ETPIC_EINVAL, "null particle or position array");
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned *fails = reinterpret_cast<unsigned *>(ctx->d_red);
    k_fill_u32<<<1, kBlock, 0, st>>>(fails, 1, 0u);
    k_locate<<<grid_for(p->n), kBlock, 0, st>>>(p->n, xyz[0], xyz[1], xyz[2], hint, ctx->host.nt, ctx->d_topo,
                                                ctx->d_grad64, ctx->d_xyz, ctx->grid, p->lam[0], p->lam[1],
                                                p->lam[2], p->tet, fails, precision == ETPIC_MIXED_FIXED ? 1 : 0);
    HIP_TRY(hipGetLastError());
    unsigned nfail = 0;
    HIP_TRY(hipMemcpyAsync(&nfail, fails, sizeof nfail, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (nfail)
        return fail(ETPIC_EPARTICLE, "%u of %lld points not located (outside the mesh, non-finite, or not reachable by "
                    "a straight walk from the start tet); their tet is set to -1", nfail, (long long)p->n);
    return ETPIC_OK;
}

int etpic_particles_positions(etpic_ctx *ctx, const etpic_particles *p, int precision, double *const xyz[3],
                              void *stream) {
    if (!ctx || !p || !xyz) return fail(ETPIC_EINVAL, "null argument");
    if (int r = check_precision(precision, true)) return r;
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (p->n < 0 || p->n > (int64_t)kWalkQueueCap * 64) return fail(ETPIC_EINVAL, "particle count outside [0, 2^29]");
    if (p->n == 0) return ETPIC_OK;
    if (!p->lam[0] || !p->lam[1] || !p->lam[2] || !p->tet || !xyz[0] || !xyz[1] || !xyz[2])
        return fail(ETPIC_EINVAL, "null particle or position array");
    if (int r = set_device(ctx)) return r;
    k_positions<<<grid_for(p->n), kBlock, 0, static_cast<hipStream_t>(stream)>>>(
        p->n, ctx->host.nt, p->lam[0], p->lam[1], p->lam[2], p->tet, ctx->d_topo, ctx->d_xyz, xyz[0], xyz[1], xyz[2],
        ctx->d_status, precision == ETPIC_MIXED_FIXED ? 1 : 0);
    HIP_TRY(hipGetLastError());
    return ETPIC_OK;
}

// ------------------------------------------------------------------ checkpoints
namespace {
// the particle arrays in the checkpoint file's order
void particle_arrays(const etpic_particles *p, void *arr[etpic::ckpt::kArrays]) {
    arr[0] = p->tet;
    for (int k = 0; k < 3; ++k) {
        arr[1 + k] = p->lam[k];
        arr[4 + k] = p->vel[k];
    }
    arr[7] = p->id;
}
}  // namespace

int etpic_checkpoint_write(etpic_ctx *ctx, const etpic_particles *p, int precision, int64_t step, const char *path,
                           void *stream) {
    if (!ctx || !p || !path) return fail(ETPIC_EINVAL, "null argument");
    if (int r = check_precision(precision, true)) return r;
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (int r = check_particles(ctx, p)) return r;
    if (int r = set_device_only(ctx)) return r;
    etpic::ckpt::Header h{};
    h.precision = (uint32_t)precision;
    h.n = p->n;
    h.step = step;
    h.n_tet = ctx->host.nt;
    h.n_vert = ctx->host.nv;
    h.mesh_hash = ctx->mesh_hash;
    h.has_id = p->id ? 1u : 0u;
    void *arr[etpic::ckpt::kArrays];
    particle_arrays(p, arr);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t herr = hipSuccess;
    auto fetch = [&](int k, size_t off, void *buf, size_t len) -> std::string {
        herr = hipMemcpyAsync(buf, static_cast<const char *>(arr[k]) + off, len, hipMemcpyDeviceToHost, st);
        if (herr == hipSuccess) herr = hipStreamSynchronize(st);
        return herr == hipSuccess ? std::string() : std::string("device to host copy: ") + hipGetErrorString(herr);
    };
    const std::string e = etpic::ckpt::write(path, h, fetch);
    if (!e.empty()) return fail(herr != hipSuccess ? ETPIC_EHIP : ETPIC_EIO, "checkpoint write: %s", e.c_str());
    return ETPIC_OK;
}

int etpic_checkpoint_info(const char *path, int64_t *n, int *precision, int64_t *step, int *has_id) {
    if (!path) return fail(ETPIC_EINVAL, "null path");
    etpic::ckpt::Header h{};
    const std::string e = etpic::ckpt::read_header(path, h);
    if (!e.empty()) return fail(ETPIC_EIO, "checkpoint: %s", e.c_str());
    if (n) *n = h.n;
    if (precision) *precision = (int)h.precision;
    if (step) *step = h.step;
    if (has_id) *has_id = (int)h.has_id;
    return ETPIC_OK;
}

int etpic_checkpoint_read(etpic_ctx *ctx, const etpic_particles *p, int precision, const char *path, int64_t *step,
                          void *stream) {
    if (!ctx || !p || !path) return fail(ETPIC_EINVAL, "null argument");
    if (int r = check_precision(precision, true)) return r;
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (int r = check_particles(ctx, p)) return r;
    etpic::ckpt::Header h{};
    {
        const std::string e = etpic::ckpt::read_header(path, h);
        if (!e.empty()) return fail(ETPIC_EIO, "checkpoint: %s", e.c_str());
    }
    if ((int)h.precision != precision)
        return fail(ETPIC_EINVAL, "checkpoint precision %u, particles given as %d", h.precision, precision);
    if (h.n != p->n)
        return fail(ETPIC_EINVAL, "checkpoint holds %lld particles, arrays hold %lld", (long long)h.n, (long long)p->n);
    if (h.n > 0 && (h.has_id != 0) != (p->id != nullptr))
        return fail(ETPIC_EINVAL, h.has_id ? "checkpoint has particle ids, no id array given"
                                           : "checkpoint has no particle ids, an id array was given");
    if (h.n_tet != ctx->host.nt || h.n_vert != ctx->host.nv || h.mesh_hash != ctx->mesh_hash)
        return fail(ETPIC_EMESH, "checkpoint taken on another mesh (%lld tets, %lld vertices)", (long long)h.n_tet,
                    (long long)h.n_vert);
    if (int r = set_device_only(ctx)) return r;
    void *arr[etpic::ckpt::kArrays];
    particle_arrays(p, arr);
    hipStream_t st = static_cast<hipStream_t>(stream);
    hipError_t herr = hipSuccess;
    auto store = [&](int k, size_t off, void *buf, size_t len) -> std::string {
        herr = hipMemcpyAsync(static_cast<char *>(arr[k]) + off, buf, len, hipMemcpyHostToDevice, st);
        if (herr == hipSuccess) herr = hipStreamSynchronize(st);
        return herr == hipSuccess ? std::string() : std::string("host to device copy: ") + hipGetErrorString(herr);
    };
    const std::string e = etpic::ckpt::read(path, h, store);
    if (!e.empty()) return fail(herr != hipSuccess ? ETPIC_EHIP : ETPIC_EIO, "checkpoint read: %s", e.c_str());
    if (step) *step = h.step;
    return ETPIC_OK;
}

int etpic_vertex_charge(etpic_ctx *ctx, const etpic_particles *p, int precision, const etpic_species *sp, double *rho,
                        void *stream) {
    if (!ctx || !sp || !rho) return fail(ETPIC_EINVAL, "null argument");
    if (int r = check_precision(precision, true)) return r;
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (int r = check_particles(ctx, p)) return r;
    if (p->n == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int fixed = precision == ETPIC_MIXED_FIXED ? 1 : 0;
    const int64_t n = p->n;
    k_charge<<<grid_for((n + kChargePer - 1) / kChargePer), kBlock, 0, st>>>(
        n, ctx->host.nt, p->lam[0], p->lam[1], p->lam[2], p->tet, ctx->d_topo, sp->q * sp->w, rho, ctx->d_status,
        fixed);
    HIP_TRY(hipGetLastError());
    return ETPIC_OK;
}

int etpic_gauss_residual(etpic_ctx *ctx, const double *dG, const double *rho_new, const double *rho_old,
                         double out_host[2], void *stream) {
    if (!ctx || !dG || !rho_new || !rho_old || !out_host) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t nv = ctx->host.nv;
    const int nblk = (int)std::min<int64_t>(std::max<int64_t>(grid_for(nv), 1), kResBlocks);
    double *part = reinterpret_cast<double *>(ctx->d_red);
    // the pair goes straight to the context's pinned words: no copy to wait for
    double *res = reinterpret_cast<double *>(ctx->h_runstat + 1);
    k_gauss_part<<<nblk, kBlock, 0, st>>>(nv, ctx->d_v2e_ptr, ctx->d_v2e_code, dG, rho_new, rho_old, part);
    k_gauss_final<<<1, kBlock, 0, st>>>(part, nblk, res);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(st));
    out_host[0] = res[0];
    out_host[1] = res[1];
    if (!std::isfinite(out_host[0]) || !std::isfinite(out_host[1]))
        return fail(ETPIC_ENAN, "continuity residual: non-finite current or charge (max|r| %g, max|rho_old| %g)",
                    out_host[0], out_host[1]);
    return ETPIC_OK;
}

int etpic_stream_probe(etpic_ctx *ctx, const etpic_particles *p, int precision, uint32_t flags, void *stream) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    if (int r = check_particles(ctx, p)) return r;
    if (int r = check_precision(precision, true)) return r;
    if (p->n == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int remap = (flags & ETPIC_STEP_XCD_REMAP) ? 1 : 0;
    if (precision == ETPIC_FP64)
        k_stream<double><<<grid_for(p->n), kBlock, 0, st>>>(
            p->n, p->lam[0], p->lam[1], p->lam[2], static_cast<double *>(p->vel[0]), static_cast<double *>(p->vel[1]),
            static_cast<double *>(p->vel[2]), p->tet, 0.0, remap, 0);
    else
        k_stream<float><<<grid_for(p->n), kBlock, 0, st>>>(
            p->n, p->lam[0], p->lam[1], p->lam[2], static_cast<float *>(p->vel[0]), static_cast<float *>(p->vel[1]),
            static_cast<float *>(p->vel[2]), p->tet, 0.0, remap, precision == ETPIC_MIXED_FIXED ? 1 : 0);
    HIP_TRY(hipGetLastError());
    return ETPIC_OK;
}

int etpic_gauss_residual_noalloc(etpic_ctx *ctx, const double *dG, const double *rho_new, const double *rho_old,
                                 double out_host[2], void *stream) {
    if (!ctx || !dG || !rho_new || !rho_old || !out_host) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (!ctx->d_scratch) return fail(ETPIC_ESTATE, "residual scratch address not taken");
    const int64_t nv = ctx->host.nv;
    if (nv > (int64_t)INT32_MAX) return fail(ETPIC_EINVAL, "%lld vertices beyond the 32-bit limit", (long long)nv);
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int nblk = (int)std::min<int64_t>(std::max<int64_t>(grid_for(nv), 1), kResBlocks);
    double *part = ctx->d_scratch, *res = ctx->d_scratch + 2 * kResBlocks;
    k_gauss_part<<<nblk, kBlock, 0, st>>>(nv, ctx->d_v2e_ptr, ctx->d_v2e_code, dG, rho_new, rho_old, part);
    k_gauss_final<<<1, kBlock, 0, st>>>(part, nblk, res);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(out_host, res, 2 * sizeof(double), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (!std::isfinite(out_host[0]) || !std::isfinite(out_host[1]))
        return fail(ETPIC_ENAN, "continuity residual: non-finite current or charge (max|r| %g, max|rho_old| %g)",
                    out_host[0], out_host[1]);
    return ETPIC_OK;
}

int etpic_sort(etpic_ctx *ctx, const etpic_particles *src, const etpic_particles *dst, int precision,
               void *stream) {
    if (int r = check_sort_pair(ctx, src, dst)) return r;
    if (int r = check_precision(precision, true)) return r;
    if (src->n == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (precision == ETPIC_FP64) return ctx->sort<double>(src, dst, st);
    return ctx->sort<float>(src, dst, st, nullptr, nullptr, 0, precision == ETPIC_MIXED_FIXED ? 1 : 0);
}

}  // extern "C"

namespace {

// Iterations of a solve: launch(k, false) enqueues iteration k, whose product
// kernel first tests the residual of the ones before and reports in W;
// launch(max_iter, true) the test alone.  The host enqueues up to kSolveLead
// iterations beyond the last report, so the device never waits for it (a read
// of the scalars every 5 or 10 iterations left it idle for 25 us each time:
// two steps of the coupled loop on 59,900 edges 7.9 -> 6.6 ms with the loads
// below, a field step on 460,000 edges 2.30 -> 2.17 ms); those enqueued past
// convergence return at once.  Returns once the stream has drained, the last
// report in W.
constexpr int kSolveLead = kSolveReport + 2;

template <typename Launch>
int watch_solve(SolveWatch &W, hipStream_t st, int max_iter, Launch &&launch) {
    __atomic_store_n(&W.word, 0ull, __ATOMIC_RELAXED);
    W.r2 = W.b2 = 0.0;
    for (int k = 0; k <= max_iter; ++k) {
        unsigned long long w = 0;
        for (unsigned spins = 1;; ++spins) {
            w = __atomic_load_n(&W.word, __ATOMIC_RELAXED);
            if ((w & 1) || (int64_t)(w >> 1) > (int64_t)k - kSolveLead) break;
            // an error, or a stream that ran dry without a report, ends the wait
            if ((spins & 1023) == 0 && hipStreamQuery(st) != hipErrorNotReady) {
                w = __atomic_load_n(&W.word, __ATOMIC_RELAXED);
                if ((w & 1) || (int64_t)(w >> 1) > (int64_t)k - kSolveLead) break;
                HIP_TRY(hipStreamSynchronize(st));
                return fail(ETPIC_EHIP, "solver: no report from iteration %d", k - kSolveLead);
            }
        }
        if (w & 1) break;
        launch(k, k == max_iter);
        HIP_TRY(hipGetLastError());
    }
    HIP_TRY(hipStreamSynchronize(st));
    return ETPIC_OK;
}

// A solve in one launch: launch(blocks) enqueues it for `rows` rows.  Not
// tried (kNotTried) if there are more rows than one block per CU takes
// (kResMaxBlocks x kResRows = 65,536: their vectors and matrix entries fill the
// registers) or if the last trials say so; kFailed if the blocks did
// not meet or one left a wait: the start has to be enqueued again then.
enum OneLaunch { kNotTried, kTook, kFailed };

template <typename Launch>
int resident_solve(SolveWatch &W, etpic::OneLaunchTrials &trials, hipStream_t st, int64_t rows, OneLaunch &way,
                   Launch &&launch) {
    way = kNotTried;
    const int64_t blocks = (rows + kResRows - 1) / kResRows;
    if (blocks > kResMaxBlocks || !trials.tries()) return ETPIC_OK;
    __atomic_store_n(&W.word, 0ull, __ATOMIC_RELAXED);
    __atomic_store_n(&W.gave_up, 0ull, __ATOMIC_RELAXED);
    launch((unsigned)blocks);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(st));
    way = etpic::one_launch_took(W) ? kTook : kFailed;
    trials.ended(way == kTook);
    return ETPIC_OK;
}

// Field solver arrays: CSR row pointers, columns, M and K values, Dirichlet
// mask, face -> edge table, Jacobi inverse diagonal, 9 complex work vectors,
// block partials and the 12 iteration scalars.
struct FieldPtrs2 {
    int32_t *rowptr, *col, *face_edge;
    double *M, *K, *partial, *sc;
    uint8_t *dir;
    double2 *dinv, *vec;
};
FieldPtrs2 field_layout(Carve &cv, int64_t ne, int64_t nf, int64_t nnz) {
    FieldPtrs2 f;
    const int64_t nb = std::max<int64_t>(grid_for(ne), kNsBlocks);
    f.rowptr = cv.take<int32_t>(ne + 1);
    f.col = cv.take<int32_t>(nnz);
    f.M = cv.take<double>(nnz);
    f.K = cv.take<double>(nnz);
    f.dir = cv.take<uint8_t>(ne);
    f.face_edge = cv.take<int32_t>(3 * nf);
    f.dinv = cv.take<double2>(ne);
    f.vec = cv.take<double2>(9 * ne);
    f.partial = cv.take<double>(4 * (nb + kNsBlocks) + kResSlots);
    f.sc = cv.take<double>(12);
    return f;
}

// The host field system for (eps, mu): the one a size query built, else a new one.
int field_system(etpic_ctx *ctx, double eps, double mu) {
    if (ctx->field_pending && ctx->field_pending_eps == eps && ctx->field_pending_mu == mu) return ETPIC_OK;
    std::string err;
    auto S = std::make_unique<etpic::FieldSystem>();
    if (etpic::build_field_system(ctx->host, eps, mu, *S, err) != 0) return fail(ETPIC_EINVAL, "field: %s", err.c_str());
    ctx->field_pending = std::move(S);
    ctx->field_pending_eps = eps;
    ctx->field_pending_mu = mu;
    return ETPIC_OK;
}

}  // namespace

extern "C" {

int etpic_field_bytes(etpic_ctx *ctx, double eps, double mu, size_t *bytes) {
    if (!ctx || !bytes) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (!(eps > 0.0) || !(mu > 0.0)) return fail(ETPIC_EINVAL, "eps, mu must be positive");
    if (int r = field_system(ctx, eps, mu)) return r;
    const etpic::FieldSystem &S = *ctx->field_pending;
    Carve cv;
    (void)field_layout(cv, S.ne, S.nf, S.nnz);
    *bytes = cv.used;
    return ETPIC_OK;
}

int etpic_field_setup(etpic_ctx *ctx, double dt, double omega, double eps, double mu, void *dev_buf, size_t bytes) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (!(dt > 0.0) || !std::isfinite(omega) || !(eps > 0.0) || !(mu > 0.0))
        return fail(ETPIC_EINVAL, "dt, eps, mu must be positive and omega finite");
    if (int r = field_system(ctx, eps, mu)) return r;
    const etpic::FieldSystem &S = *ctx->field_pending;
    size_t need = 0;
    {
        Carve cv;
        (void)field_layout(cv, S.ne, S.nf, S.nnz);
        need = cv.used;
    }
    if (int r = check_buffer(dev_buf, bytes, need, "field")) return r;
    const int64_t ne = S.ne;
    // Jacobi preconditioner: inverse diagonal of A = alpha M + beta K
    const double ar = 1.0 - 0.25 * omega * omega * dt * dt, ai = omega * dt, beta = 0.25 * dt * dt;
    std::vector<double2> dinv((size_t)ne);
    for (int64_t i = 0; i < ne; ++i) {
        double mii = 0.0, kii = 0.0;
        for (int32_t j = S.rowptr[i]; j < S.rowptr[i + 1]; ++j)
            if (S.col[j] == i) {
                mii = S.M[j];
                kii = S.K[j];
            }
        const double dr = ar * mii + beta * kii, di = ai * mii, den = dr * dr + di * di;
        if (!(den > 0.0)) return fail(ETPIC_EMESH, "field: zero diagonal at edge %lld", (long long)i);
        dinv[i] = make_double2(dr / den, -di / den);
    }
    if (int r = set_device_only(ctx)) return r;
    HIP_TRY(hipDeviceSynchronize());
    FieldState &F = ctx->field;
    F.release();
    F.dt = dt;
    F.omega = omega;
    F.eps = eps;
    F.mu = mu;
    F.ne = S.ne;
    F.nf = S.nf;
    F.nnz = S.nnz;
    F.nb = std::max<int64_t>(grid_for(ne), kNsBlocks);
    Carve cv;
    cv.base = static_cast<char *>(dev_buf);
    cv.cap = bytes;
    const FieldPtrs2 f = field_layout(cv, S.ne, S.nf, S.nnz);
    F.rowptr = f.rowptr;
    F.col = f.col;
    F.M = f.M;
    F.K = f.K;
    F.dir = f.dir;
    F.face_edge = f.face_edge;
    F.dinv = f.dinv;
    F.vec = f.vec;
    F.partial = f.partial;
    F.sc = f.sc;
    HIP_TRY(hipMemcpy(F.rowptr, S.rowptr.data(), sizeof(int32_t) * (ne + 1), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(F.col, S.col.data(), sizeof(int32_t) * S.nnz, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(F.M, S.M.data(), sizeof(double) * S.nnz, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(F.K, S.K.data(), sizeof(double) * S.nnz, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(F.dir, S.dirichlet.data(), sizeof(uint8_t) * ne, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(F.face_edge, S.face_edge.data(), sizeof(int32_t) * 3 * S.nf, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(F.dinv, dinv.data(), sizeof(double2) * ne, hipMemcpyHostToDevice));
    F.ready = true;
    ctx->field_pending.reset();
    return ETPIC_OK;
}

int etpic_field_nnz(const etpic_ctx *ctx, int64_t *nnz_out) {
    if (!ctx || !nnz_out) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->field.ready) return fail(ETPIC_ESTATE, "etpic_field_setup not called");
    *nnz_out = ctx->field.nnz;
    return ETPIC_OK;
}

int etpic_field_spmv(etpic_ctx *ctx, const double *x, double *y, double alpha_re, double alpha_im, double beta,
                     void *stream) {
    if (!ctx || !x || !y) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->field.ready) return fail(ETPIC_ESTATE, "etpic_field_setup not called");
    if (int r = set_device(ctx)) return r;
    const FieldState &F = ctx->field;
    k_field_spmv<<<grid_for(F.ne * kRowLanes), kBlock, 0, static_cast<hipStream_t>(stream)>>>(
        F.csr(), make_double2(alpha_re, alpha_im), beta, reinterpret_cast<const double2 *>(x),
        reinterpret_cast<double2 *>(y));
    HIP_TRY(hipGetLastError());
    return ETPIC_OK;
}

int etpic_field_step(etpic_ctx *ctx, double t_next, double *u, double *v, double *a, double *b, const double *gdd,
                     double tol, int max_iter, int *iters_out, double *resid_out, void *stream) {
    if (!ctx || !u || !v || !a || !b) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->field.ready) return fail(ETPIC_ESTATE, "etpic_field_setup not called");
    if (!(tol > 0.0) || max_iter < 1 || !std::isfinite(t_next)) return fail(ETPIC_EINVAL, "bad tol / max_iter / time");
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const FieldState &F = ctx->field;
    const int64_t ne = F.ne;
    const unsigned ge = grid_for(ne), gr = grid_for(ne * kRowLanes);
    const double dt = F.dt, w = F.omega;
    const double2 alpha = make_double2(1.0 - 0.25 * w * w * dt * dt, w * dt);
    const double beta = 0.25 * dt * dt;
    const double c = std::cos(w * t_next), s = std::sin(w * t_next);
    double2 *U = reinterpret_cast<double2 *>(u), *V = reinterpret_cast<double2 *>(v), *A = reinterpret_cast<double2 *>(a);
    double2 *us = F.v(0), *vs = F.v(1), *wv = F.v(2), *rhs = F.v(3), *x = F.v(4), *r = F.v(5), *z = F.v(6), *p = F.v(7),
            *q = F.v(8);
    k_nm_predict<<<ge, kBlock, 0, st>>>(ne, U, V, A, us, vs, wv, dt, w);
    k_nm_rhs<<<gr, kBlock, 0, st>>>(F.csr(), wv, us, gdd, c, s, rhs);
    // partial sets: the start and the update write the first, the product the second
    double *pa = F.partial, *pb = F.partial + 4 * F.nb;
    const unsigned ga = (unsigned)std::min<int64_t>((ne * kRowLanes + kNsThreads - 1) / kNsThreads, kNsBlocks);
    const unsigned gu = (unsigned)std::min<int64_t>((ne + kNsVecThreads - 1) / kNsVecThreads, kNsBlocks);
    const double tol2 = tol * tol;
    SolveWatch &W = *ctx->h_watch;
    auto start = [&] {
        k_cocg_init<<<ge, kBlock, 0, st>>>(ne, rhs, F.dinv, x, r, z, p, q, pa, F.sc);
    };
    start();
    HIP_TRY(hipGetLastError());
    unsigned long long *slots = reinterpret_cast<unsigned long long *>(F.partial + 4 * (F.nb + kNsBlocks));
    OneLaunch way;
    if (int rc = resident_solve(W, ctx->field_trials, st, ne, way, [&](unsigned blocks) {
            k_cocg_resident<<<blocks, kResThreads, 0, st>>>(F.csr(), alpha, beta, F.sc, F.dinv, x, r, z, pa, ge, slots,
                                                            tol2, max_iter, &W);
        }))
        return rc;
    if (way == kFailed) start();
    if (way != kTook) if (int rc = watch_solve(W, st, max_iter, [&](int k, bool check_only) {
            k_cocg_apply<<<ga, kNsThreads, 0, st>>>(F.csr(), alpha, beta, F.sc, z, p, q, pa, k == 0 ? (int64_t)ge : gu,
                                                    pb, k, tol2, check_only ? 1 : 0, &W);
            if (!check_only)
                k_cocg_update<<<gu, kNsVecThreads, 0, st>>>(ne, F.sc, F.dinv, p, q, x, r, z, pb, ga, pa, k);
        }))
        return rc;
    const double rel = W.b2 > 0.0 ? std::sqrt(W.r2 / W.b2) : 0.0;
    const int it = (int)(W.word >> 1) - 1;
    if (iters_out) *iters_out = it;
    if (resid_out) *resid_out = rel;
    if (!(W.word & 1) || !std::isfinite(rel)) return fail(ETPIC_ENOCONV, "COCG: relative residual %.3e after %d iterations", rel, it);
    k_nm_faraday<<<grid_for(F.nf), kBlock, 0, st>>>(F.nf, F.face_edge, U, us, x, reinterpret_cast<double2 *>(b), dt, w);
    k_nm_correct<<<ge, kBlock, 0, st>>>(ne, us, vs, x, U, V, A, dt);
    HIP_TRY(hipGetLastError());
    return ETPIC_OK;
}

}  // extern "C"

namespace {

// Gauss-law solver arrays: CSR row pointers, columns, edge -> vertex table,
// values, Jacobi inverse diagonal, wall mask, 8 work vectors, block partials,
// the 12 iteration scalars, and zero face / edge envelopes.
struct NsPtrs {
    int32_t *rowptr, *col, *ev;
    double *S, *dinv, *vec, *partial, *sc, *bzero, *ezero;
    uint8_t *wall;
};
NsPtrs ns_layout(Carve &cv, int64_t nv, int64_t ne, int64_t nf, int64_t nnz) {
    NsPtrs n;
    n.rowptr = cv.take<int32_t>(nv + 1);
    n.col = cv.take<int32_t>(nnz);
    n.ev = cv.take<int32_t>(2 * ne);
    n.S = cv.take<double>(nnz);
    n.dinv = cv.take<double>(nv);
    n.wall = cv.take<uint8_t>(nv);
    n.vec = cv.take<double>(8 * nv);
    n.partial = cv.take<double>(8 * kNsBlocks + kResSlots);
    n.sc = cv.take<double>(12);
    n.bzero = cv.take<double>(2 * nf);
    n.ezero = cv.take<double>(2 * ne);
    return n;
}

int ns_system(etpic_ctx *ctx, double eps) {
    if (ctx->ns_pending && ctx->ns_pending_eps == eps) return ETPIC_OK;
    std::string err;
    auto S = std::make_unique<etpic::NsSystem>();
    if (etpic::build_ns_system(ctx->host, eps, *S, err) != 0) return fail(ETPIC_EINVAL, "ns: %s", err.c_str());
    ctx->ns_pending = std::move(S);
    ctx->ns_pending_eps = eps;
    return ETPIC_OK;
}

}  // namespace

extern "C" {

int etpic_ns_bytes(etpic_ctx *ctx, double eps, size_t *bytes) {
    if (!ctx || !bytes) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (!(eps > 0.0) || !std::isfinite(eps)) return fail(ETPIC_EINVAL, "eps must be positive");
    if (int r = ns_system(ctx, eps)) return r;
    Carve cv;
    (void)ns_layout(cv, ctx->ns_pending->nv, ctx->host.ne, ctx->host.nf, ctx->ns_pending->nnz);
    *bytes = cv.used;
    return ETPIC_OK;
}

int etpic_ns_setup(etpic_ctx *ctx, double eps, void *dev_buf, size_t bytes) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    if (!ctx->has_mesh) return fail(ETPIC_ESTATE, "no mesh uploaded");
    if (!(eps > 0.0) || !std::isfinite(eps)) return fail(ETPIC_EINVAL, "eps must be positive");
    if (int r = ns_system(ctx, eps)) return r;
    const etpic::NsSystem &S = *ctx->ns_pending;
    const int64_t nv = S.nv, ne = ctx->host.ne, nf = ctx->host.nf;
    size_t need = 0;
    {
        Carve cv;
        (void)ns_layout(cv, nv, ne, nf, S.nnz);
        need = cv.used;
    }
    if (int r = check_buffer(dev_buf, bytes, need, "ns")) return r;
    std::vector<double> dinv((size_t)nv, 0.0);
    for (int64_t i = 0; i < nv; ++i) {
        double d = 0.0;
        for (int32_t j = S.rowptr[i]; j < S.rowptr[i + 1]; ++j)
            if (S.col[j] == i) d = S.S[j];
        if (!(d > 0.0)) return fail(ETPIC_EMESH, "ns: non-positive diagonal at node %lld", (long long)i);
        dinv[i] = 1.0 / d;
    }
    if (int r = set_device_only(ctx)) return r;
    HIP_TRY(hipDeviceSynchronize());
    NsState &N = ctx->ns;
    N.release();
    N.eps = eps;
    N.nv = nv;
    N.ne = ne;
    N.nnz = S.nnz;
    for (uint8_t b : S.wall) N.n_wall += b;
    Carve cv;
    cv.base = static_cast<char *>(dev_buf);
    cv.cap = bytes;
    const NsPtrs n = ns_layout(cv, nv, ne, nf, S.nnz);
    N.rowptr = n.rowptr;
    N.col = n.col;
    N.ev = n.ev;
    N.S = n.S;
    N.dinv = n.dinv;
    N.wall = n.wall;
    N.vec = n.vec;
    N.partial = n.partial;
    N.sc = n.sc;
    N.bzero = n.bzero;
    N.ezero = n.ezero;
    HIP_TRY(hipMemset(N.sc, 0, sizeof(double) * 12));
    HIP_TRY(hipMemset(N.vec, 0, sizeof(double) * 8 * nv));
    HIP_TRY(hipMemset(N.bzero, 0, sizeof(double) * 2 * nf));
    HIP_TRY(hipMemset(N.ezero, 0, sizeof(double) * 2 * ne));
    HIP_TRY(hipMemcpy(N.rowptr, S.rowptr.data(), sizeof(int32_t) * (nv + 1), hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(N.col, S.col.data(), sizeof(int32_t) * S.nnz, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(N.ev, ctx->host.edges.data(), sizeof(int32_t) * 2 * ne, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(N.S, S.S.data(), sizeof(double) * S.nnz, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(N.dinv, dinv.data(), sizeof(double) * nv, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(N.wall, S.wall.data(), sizeof(uint8_t) * nv, hipMemcpyHostToDevice));
    HIP_TRY(hipDeviceSynchronize());
    N.ready = true;
    ctx->ns_pending.reset();
    return ETPIC_OK;
}

int etpic_ns_info(const etpic_ctx *ctx, int64_t *nnz_out, int64_t *wall_nodes_out) {
    if (!ctx || !nnz_out) return fail(ETPIC_EINVAL, "null argument");
    if (!ctx->ns.ready) return fail(ETPIC_ESTATE, "etpic_ns_setup not called");
    *nnz_out = ctx->ns.nnz;
    if (wall_nodes_out) *wall_nodes_out = ctx->ns.n_wall;
    return ETPIC_OK;
}

}  // extern "C"

namespace {

// The CG of eq. ns_equation on `st` (synchronises it), from x = 0 or, warm,
// from the x of the previous solve; outputs scaled by e^{-j w t} = c - j s.
int ns_solve_impl(etpic_ctx *ctx, const NsRhs &R, double *x, double c, double s, double2 *x_out, double2 *e_out,
                  double *edc_out, const double *edc_add, double tol, int max_iter, bool warm, int *iters_out,
                  double *resid_out, hipStream_t st) {
    const NsState &N = ctx->ns;
    const int64_t nv = N.nv;
    const unsigned gv = (unsigned)std::min<int64_t>((nv + kNsVecThreads - 1) / kNsVecThreads, kNsBlocks);
    const unsigned gr = (unsigned)std::min<int64_t>((nv * kRowLanes + kNsThreads - 1) / kNsThreads, kNsBlocks);
    double *r = N.v(1), *z = N.v(2), *p = N.v(3), *q = N.v(4);
    // partials: pa from the product (gr blocks), pb from the start and the update
    double *pa = N.partial, *pb = N.partial + 4 * kNsBlocks;
    const int64_t nb = warm ? gr : gv;
    auto start = [&] {
        if (warm)
            k_ns_start_warm<<<gr, kNsThreads, 0, st>>>(N.csr(), ctx->d_v2e_ptr, ctx->d_v2e_code, R, N.wall, N.dinv, x, r,
                                                       z, p, q, pb, N.sc);
        else
            k_ns_start<<<gv, kNsVecThreads, 0, st>>>(nv, ctx->d_v2e_ptr, ctx->d_v2e_code, R, N.wall, N.dinv, x, r, z, p, q,
                                                     pb, N.sc);
    };
    start();
    HIP_TRY(hipGetLastError());
    const double tol2 = tol * tol;
    SolveWatch &W = *ctx->h_watch;
    unsigned long long *slots = reinterpret_cast<unsigned long long *>(N.partial + 8 * kNsBlocks);
    OneLaunch way;
    if (int rc = resident_solve(W, ctx->ns_trials, st, nv, way, [&](unsigned blocks) {
            k_ns_resident<<<blocks, kResThreads, 0, st>>>(N.csr(), N.sc, N.dinv, x, r, z, pb, nb, slots, tol2, max_iter,
                                                          &W);
        }))
        return rc;
    if (way == kFailed) start();
    if (way != kTook) if (int rc = watch_solve(W, st, max_iter, [&](int k, bool check_only) {
            k_ns_apply<<<gr, kNsThreads, 0, st>>>(N.csr(), N.sc, z, p, q, pb, k == 0 ? nb : (int64_t)gv, pa, k, tol2,
                                                  check_only ? 1 : 0, &W);
            if (!check_only)
                k_ns_update<<<gv, kNsVecThreads, 0, st>>>(nv, N.sc, N.dinv, p, q, x, r, z, pa, gr, pb, k);
        }))
        return rc;
    const double bnorm2 = W.b2;
    if (!(bnorm2 > 0.0) && warm) HIP_TRY(hipMemsetAsync(x, 0, sizeof(double) * nv, st));   // no source: x = 0
    const double rel = bnorm2 > 0.0 ? std::sqrt(W.r2 / bnorm2) : 0.0;
    const int it = (int)(W.word >> 1) - 1;
    if (iters_out) *iters_out = it;
    if (resid_out) *resid_out = rel;
    if (!(W.word & 1) || !std::isfinite(rel))
        return fail(ETPIC_ENOCONV, "ns CG: relative residual %.3e after %d iterations", rel, it);
    if (x_out || e_out || edc_out)
        k_ns_out<<<grid_for(std::max(N.ne, nv)), kBlock, 0, st>>>(N.ne, nv, N.ev, x, c, s, x_out, e_out, edc_out,
                                                                  edc_add);
    HIP_TRY(hipGetLastError());
    return ETPIC_OK;
}

// The field step's source with its gradient part removed in the [*eps]
// inner product: gs = gdd - [*eps] D (D^T [*eps] D)^-1 D^T gdd, the inverse
// taken at the inner nodes (wall grounded).  On boundary edges D y = 0 and
// the field step's mass row is the identity, so gs = gdd there.  Work
// vectors: the field step's F.v(3), F.v(4); warm start from N.v(7).
int sol_source_impl(etpic_ctx *ctx, const double *gdd, double *gs, double tol, int max_iter, bool warm,
                    int *iters_out, double *resid_out, hipStream_t st) {
    const FieldState &F = ctx->field;
    double2 *dy = F.v(3), *m = F.v(4);
    if (int r = ns_solve_impl(ctx, NsRhs{gdd, nullptr, 1.0, nullptr, 0}, ctx->ns.v(7), 1.0, 0.0, nullptr, dy, nullptr,
                              nullptr, tol, max_iter, warm, iters_out, resid_out, st))
        return r;
    k_field_spmv<<<grid_for(F.ne * kRowLanes), kBlock, 0, st>>>(F.csr(), make_double2(1.0, 0.0), 0.0, dy, m);
    k_sol_add<<<grid_for(F.ne), kBlock, 0, st>>>(F.ne, gdd, m, gs);
    HIP_TRY(hipGetLastError());
    return ETPIC_OK;
}

// Both solvers set up on this context with the same eps.
int check_split_setup(const etpic_ctx *ctx) {
    if (!ctx->ns.ready) return fail(ETPIC_ESTATE, "etpic_ns_setup not called");
    if (!ctx->field.ready) return fail(ETPIC_ESTATE, "etpic_field_setup not called");
    if (std::fabs(ctx->field.eps - ctx->ns.eps) > 1e-15 * ctx->ns.eps)
        return fail(ETPIC_EINVAL, "etpic_field_setup and etpic_ns_setup were given different eps");
    return ETPIC_OK;
}

}  // namespace

extern "C" {

int etpic_ns_solve(etpic_ctx *ctx, const double *G, const double *rho0, double t, double omega, double *x_out,
                   double *e_out, double tol, int max_iter, uint32_t flags, int *iters_out, double *resid_out,
                   void *stream) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    if (!x_out && !e_out) return fail(ETPIC_EINVAL, "no output: x_out and e_out are both NULL");
    if (!ctx->ns.ready) return fail(ETPIC_ESTATE, "etpic_ns_setup not called");
    if (!(tol > 0.0) || max_iter < 1 || !std::isfinite(t) || !std::isfinite(omega))
        return fail(ETPIC_EINVAL, "bad tol / max_iter / time / omega");
    if (flags & ~(uint32_t)ETPIC_NS_WARM) return fail(ETPIC_EINVAL, "unknown flags 0x%x", flags);
    if (int r = set_device(ctx)) return r;
    return ns_solve_impl(ctx, NsRhs{G, rho0, 1.0, nullptr, 0}, ctx->ns.v(0), std::cos(omega * t),
                         std::sin(omega * t), reinterpret_cast<double2 *>(x_out), reinterpret_cast<double2 *>(e_out),
                         nullptr, nullptr, tol, max_iter, (flags & ETPIC_NS_WARM) != 0, iters_out, resid_out,
                         static_cast<hipStream_t>(stream));
}

int etpic_ns_run_steps(etpic_ctx *ctx, const etpic_particles *p, int precision, const etpic_species *sp,
                       const etpic_fields *ext, int64_t step0, int nsteps, int steps_per_solve, double dt,
                       double omega, double *G, const double *rho0, double *e_work, double tol, int max_iter,
                       uint32_t flags, int *iters_out, void *stream) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    if (!ctx->ns.ready) return fail(ETPIC_ESTATE, "etpic_ns_setup not called");
    if (!G || !e_work) return fail(ETPIC_EINVAL, "null G or e_work");
    if (ext && (!ext->e_env || !ext->b_env)) return fail(ETPIC_EINVAL, "external fields without e_env / b_env");
    if (ext && (ext->e_dc == e_work || ext->e_env == e_work || ext->b_env == e_work || ext->b_dc == e_work))
        return fail(ETPIC_EINVAL, "e_work aliases an external field array");
    if (G == e_work || (rho0 && rho0 == e_work)) return fail(ETPIC_EINVAL, "e_work aliases G or rho0");
    if (nsteps < 0 || steps_per_solve < 1) return fail(ETPIC_EINVAL, "bad step counts");
    if (!(tol > 0.0) || max_iter < 1) return fail(ETPIC_EINVAL, "bad tol / max_iter");
    const etpic_fields f{ext ? ext->e_env : ctx->ns.ezero, e_work, ext ? ext->b_env : ctx->ns.bzero,
                         ext ? ext->b_dc : nullptr};
    if (int r = check_step_args(ctx, sp, &f, dt, omega)) return r;
    if (int r = check_particles(ctx, p)) return r;
    if (int r = check_precision(precision, false)) return r;
    if (nsteps == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const uint32_t sf = flags & ~((uint32_t)ETPIC_NS_WARM | kFlagFixed);
    std::vector<StepPlan> plans((size_t)std::min(steps_per_solve, nsteps));
    int total = 0;
    for (int j = 0; j < nsteps; j += steps_per_solve) {
        const int n = std::min(steps_per_solve, nsteps - j);
        int it = 0;
        const bool warm = j > 0 || (flags & ETPIC_NS_WARM);
        if (int r = ns_solve_impl(ctx, NsRhs{G, rho0, 1.0, nullptr, 0}, ctx->ns.v(0), 1.0, 0.0, nullptr, nullptr,
                                  e_work, ext ? ext->e_dc : nullptr, tol, max_iter, warm, &it, nullptr, st)) {
            if (iters_out) *iters_out = total + it;
            return r;
        }
        total += it;
        if (p->n == 0) continue;
        for (int i = 0; i < n; ++i) plans[i] = StepPlan{{&f, nullptr, nullptr}, {1.0, 0.0, 0.0}, (double)(step0 + j + i) * dt};
        const int r = precision == ETPIC_FP64 ? ctx->run_steps<double>(p, sp, plans.data(), n, dt, omega, G, nullptr, sf, stream)
                                              : ctx->run_steps<float>(p, sp, plans.data(), n, dt, omega, G, nullptr, sf, stream);
        if (r) return r;
    }
    if (iters_out) *iters_out = total;
    return ETPIC_OK;
}

int etpic_ns_correct(etpic_ctx *ctx, const double *G, const double *rho0, double t, double omega, const double *u,
                     double *e_out, double tol, int max_iter, uint32_t flags, int *iters_out, double *resid_out,
                     void *stream) {
    if (!ctx || !u || !e_out) return fail(ETPIC_EINVAL, "null argument");
    if (int r = check_split_setup(ctx)) return r;
    if (!(tol > 0.0) || max_iter < 1 || !std::isfinite(t) || !std::isfinite(omega))
        return fail(ETPIC_EINVAL, "bad tol / max_iter / time / omega");
    if (flags & ~(uint32_t)ETPIC_NS_WARM) return fail(ETPIC_EINVAL, "unknown flags 0x%x", flags);
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const FieldState &F = ctx->field;
    NsState &N = ctx->ns;
    double2 *mu = F.v(3);   // [*eps] u (the field step's right-hand-side vector, free between steps)
    k_field_spmv<<<grid_for(F.ne * kRowLanes), kBlock, 0, st>>>(F.csr(), make_double2(1.0, 0.0), 0.0,
                                                                reinterpret_cast<const double2 *>(u), mu);
    HIP_TRY(hipGetLastError());
    const double c = std::cos(omega * t), s = std::sin(omega * t);
    const bool warm = (flags & ETPIC_NS_WARM) != 0;
    int it_re = 0, it_im = 0;
    double res_re = 0.0, res_im = 0.0;
    // e^{-j w t} (D^T G + rho0) = (c - j s)(D^T G + rho0): real and imaginary parts solved apart
    if (int r = ns_solve_impl(ctx, NsRhs{G, rho0, c, mu, 0}, N.v(5), 1.0, 0.0, nullptr, nullptr, nullptr, nullptr, tol,
                              max_iter, warm, &it_re, &res_re, st)) {
        if (iters_out) *iters_out = it_re;
        if (resid_out) *resid_out = res_re;
        return r;
    }
    if (int r = ns_solve_impl(ctx, NsRhs{G, rho0, -s, mu, 1}, N.v(6), 1.0, 0.0, nullptr, nullptr, nullptr, nullptr, tol,
                              max_iter, warm, &it_im, &res_im, st)) {
        if (iters_out) *iters_out = it_re + it_im;
        if (resid_out) *resid_out = res_im;
        return r;
    }
    if (iters_out) *iters_out = it_re + it_im;
    if (resid_out) *resid_out = std::max(res_re, res_im);
    k_ns_combine<<<grid_for(N.ne), kBlock, 0, st>>>(N.ne, N.ev, N.v(5), N.v(6), reinterpret_cast<const double2 *>(u),
                                                    reinterpret_cast<double2 *>(e_out));
    HIP_TRY(hipGetLastError());
    return ETPIC_OK;
}

int etpic_sol_source(etpic_ctx *ctx, const double *gdd, double *gs_out, double tol, int max_iter, uint32_t flags,
                     int *iters_out, double *resid_out, void *stream) {
    if (!ctx || !gdd || !gs_out) return fail(ETPIC_EINVAL, "null argument");
    if (int r = check_split_setup(ctx)) return r;
    if (!(tol > 0.0) || max_iter < 1) return fail(ETPIC_EINVAL, "bad tol / max_iter");
    if (flags & ~(uint32_t)ETPIC_NS_WARM) return fail(ETPIC_EINVAL, "unknown flags 0x%x", flags);
    if (int r = set_device(ctx)) return r;
    return sol_source_impl(ctx, gdd, gs_out, tol, max_iter, (flags & ETPIC_NS_WARM) != 0, iters_out, resid_out,
                           static_cast<hipStream_t>(stream));
}

int etpic_em_steps(etpic_ctx *ctx, const etpic_particles *p, int precision, const etpic_species *sp, int64_t step0,
                   int nsteps, double *u, double *v, double *a, double *b, double *e, double *G, double *G_hist,
                   const double *rho0, double tol, int max_iter, uint32_t flags, int *iters_out, void *stream) {
    if (!ctx || !u || !v || !a || !b || !e || !G || !G_hist) return fail(ETPIC_EINVAL, "null argument");
    if (int r = check_split_setup(ctx)) return r;
    if (nsteps < 0) return fail(ETPIC_EINVAL, "negative step count");
    if (e == u || G == G_hist || G_hist == u || G_hist == e) return fail(ETPIC_EINVAL, "aliased state arrays");
    if (!(tol > 0.0) || max_iter < 1) return fail(ETPIC_EINVAL, "bad tol / max_iter");
    const double dt = ctx->field.dt, omega = ctx->field.omega;
    const etpic_fields f{e, nullptr, b, nullptr};
    if (int r = check_step_args(ctx, sp, &f, dt, omega)) return r;
    if (int r = check_particles(ctx, p)) return r;
    if (int r = check_precision(precision, false)) return r;
    if (nsteps == 0) return ETPIC_OK;
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t ne = ctx->field.ne;
    double *h1 = G_hist, *h2 = G_hist + ne;
    const uint32_t sf = flags & ~((uint32_t)(ETPIC_NS_WARM | ETPIC_EM_SPLIT) | kFlagFixed);
    const bool split = (flags & ETPIC_EM_SPLIT) != 0;
    int total = 0;
    for (int j = 0; j < nsteps; ++j) {
        const double t = (double)(step0 + j) * dt, t_next = (double)(step0 + j + 1) * dt;
        if (p->n > 0) {
            const StepPlan plan{{&f, nullptr, nullptr}, {1.0, 0.0, 0.0}, t};
            const int r = precision == ETPIC_FP64 ? ctx->run_steps<double>(p, sp, &plan, 1, dt, omega, G, nullptr, sf, stream)
                                                  : ctx->run_steps<float>(p, sp, &plan, 1, dt, omega, G, nullptr, sf, stream);
            if (r) return r;
        }
        k_em_gdd<<<grid_for(ne), kBlock, 0, st>>>(ne, G, h1, h2, h2, 1.0 / (dt * dt));
        HIP_TRY(hipGetLastError());
        const bool warm = j > 0 || (flags & ETPIC_NS_WARM);
        int it = 0;
        if (split) {   // the solenoidal system's source
            if (int r = sol_source_impl(ctx, h2, h2, tol, max_iter, warm, &it, nullptr, st)) {
                if (iters_out) *iters_out = total + it;
                return r;
            }
            total += it;
        }
        if (int r = etpic_field_step(ctx, t_next, u, v, a, b, h2, tol, max_iter, &it, nullptr, stream)) {
            if (iters_out) *iters_out = total + it;
            return r;
        }
        total += it;
        k_em_shift<<<grid_for(ne), kBlock, 0, st>>>(ne, G, h1, h2);
        HIP_TRY(hipGetLastError());
        if (split) {   // e = u + e^{-j w t} D y, y from eq. ns_equation
            if (int r = ns_solve_impl(ctx, NsRhs{G, rho0, 1.0, nullptr, 0}, ctx->ns.v(0), std::cos(omega * t_next),
                                      std::sin(omega * t_next), nullptr, reinterpret_cast<double2 *>(e), nullptr,
                                      nullptr, tol, max_iter, warm, &it, nullptr, st)) {
                if (iters_out) *iters_out = total + it;
                return r;
            }
            k_em_add<<<grid_for(ne), kBlock, 0, st>>>(ne, reinterpret_cast<const double2 *>(u),
                                                      reinterpret_cast<double2 *>(e));
            HIP_TRY(hipGetLastError());
        } else {
            const uint32_t cf = warm ? (uint32_t)ETPIC_NS_WARM : 0u;
            if (int r = etpic_ns_correct(ctx, G, rho0, t_next, omega, u, e, tol, max_iter, cf, &it, nullptr, stream)) {
                if (iters_out) *iters_out = total + it;
                return r;
            }
        }
        total += it;
    }
    if (iters_out) *iters_out = total;
    return ETPIC_OK;
}

int etpic_kernel_time(etpic_ctx *ctx, double ms_out[4], int64_t launches_out[2], int reset) {
    if (!ctx || !ms_out) return fail(ETPIC_EINVAL, "null argument");
    if (int r = set_device(ctx)) return r;
    double tot[4] = {0.0, 0.0, 0.0, 0.0};
    int64_t cnt[2] = {0, 0};
    for (const auto &t : ctx->timing) {
        const int sorting = t.sorting ? 1 : 0;
        // intervals: coefficient pass, particle kernel, walk, edge gather
        float m[4] = {0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < 4; ++k)
            if (t.has & (1u << k)) {
                HIP_TRY(hipEventSynchronize(t.ev[2 * k + 1]));
                HIP_TRY(hipEventElapsedTime(&m[k], t.ev[2 * k], t.ev[2 * k + 1]));
            }
        // a launch of several steps books its time evenly over them
        const double per = m[1] / (double)t.steps;
        tot[3] += sorting * per;
        tot[0] += (t.steps - sorting) * per;
        tot[1] += m[0];
        tot[2] += m[2] + m[3];
        if (t.has & 2u) {
            cnt[1] += sorting;
            cnt[0] += t.steps - sorting;
        }
    }
    for (int k = 0; k < 4; ++k) ms_out[k] = tot[k];
    if (launches_out) {
        launches_out[0] = cnt[0];
        launches_out[1] = cnt[1];
    }
    if (reset) {
        for (auto &e : ctx->timing) ctx->spare.push_back(e);
        ctx->timing.clear();
    }
    return ETPIC_OK;
}

int etpic_last_push_slices(const etpic_ctx *ctx, int *slices) {
    if (!ctx || !slices) return fail(ETPIC_EINVAL, "null argument");
    *slices = ctx->last_slices;
    return ETPIC_OK;
}

int etpic_check(etpic_ctx *ctx, void *stream, uint32_t *device_flags) {
    if (!ctx) return fail(ETPIC_EINVAL, "null context");
    if (int r = set_device(ctx)) return r;
    hipStream_t st = static_cast<hipStream_t>(stream);
    unsigned word = 0;
    HIP_TRY(hipMemcpyAsync(&word, ctx->d_status, sizeof word, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    k_fill_u32<<<1, 64, 0, st>>>(ctx->d_status, 1, 0u);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipStreamSynchronize(st));
    if (device_flags) *device_flags = word;
    if (word & ETPIC_DEV_BADTET) return fail(ETPIC_EPARTICLE, "particle tet index out of range");
    if (word & ETPIC_DEV_HOPCAP) return fail(ETPIC_EWALK, "walk hop cap (%d) reached", ETPIC_HOP_CAP);
    if (word & ETPIC_DEV_NAN) return fail(ETPIC_ENAN, "non-finite velocity");
    return ETPIC_OK;
}

}  // extern "C"
