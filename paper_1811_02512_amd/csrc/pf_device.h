// libpf device-side building blocks shared by the kernel files (gfx950):
// views of the interleaved workspaces, 2x2 block helpers, level loops,
// the factor / solve node routines, the LDS tail and the mismatch pass.
// Included by every .hip file of the library; everything here has
// internal linkage (one copy per translation unit).
//
// Kernel map (paper sections in brackets):
//   k_ybus        FormMatrixA, four threads per (case, bus row)    [III-A]
//   k_mismatch    injections, mismatch, max-norm, one WG per case  [II-A]
//   k_jacobian    Jacobian blocks into the filled layout            [III]
//   k_factor      FactorizeGraphA, level by level, one WG per case  [III-B]
//   k_solve       forward / normalisation / backward substitution  [III-C]
//   k_newton      the whole Newton loop of one case per workgroup   [III]
//   k_adjoint, k_adj_*  adjoint gradients (beyond the paper)
//   k_fd_*, k_fdpf  fast decoupled matrices, LDL^T, iteration       [III, Table III]
//   k_branch_flows  post-convergence branch flows                   [II-A]
//   k_se_*        WLS state estimation: state, measurements, gain   [IV]
//
// Work decomposition inside a workgroup: hierarchical levels run one after
// the other with a workgroup barrier between them; inside a level, each
// node gets a group of g lanes (g from the symbolic's per-level mapping);
// the lanes of a group split the node's destinations and its descendant
// list, and combine partial sums with a butterfly over the group.  The top
// levels whose values fit (the "tail") run in LDS, right-looking by operation
// lists; substitutions take the top clique of the elimination tree column by
// column in one wavefront's registers.  Outside the tail the Newton and fast
// decoupled kernels reuse the same LDS for a copy of every bus's (e, f)
// (mismatch, Jacobian) and for the sweeps' solution vector.
//
// Memory layout across cases: a batch is cut into groups of C cases whose
// per-case arrays are interleaved in chunks (64 bytes for filled values: one
// slot record or two diagonal blocks; 32 bytes for bus records and the
// rhs), so one 128-byte line holds the same record of two or four cases.
// The C workgroups of a group are launched 8 blocks apart, which places them
// on the same XCD at the same time: they walk the same pattern in near
// lockstep and share every line they fetch through that XCD's L2.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "pf.h"
#include "pf_internal.h"
#include "pf_kernels.h"

// The library's internal headers work in namespace pf.
using namespace pf;

// ===========================================================================
// device helpers
// ===========================================================================
extern __shared__ __align__(16) double pf_smem[];  // dynamic LDS: tail, (e, f) copy, vectors, PV mask

namespace {

constexpr int kMaxThreads = 1024;
// The level-scheduled kernels are bounded at 512 threads per workgroup, which
// leaves them 256 VGPRs per lane: their per-node working set (two 2x2
// destination pairs, prefetched records, reduction partials) then fits in
// registers without spilling.
constexpr int kLevelThreads = 512;
constexpr int kXcds = 8;
constexpr int kWave = 64;  // CDNA wavefront
constexpr size_t kSolveLdsMax = 159 * 1024;  // of the 160 KB of LDS per workgroup on gfx950
// Value of the workgroup's zero-pivot marker while no pivot has failed; a
// failing pivot lowers it to its node's level-ordered index, so that the
// marker ends at the first failure in level order, then ascending position
// (the order of a sequential factorisation over the partition).
constexpr int kNoPivot = 0x7fffffff;

__device__ __forceinline__ void mark_pivot(int* s_bad, int x) { atomicMin(s_bad, x); }

// The workgroup's size in a scalar register: blockDim.x is a load from the
// dispatch's argument block, which the compiler repeats inside loops (and
// waits for, with everything else in flight) rather than keeping its result.
__device__ __forceinline__ int wg_size()
{
    return __builtin_amdgcn_readfirstlane((int)blockDim.x);
}

// Orders the LDS accesses of one wavefront's lanes (they run in lockstep,
// and a wavefront's LDS operations are performed in issue order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// threadIdx.x as a value the compiler takes for a new one at each call: what
// it derives from it (the addresses of a pass) is computed in that pass and
// not kept in registers through the whole iteration.
__device__ __forceinline__ int fresh_thread()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// The value of lane q of the wavefront, whose lanes all run here.
__device__ __forceinline__ double lane_value(double v, int q)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), q),
                            __builtin_amdgcn_readlane(__double2loint(v), q));
}

// One case's doubles inside an interleaved group of C cases: element d
// lives at base + (d / K) * K C + K (case % C) + d % K, i.e. chunks of K
// doubles of the C cases alternate.  The filled values use K = 8 (a slot
// record W, U is one 64-byte chunk, in a single cache line); the Newton
// bus records and rhs use K = 4 (the 32-byte voltage part of a bus record,
// which is what neighbours gather, shares its line with three other
// cases' only).  C = 1 is the plain contiguous layout.
struct View {
    double* base;
    int lane;  // K * (case % C)
    int sh;    // log2(K C)
    int cs;    // log2(K)
    __device__ __forceinline__ double* at(int64_t d) const
    {
        return base + ((d >> cs) << sh) + lane + (d & ((1 << cs) - 1));
    }
    __device__ __forceinline__ Blk blk(int64_t d) const { return bload(at(d)); }
    __device__ __forceinline__ void put(int64_t d, const Blk& v) const { bstore(at(d), v); }
    __device__ __forceinline__ double2 v2(int64_t d) const
    {
        return *reinterpret_cast<const double2*>(at(d));
    }
    __device__ __forceinline__ void put2(int64_t d, double2 v) const
    {
        *reinterpret_cast<double2*>(at(d)) = v;
    }
};

__device__ __forceinline__ int ilog2(int c) { return 31 - __clz(c); }

// Case of block b when groups of C cases are placed 8 blocks apart (same
// XCD under the round-robin workgroup dispatch); -1 for padding blocks.
__device__ __forceinline__ int case_of_block(int b, int C, int B)
{
    int c = b;
    if (C > 1) {
        const int span = kXcds * C;
        const int hi = b / span, rem = b - hi * span;
        c = (hi * kXcds + (rem & (kXcds - 1))) * C + rem / kXcds;
    }
    // the divisions run on the vector unit: back to a scalar, so that all the
    // case's base addresses are scalars too
    return __builtin_amdgcn_readfirstlane(c < B ? c : -1);
}

// Case (-1: none) and first item of this workgroup of a per-item kernel with
// per_case workgroups a case.  Workgroups go round-robin over the XCDs, so a
// case's own are taken 8 apart: its vectors, which the items gather from, are
// then fetched into one XCD's L2 instead of all eight's (10,000 buses x 512
// cases of branch flows 119 -> 81 us).  per_case 0, few cases: a case is
// spread over all of them.
__device__ __forceinline__ int2 item_block(int per_case, int B)
{
    if (per_case == 0) return make_int2(blockIdx.y, blockIdx.x * blockDim.x);
    const int i = blockIdx.x / kXcds, k = i / per_case;
    const int c = k * kXcds + (blockIdx.x & (kXcds - 1));
    return make_int2(__builtin_amdgcn_readfirstlane(c < B ? c : -1),
                     (i - k * per_case) * blockDim.x);
}

// Filled values of case c (64-byte chunks).
__device__ __forceinline__ View case_view(double* buf, int64_t stride, int C, int c)
{
    View v;
    v.base = buf + (int64_t)(c / C) * C * stride;
    v.lane = 8 * (c % C);
    v.sh = 3 + ilog2(C);
    v.cs = 3;
    return v;
}

// The Newton workspace's part after the filled values (bus records, rhs) of
// case c, offsets relative to its start (32-byte chunks).
__device__ __forceinline__ View case_bus_view(double* buf, int64_t stride, int C, int c,
                                              int64_t vals)
{
    View v;
    v.base = buf + (int64_t)(c / C) * C * stride + vals * C;
    v.lane = 4 * (c % C);
    v.sh = 2 + ilog2(C);
    v.cs = 2;
    return v;
}

// Offsets of the Newton workspace of one case (doubles):
//   D [nn][4] (padded) | LU [nnz_l][8] | bus records [n][8] | rhs [nn][2]
// D and LU through the values view; BUS and RHS relative to the bus view.
// bus record: e, f, |V|, theta | P, Q, -, -  (e + jf = V, P + jQ = S).
struct Off {
    int64_t D, LU, BUS, RHS;
};
__device__ __forceinline__ Off ws_off(const DevSym& S)
{
    Off o;
    o.D = 0;
    o.LU = S.lu_off;
    o.BUS = 0;
    o.RHS = 8 * (int64_t)S.n;
    return o;
}

// Voltage accessors: stored rectangular voltages, or computed from polar.
struct EFView {
    View v;
    int64_t bus_off;
    __device__ __forceinline__ void get(int k, double& ek, double& fk) const
    {
        const double2 t = v.v2(bus_off + 8 * (int64_t)k);
        ek = t.x;
        fk = t.y;
    }
};
// (e, f) of every bus copied into LDS (the Newton mismatch pass).
struct EFLds {
    double2* s;
    __device__ __forceinline__ void get(int k, double& ek, double& fk) const
    {
        const double2 t = s[k];
        ek = t.x;
        fk = t.y;
    }
};
struct EFPolar {
    const double* Vm;
    const double* Va;
    __device__ __forceinline__ void get(int k, double& ek, double& fk) const
    {
        double s, c;
        sincos(Va[k], &s, &c);
        ek = Vm[k] * c;
        fk = Vm[k] * s;
    }
};

// P_i + jQ_i = V_i conj(sum_k Y_ik V_k)  (nodal: one row of Y, entries
// [q0, q1), summed in order).  The first four entries' indices, admittances
// and voltages are requested together (in-bounds loads of entry q0 stand in
// for absent ones), the rest two at a time.
template <class EF>
__device__ __forceinline__ void injection_row(const DevSym& S, const double* __restrict__ yv,
                                              const EF& ef, int i, int q0, int q1, double& P,
                                              double& Q)
{
    const double2* y2 = reinterpret_cast<const double2*>(yv);
    double ei, fi;
    ef.get(i, ei, fi);
    int kq[4];
    double2 yq[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int q = q0 + k < q1 ? q0 + k : q0;
        kq[k] = S.ycol[q];
        yq[k] = y2[q];
    }
    double ek[4], fk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) ef.get(kq[k], ek[k], fk[k]);
    double ir = 0.0, ii = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        if (q0 + k < q1) {
            ir = fma(yq[k].x, ek[k], fma(-yq[k].y, fk[k], ir));
            ii = fma(yq[k].x, fk[k], fma(yq[k].y, ek[k], ii));
        }
    }
    int q = q0 + 4;
    for (; q + 1 < q1; q += 2) {
        const int k0 = S.ycol[q], k1 = S.ycol[q + 1];
        const double2 y0 = y2[q], y1 = y2[q + 1];
        double e0, f0, e1, f1;
        ef.get(k0, e0, f0);
        ef.get(k1, e1, f1);
        ir = fma(y0.x, e0, fma(-y0.y, f0, ir));
        ii = fma(y0.x, f0, fma(y0.y, e0, ii));
        ir = fma(y1.x, e1, fma(-y1.y, f1, ir));
        ii = fma(y1.x, f1, fma(y1.y, e1, ii));
    }
    if (q < q1) {
        const int k0 = S.ycol[q];
        const double2 y0 = y2[q];
        double e0, f0;
        ef.get(k0, e0, f0);
        ir = fma(y0.x, e0, fma(-y0.y, f0, ir));
        ii = fma(y0.x, f0, fma(y0.y, e0, ii));
    }
    P = ei * ir + fi * ii;
    Q = fi * ir - ei * ii;
}

template <class EF>
__device__ __forceinline__ void injection(const DevSym& S, const double* __restrict__ yv,
                                          const EF& ef, int i, double& P, double& Q)
{
    injection_row(S, yv, ef, i, S.yptr[i], S.yptr[i + 1], P, Q);
}

// PV flags of one case's buses, one bit per bus, in LDS after the tail.
struct PvMask {
    const uint32_t* m;
    __device__ __forceinline__ bool operator()(int k) const { return (m[k >> 5] >> (k & 31)) & 1u; }
};

__device__ __forceinline__ uint32_t* pv_words(const DevSym& S)
{
    const int off = S.tail_lds > S.ef_lds ? S.tail_lds : S.ef_lds;
    return reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(pf_smem) + off);
}

// Fills the mask m from the case's bus types (a ballot per wavefront); the
// caller synchronises before use.
__device__ __forceinline__ void pv_fill_at(uint32_t* m, const DevSym& S, const int8_t* type)
{
    for (int base = 0; base < S.n; base += blockDim.x) {
        const int i = base + threadIdx.x;
        const unsigned long long bits = __ballot(i < S.n && type[i] == T_PV);
        if ((threadIdx.x & 63) == 0 && i < S.n) {
            m[i >> 5] = (uint32_t)bits;
            m[(i >> 5) + 1] = (uint32_t)(bits >> 32);
        }
    }
}

__device__ __forceinline__ void pv_fill(const DevSym& S, const int8_t* type)
{
    pv_fill_at(pv_words(S), S, type);
}

// First four admittance entries of one row: indices and values, then the
// voltages they multiply (two dependent batches of loads, no stores).
struct RowHead {
    double2 y[4];
    double e[4], f[4];
};

template <class EF>
__device__ __forceinline__ void row_head_idx(const DevSym& S, const double* __restrict__ yv,
                                             int q0, int q1, int (&k)[4], RowHead& h)
{
    const double2* y2 = reinterpret_cast<const double2*>(yv);
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const int q = q0 + t < q1 ? q0 + t : q0;
        k[t] = S.ycol[q];
        h.y[t] = y2[q];
    }
}

template <class EF>
__device__ __forceinline__ void row_head_v(const EF& ef, const int (&k)[4], RowHead& h)
{
#pragma unroll
    for (int t = 0; t < 4; ++t) ef.get(k[t], h.e[t], h.f[t]);
}

// Sum of the row (head from registers, the rest loaded two at a time), in
// entry order, and the injection at bus voltage (ei, fi).
template <class EF>
__device__ __forceinline__ void row_finish(const DevSym& S, const double* __restrict__ yv,
                                           const EF& ef, int q0, int q1, const RowHead& h,
                                           double ei, double fi, double& P, double& Q)
{
    const double2* y2 = reinterpret_cast<const double2*>(yv);
    double ir = 0.0, ii = 0.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (q0 + t < q1) {
            ir = fma(h.y[t].x, h.e[t], fma(-h.y[t].y, h.f[t], ir));
            ii = fma(h.y[t].x, h.f[t], fma(h.y[t].y, h.e[t], ii));
        }
    }
    int q = q0 + 4;
    for (; q + 1 < q1; q += 2) {
        const int k0 = S.ycol[q], k1 = S.ycol[q + 1];
        const double2 y0 = y2[q], y1 = y2[q + 1];
        double e0, f0, e1, f1;
        ef.get(k0, e0, f0);
        ef.get(k1, e1, f1);
        ir = fma(y0.x, e0, fma(-y0.y, f0, ir));
        ii = fma(y0.x, f0, fma(y0.y, e0, ii));
        ir = fma(y1.x, e1, fma(-y1.y, f1, ir));
        ii = fma(y1.x, f1, fma(y1.y, e1, ii));
    }
    if (q < q1) {
        const int k0 = S.ycol[q];
        const double2 y0 = y2[q];
        double e0, f0;
        ef.get(k0, e0, f0);
        ir = fma(y0.x, e0, fma(-y0.y, f0, ir));
        ii = fma(y0.x, f0, fma(y0.y, e0, ii));
    }
    P = ei * ir + fi * ii;
    Q = fi * ir - ei * ii;
}

// Jacobian source: the Newton state of one case (bus records in the view).
// diag_in / off_in only issue loads, diag_of / off_of only compute, so that a
// caller can have all of a node's loads in flight before it waits for any.
// Invalid indices are never dereferenced: a fill slot (no admittance entry)
// reads entry 0 and is then zeroed.
struct SrcState {
    const double* yv;
    PvMask type;
    View w;
    int64_t bus_off;
    // (e, f) of every bus in LDS, or null: diag_in / off_in then read (e, f)
    // there and |V| is taken as sqrt(e^2 + f^2)
    const double2* efs;
    // the right-hand side of the Newton step sits in the bus record beside P, Q
    static constexpr bool kRhsInRecord = true;
    struct DiagIn {
        double2 y;
        Blk r;  // e, f, |V|, theta of the node's bus
        double2 s;  // P, Q
        double2 f;  // F_P, F_Q (the rhs)
        bool pv;
    };
    struct OffIn {
        Blk rk;
        double2 yl, yu;
        bool pk, fill;
    };
    __device__ __forceinline__ DiagIn diag_in(int, int bus, int yd) const
    {
        const double2* y2 = reinterpret_cast<const double2*>(yv);
        const int64_t rec = bus_off + 8 * (int64_t)bus;
        Blk r;
        if (efs) {
            const double2 t = efs[bus];
            r = {t.x, t.y, 0.0, 0.0};
        } else {
            r = w.blk(rec);
        }
        const Blk pqf = w.blk(rec + 4);  // P, Q, F_P, F_Q
        return {y2[yd], r, {pqf.a, pqf.b}, {pqf.c, pqf.d}, type(bus)};
    }
    __device__ __forceinline__ double2 rhs_at(int bus) const
    {
        return w.v2(bus_off + 8 * (int64_t)bus + 6);
    }
    __device__ __forceinline__ double vm_of(const Blk& r) const
    {
        return efs ? sqrt(fma(r.a, r.a, r.b * r.b)) : r.c;
    }
    __device__ __forceinline__ Blk diag_of(const DiagIn& d) const
    {
        return jac_diag(d.y.x, d.y.y, d.s.x, d.s.y, vm_of(d.r), d.pv);
    }
    __device__ __forceinline__ OffIn off_in(int, int bk, int ylo, int yup) const
    {
        const double2* y2 = reinterpret_cast<const double2*>(yv);
        const bool fill = ylo < 0;
        Blk rk;
        if (efs) {
            const double2 t = efs[bk];
            rk = {t.x, t.y, 0.0, 0.0};
        } else {
            rk = w.blk(bus_off + 8 * (int64_t)bk);
        }
        return {rk, y2[fill ? 0 : ylo], y2[fill ? 0 : yup], type(bk), fill};
    }
    __device__ __forceinline__ void off_of(const DiagIn& dj, const OffIn& o, Blk& lo,
                                           Blk& up) const
    {
        if (o.fill) {
            lo = bzero();
            up = bzero();
            return;
        }
        const double vk = vm_of(o.rk);
        lo = jac_off(o.yl.x, o.yl.y, o.rk.a, o.rk.b, dj.r.a, dj.r.b, vm_of(dj.r), o.pk, dj.pv);
        up = jac_off(o.yu.x, o.yu.y, dj.r.a, dj.r.b, o.rk.a, o.rk.b, vk, dj.pv, o.pk);
    }
    // the same straight from the bus records (the LDS copy may be gone)
    __device__ __forceinline__ Blk diag(int, int bus, int yd) const
    {
        const double2 y = reinterpret_cast<const double2*>(yv)[yd];
        const double vm = *w.at(bus_off + 8 * (int64_t)bus + 2);
        const double2 s = w.v2(bus_off + 8 * (int64_t)bus + 4);
        return jac_diag(y.x, y.y, s.x, s.y, vm, type(bus));
    }
    // block (k, j) below the diagonal and (j, k) above it; zero at fill
    __device__ __forceinline__ void off(int, int bj, int bk, int ylo, int yup, Blk& lo,
                                        Blk& up) const
    {
        if (ylo < 0) {
            lo = bzero();
            up = bzero();
            return;
        }
        const Blk rj = w.blk(bus_off + 8 * (int64_t)bj);  // e, f, |V|, theta
        const Blk rk = w.blk(bus_off + 8 * (int64_t)bk);
        const bool pj = type(bj), pk = type(bk);
        const double2 yl = reinterpret_cast<const double2*>(yv)[ylo];
        const double2 yu = reinterpret_cast<const double2*>(yv)[yup];
        lo = jac_off(yl.x, yl.y, rk.a, rk.b, rj.a, rj.b, rj.c, pk, pj);
        up = jac_off(yu.x, yu.y, rj.a, rj.b, rk.a, rk.b, rk.c, pj, pk);
    }
};

// Jacobian source: an assembled matrix in the filled layout.
// LOWER_ONLY (a symmetric matrix, factorised with the upper factor taken
// from the lower one): off_in reads the lower block alone.
template <bool LOWER_ONLY>
struct SrcLoadT {
    static constexpr bool kRhsInRecord = false;
    View w;
    int64_t lu_off;
    struct DiagIn {
        Blk a;
    };
    struct OffIn {
        Blk lo, up;
    };
    __device__ __forceinline__ DiagIn diag_in(int j, int, int) const
    {
        return {w.blk(4 * (int64_t)j)};
    }
    __device__ __forceinline__ Blk diag_of(const DiagIn& d) const { return d.a; }
    __device__ __forceinline__ OffIn off_in(int s, int, int, int) const
    {
        return {w.blk(lu_off + 8 * (int64_t)s),
                LOWER_ONLY ? bzero() : w.blk(lu_off + 8 * (int64_t)s + 4)};
    }
    __device__ __forceinline__ void off_of(const DiagIn&, const OffIn& o, Blk& lo,
                                           Blk& up) const
    {
        lo = o.lo;
        up = o.up;
    }
    __device__ __forceinline__ Blk diag(int j, int, int) const { return w.blk(4 * (int64_t)j); }
    __device__ __forceinline__ void off(int s, int, int, int, int, Blk& lo, Blk& up) const
    {
        lo = w.blk(lu_off + 8 * (int64_t)s);
        up = w.blk(lu_off + 8 * (int64_t)s + 4);
    }
};
using SrcLoad = SrcLoadT<false>;

// Level-ordered node record, the part the sweeps use ({j, bus, r0, r1},
// {s0, s1, ydiag, 0}); the admittance-row range is read by the mismatch only.
struct NodeRec {
    int4 a, b;
};

__device__ __forceinline__ NodeRec load_rec(const DevSym& S, int x)
{
    return {S.node_info[3 * x], S.node_info[3 * x + 1]};
}

// How one case's work is split over the workgroups of a launch.
// OneGroup: the whole case in one workgroup, levels separated by workgroup
// barriers.
struct OneGroup {
    static constexpr bool kSpread = false;
    static constexpr bool kSub = false;
    __device__ __forceinline__ int rank() const { return 0; }
    __device__ __forceinline__ int size() const { return 1; }
    __device__ __forceinline__ void sync() const { __syncthreads(); }
};

// Spread: the case's wide phases (loops over buses, the levels below the LDS
// tail) over the workgroups of a cooperative launch that own the case (all
// of them, or a group in a batch of grids), which meet at grid barriers;
// the tail stays on the group's first workgroup while the others wait.  The
// barrier words live in three 128-byte lines of the case's workspace,
// zeroed (the pivot marker set to kNoPivot) before the launch:
//   line 0: arrivals (count of workgroups that reached a barrier, over all
//           barriers so far); line 1: release (number of the last barrier
//           every workgroup has reached); line 2: abort flag, zero-pivot
//           marker, then per parity of the iteration count a NaN flag and
//           the bits of the mismatch maximum (a non-negative double, whose
//           bit patterns order as unsigned integers do).
// A workgroup makes its writes visible before it arrives (an agent-scope
// release fence: its XCD's L2 written back) and discards stale cached lines
// after it is released (an agent-scope acquire fence), so what any workgroup
// wrote before a barrier is what every workgroup reads after it: each
// arrival is counted only after its writes have reached memory, the release
// word is stored only after every arrival has been counted, and a workgroup
// reads only after it has seen the release word and invalidated its caches.
// A wait that lasts longer than wait_ticks of the constant 100 MHz clock
// (one second unless a caller lowers it) sets the abort flag; from then on
// no barrier waits, so every workgroup runs to its end and the case reports
// the failure.
constexpr int kSpreadWords = 96;  // 32-bit words of the three lines

struct Spread {
    static constexpr bool kSpread = true;
    static constexpr bool kSub = false;  // every level below the tail shared
    unsigned* arrive;
    unsigned* release;
    int* flags;        // abort, pivot marker, NaN flag [2]
    uint64_t* maxbits; // [2]
    unsigned* count;   // LDS: barriers this workgroup has passed
    // levels [back_lo, tail level) of the backward substitution run on
    // workgroup 0 right after the tail's (narrow levels: workgroup barriers
    // are cheaper there than grid barriers)
    int back_lo;
    unsigned long long wait_ticks;
    int rk, sz;  // this workgroup's rank in the case's group, the group's size
    __device__ __forceinline__ int rank() const { return rk; }
    __device__ __forceinline__ int size() const { return sz; }
    __device__ __forceinline__ int* marker() const { return flags + 1; }
    __device__ __forceinline__ bool aborted() const
    {
        return __hip_atomic_load(flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
    }
    __device__ __forceinline__ void sync() const
    {
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned k = ++*count;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            const unsigned before =
                __hip_atomic_fetch_add(arrive, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!aborted()) {
                if (before == k * (unsigned)sz - 1) {
                    __hip_atomic_store(release, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                } else {
                    const unsigned long long t0 = wall_clock64();
                    while (__hip_atomic_load(release, __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT) < k) {
                        if (aborted()) break;
                        if (wall_clock64() - t0 > wait_ticks) {
                            __hip_atomic_store(flags, 1, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                            break;
                        }
                        __builtin_amdgcn_s_sleep(1);
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
    }
};

// As Spread, with the levels below the subtree cut (DevSym::sub_cut) run by
// each workgroup on whole subtrees of its own, workgroup barriers between
// them: used by the groups of a batch of grids, where grid barriers contend
// with the other groups for the XCDs they share.  (One case alone keeps
// Spread: there the subtree levels measured slower than shared ones.)
struct SpreadSub : Spread {
    static constexpr bool kSub = true;
};

// Runs fn(x, rec, lane, g) for the nodes of levels [l0, l1), up or down,
// with a barrier of the split after every level: x indexes the level-ordered
// node records, rec is x's record, and each node gets g lanes (the level's
// mapping); the groups of g lanes of all the split's workgroups take the
// level's nodes in turn, group k of every workgroup before group k + 1 of
// any, so that a narrow level still reaches every workgroup.  The record of
// the group's next node in the level is fetched before fn runs so that its
// latency overlaps the current node's work.
template <class P, class F>
__device__ __forceinline__ void for_nodes(const P& par, const DevSym& S, int l0, int l1, bool up,
                                          F&& fn)
{
    const int T = wg_size();
    for (int li = l0; li < l1; ++li) {
        const int l = up ? li : l1 - 1 - (li - l0);
        const int g = S.level_g[l];  // a power of two
        const int lg = ilog2(g);
        const int beg = S.level_ptr[l];
        const int cnt = S.level_ptr[l + 1] - beg;
        const int step = (T >> lg) * par.size();
        const int lane = threadIdx.x & (g - 1);
        int idx = (int)(threadIdx.x >> lg) * par.size() + par.rank();
        NodeRec cur = idx < cnt ? load_rec(S, beg + idx) : NodeRec{};
        while (idx < cnt) {
            const int nxt = idx + step;
            const NodeRec pre = nxt < cnt ? load_rec(S, beg + nxt) : NodeRec{};
            fn(beg + idx, cur, lane, g);
            cur = pre;
            idx = nxt;
        }
        par.sync();
    }
}

template <class F>
__device__ __forceinline__ void for_nodes(const DevSym& S, int l0, int l1, bool up, F&& fn)
{
    for_nodes(OneGroup{}, S, l0, l1, up, static_cast<F&&>(fn));
}

// As for_nodes over levels [l0, l1) below the subtree cut, for the nodes of
// this workgroup's subtrees only (roots [k0, k1)), with a workgroup barrier
// after every level: a node's descendants belong to its own subtree, so no
// other workgroup's results are needed until the cut.
template <class F>
__device__ __forceinline__ void for_sub_levels(const DevSym& S, int k0, int k1, int l0, int l1,
                                               bool up, F&& fn)
{
    const int R1 = S.sub_roots + 1;
    const int T = wg_size();
    for (int li = l0; li < l1; ++li) {
        const int l = up ? li : l1 - 1 - (li - l0);
        const int g = S.level_g[l];
        const int b = S.level_ptr[l];
        const int e1 = b + S.sub_ptr[l * R1 + k1];
        const int lg = ilog2(g);
        const int gpb = T >> lg;
        const int lane = threadIdx.x & (g - 1);
        int e = b + S.sub_ptr[l * R1 + k0] + (int)(threadIdx.x >> lg);
        int x = e < e1 ? S.sub_idx[e] : 0;
        NodeRec cur = e < e1 ? load_rec(S, x) : NodeRec{};
        while (e < e1) {
            const int en = e + gpb;
            const int xn = en < e1 ? S.sub_idx[en] : 0;
            const NodeRec pre = en < e1 ? load_rec(S, xn) : NodeRec{};
            fn(x, cur, lane, g);
            cur = pre;
            x = xn;
            e = en;
        }
        __syncthreads();
    }
}

// The subtrees [k0, k1) of workgroup `rank` of `size`: the roots whose work
// starts in its share [rank, rank + 1) / size of the total (every workgroup
// of the group calls this; k0 = k1 = 0 without subtrees).
template <class P>
__device__ __forceinline__ void sub_share(const DevSym& S, const P& par, int& k0, int& k1)
{
    __shared__ int s_k[2];
    k0 = k1 = 0;
    if (S.sub_cut <= 0) return;
    if (threadIdx.x < 2) s_k[threadIdx.x] = 0;
    __syncthreads();
    const int R = S.sub_roots;
    const int64_t tot = S.sub_cum[R];
    const int64_t a = tot * par.rank() / par.size();
    const int64_t b = tot * (par.rank() + 1) / par.size();
    int c0 = 0, c1 = 0;
    for (int k = threadIdx.x; k < R; k += blockDim.x) {
        const int64_t v = S.sub_cum[k];
        c0 += v < a;
        c1 += v < b;
    }
    if (c0) atomicAdd(&s_k[0], c0);
    if (c1) atomicAdd(&s_k[1], c1);
    __syncthreads();
    k0 = s_k[0];
    k1 = s_k[1];
    __syncthreads();
}

// Block updates of one destination slot from pairs (a, b) = (slot(i;k), slot(i;j)):
//   W_kj -= W_ki U_ij,  V_jk -= W_ji U_ik.
// Two pairs per step; the next step's indices are fetched before this
// step's blocks so that index and value loads overlap.  Pairs past the end
// of a list are not loaded (a load no lane of the wavefront needs is
// skipped) and contribute nothing.
__device__ __forceinline__ int2 upd_at(const int2* __restrict__ upd, int u, int u1)
{
    int2 p = make_int2(0, 0);
    if (u < u1) p = upd[u];
    return p;
}

// The four blocks pair p reads: W_a = W(p.x), U_a = U(p.x), W_b, U_b of p.y.
struct PairBlk {
    Blk Wa, Ua, Wb, Ub;
};
__device__ __forceinline__ PairBlk pair_blocks(const View& w, int64_t lu, int2 p, bool has)
{
    PairBlk b{bzero(), bzero(), bzero(), bzero()};
    if (has) {
        b.Wa = w.blk(lu + 8 * (int64_t)p.x);
        b.Ua = w.blk(lu + 8 * (int64_t)p.x + 4);
        b.Wb = w.blk(lu + 8 * (int64_t)p.y);
        b.Ub = w.blk(lu + 8 * (int64_t)p.y + 4);
    }
    return b;
}

__device__ __forceinline__ void apply_updates(const int2* __restrict__ upd, int u0, int u1,
                                              const View& w, int64_t lu, Blk& Wk, Blk& Vk)
{
    if (u0 >= u1) return;
    int2 p = upd[u0];
    int2 q = upd_at(upd, u0 + 1, u1);
    for (int u = u0; u < u1; u += 2) {
        const bool has_q = u + 1 < u1;
        const int2 pn = upd_at(upd, u + 2, u1);
        const int2 qn = upd_at(upd, u + 3, u1);
        const PairBlk a = pair_blocks(w, lu, p, true);
        const PairBlk c = pair_blocks(w, lu, q, has_q);
        bmsub(Wk, a.Wa, a.Ub);
        bmsub(Vk, a.Wb, a.Ua);
        if (has_q) {
            bmsub(Wk, c.Wa, c.Ub);
            bmsub(Vk, c.Wb, c.Ua);
        }
        p = pn;
        q = qn;
    }
}

// The updates of two destinations at once, one pair of each per step, with
// the first pairs (p, q) already loaded: both chains of loads are in flight
// together.  The order of the updates of each destination is the list order.
// SYM (symmetric matrix): only W is updated (V_jk = W_kj^T throughout), so
// each pair reads two blocks instead of four.
template <bool SYM = false>
__device__ __forceinline__ void apply_updates2(const int2* __restrict__ upd, int u0, int u1,
                                               int v0, int v1, int2 p, int2 q, const View& w,
                                               int64_t lu, Blk& Wk, Blk& Vk, Blk& Wk2, Blk& Vk2)
{
    for (int a = u0, b = v0; a < u1 || b < v1; ++a, ++b) {
        const bool hp = a < u1, hq = b < v1;
        const int2 pn = upd_at(upd, a + 1, u1);
        const int2 qn = upd_at(upd, b + 1, v1);
        if (SYM) {
            Blk Wa = bzero(), Ub = bzero(), Wc = bzero(), Ud = bzero();
            if (hp) {
                Wa = w.blk(lu + 8 * (int64_t)p.x);
                Ub = w.blk(lu + 8 * (int64_t)p.y + 4);
            }
            if (hq) {
                Wc = w.blk(lu + 8 * (int64_t)q.x);
                Ud = w.blk(lu + 8 * (int64_t)q.y + 4);
            }
            if (hp) bmsub(Wk, Wa, Ub);
            if (hq) bmsub(Wk2, Wc, Ud);
        } else {
            const PairBlk x = pair_blocks(w, lu, p, hp);
            const PairBlk y = pair_blocks(w, lu, q, hq);
            if (hp) {
                bmsub(Wk, x.Wa, x.Ub);
                bmsub(Vk, x.Wb, x.Ua);
            }
            if (hq) {
                bmsub(Wk2, y.Wa, y.Ub);
                bmsub(Vk2, y.Wb, y.Ua);
            }
        }
        p = pn;
        q = qn;
    }
}

// An operation of the tail (t_op, see DevSym).
struct TailOp {
    int d, a, b, j, next;
};
__device__ __forceinline__ TailOp tail_op(const uint2& q)
{
    return {(int)(q.x & 0xfff), (int)(q.x >> 12 & 0xfff), (int)(q.x >> 24 | (q.y & 0xf) << 8),
            (int)(q.y >> 4 & 0xfff), (int)(q.y >> 16)};
}

// The tail's level loops: each lane of a wavefront holds the table entry of
// one of 64 levels (read back by lane index, where all lanes are active), and
// a thread's operations of the next two levels are requested together while
// the current ones run (a level takes less time than a load that misses L1),
// an absent one's place taken by the level's first.  Two, four and eight
// levels: 2,000 buses x 384 outages 1,446, 1,478 and 1,505 us, 2,000 x 1,024
// 1,729, 1,742 and 1,737, one 10,000-bus case 1,224, 1,224 and 1,236; each level
// is a copy of the loop's code.  The form for tails with long destinations
// looks one ahead: with four the Newton kernel had 192 instead of 138 KB of
// code, and the ordinary form ran 1 to 2% slower beside it.
constexpr int tail_ahead(bool longs) { return longs ? 1 : 2; }

// Walks a tail destination's operations: its first, its second (at `at`) and
// further ones up to kTailSerial.
template <class F>
__device__ __forceinline__ void tail_terms(const DevSym& S, const uint2& first,
                                           const uint2& second, int at, F&& term)
{
    TailOp e = tail_op(first);
    term(e);
    if (!e.next) return;
    e = tail_op(second);
    term(e);
    if (!e.next) return;
    at += e.next;
    for (int k = 2; k < kTailSerial; ++k, ++at) {
        e = tail_op(S.t_op[at]);
        term(e);
        if (!e.next) return;
    }
}

// The operations of a long destination after those, `lanes` of them at a time:
// runs term(op) for this lane's (lane < lanes); second at `at`.
template <class F>
__device__ __forceinline__ void tail_rest(const DevSym& S, int at, int lane, int lanes, F&& term)
{
    const int third = at + tail_op(S.t_op[at]).next;
    const int end = third + tail_op(S.t_op[third]).next + 1;
    for (int p = third + kTailSerial - 2 + lane; p < end; p += lanes) term(tail_op(S.t_op[p]));
}

// Runs fn(op) for the backward operations of the tail levels [0, nt),
// downward, one thread each, or with FWD, fn(op, second, index of second) for
// the updates of diagonals, upward, one thread per destination (second: its
// second term on the level, if op.next says that there is one), then, by
// wavefronts, with LONG, rest(d, index of second) for what long destinations d
// have left; a workgroup barrier after every level.
template <bool FWD, bool LONG, class F, class R>
__device__ __forceinline__ void for_tail_ops(const DevSym& S, int nt, F&& fn, R&& rest)
{
    constexpr int ahead = tail_ahead(LONG);
    const int T = wg_size();
    struct Head {
        int op0, n, two, n2;  // first operation, count; the same of second ones
    };
    for (int i0 = 0; i0 < nt; i0 += kWave) {
        const int m = nt - i0 < kWave ? nt - i0 : kWave;
        Head mine{0, 0, 0, 0};
        int longs = 0;
        {
            const int l = threadIdx.x & (kWave - 1);
            const int i = i0 + (l < m ? l : m - 1);
            const int4 h = S.t_lev[FWD ? 2 * i : 2 * (nt - 1 - i) + 1];
            if (FWD) mine = {h.x + h.y, h.z - h.y, h.x + h.z + (h.w & 0xffff), h.w >> 16};
            else mine = {h.x, h.y, 0, 0};
            if (LONG) longs = S.t_lev[2 * i + 1].z >> 16;
        }
        auto head = [&](int l) {
            const int k = l < m ? l : m - 1;
            return Head{__builtin_amdgcn_readlane(mine.op0, k),
                        __builtin_amdgcn_readlane(mine.n, k),
                        FWD ? __builtin_amdgcn_readlane(mine.two, k) : 0,
                        FWD ? __builtin_amdgcn_readlane(mine.n2, k) : 0};
        };
        auto first = [&](const Head& h, int t) { return S.t_op[h.op0 + (t < h.n ? t : 0)]; };
        auto second = [&](const Head& h, int t) { return S.t_op[t < h.n2 ? h.two + t : h.op0]; };
        auto go = [&](const Head& h, int t, const uint2& q, const uint2& r) {
            if constexpr (FWD) fn(q, r, h.two + t);
            else fn(q);
        };
        uint2 q[ahead], r[ahead];
#pragma unroll
        for (int k = 0; k < ahead; ++k) {
            const Head h = head(k);
            q[k] = first(h, threadIdx.x);
            if (FWD) r[k] = second(h, threadIdx.x);
        }
        for (int i = 0; i < m; i += ahead) {
            uint2 qn[ahead], rn[ahead];
#pragma unroll
            for (int k = 0; k < ahead; ++k) {
                const Head h = head(i + k + ahead);
                qn[k] = first(h, threadIdx.x);
                if (FWD) rn[k] = second(h, threadIdx.x);
            }
#pragma unroll
            for (int k = 0; k < ahead; ++k) {
                if (i + k >= m) break;
                const Head h = head(i + k);
                if ((int)threadIdx.x < h.n) go(h, threadIdx.x, q[k], r[k]);
                for (int t = threadIdx.x + T; t < h.n; t += T)
                    go(h, t, first(h, t), FWD ? second(h, t) : make_uint2(0, 0));
                __syncthreads();
                if constexpr (LONG) {
                    const int nl = __builtin_amdgcn_readlane(longs, i + k);
                    for (int t = (int)threadIdx.x / kWave; t < nl; t += T / kWave)
                        rest(tail_op(first(h, t)).d, h.two + t);
                    if (nl > 0) __syncthreads();
                }
            }
#pragma unroll
            for (int k = 0; k < ahead; ++k) {
                q[k] = qn[k];
                if (FWD) r[k] = rn[k];
            }
        }
    }
}

// Runs the right-looking updates of the tail levels [0, nt), upward, with a
// workgroup barrier after every level: quad(op, second, index of second, slot)
// with four lanes per destination on levels that a quarter of the workgroup's
// threads cover, else lane(same) with one thread per destination; then, by
// wavefronts, with LONG, rest(d, index of second, slot) for what long
// destinations d have left.
template <bool LONG, class Q, class F, class R>
__device__ __forceinline__ void for_tail_updates(const DevSym& S, int nt, Q&& quad, F&& lane,
                                                 R&& rest)
{
    constexpr int ahead = tail_ahead(LONG);
    const int T = wg_size(), nq = T >> 2;
    const int lq = (int)threadIdx.x >> 2;
    struct Head {
        int op0, ns, n, ns2, nd2;
        __device__ __forceinline__ int one(int i) const { return op0 + (i < n ? i : 0); }
        // position of destination index i's second operation
        __device__ __forceinline__ int two(int i) const
        {
            const bool slot = i < ns;
            const int k = slot ? i : i - ns;
            return k < (slot ? ns2 : nd2) ? op0 + n + (slot ? 0 : ns2) + k : op0;
        }
    };
    for (int i0 = 0; i0 < nt; i0 += kWave) {
        const int m = nt - i0 < kWave ? nt - i0 : kWave;
        int4 mine;
        int longs = 0;
        {
            const int l = threadIdx.x & (kWave - 1);
            const int i = i0 + (l < m ? l : m - 1);
            mine = S.t_lev[2 * i];
            if (LONG) longs = S.t_lev[2 * i + 1].z;
        }
        auto head = [&](int l) {
            const int k = l < m ? l : m - 1;
            const int c2 = __builtin_amdgcn_readlane(mine.w, k);
            return Head{__builtin_amdgcn_readlane(mine.x, k), __builtin_amdgcn_readlane(mine.y, k),
                        __builtin_amdgcn_readlane(mine.z, k), c2 & 0xffff, c2 >> 16};
        };
        // this thread's destination on a level
        auto mine_of = [&](const Head& h) { return h.n <= nq ? lq : (int)threadIdx.x; };
        uint2 q[ahead], r[ahead];
#pragma unroll
        for (int k = 0; k < ahead; ++k) {
            const Head h = head(k);
            q[k] = S.t_op[h.one(mine_of(h))];
            r[k] = S.t_op[h.two(mine_of(h))];
        }
        for (int i = 0; i < m; i += ahead) {
            uint2 qn[ahead], rn[ahead];
#pragma unroll
            for (int k = 0; k < ahead; ++k) {
                const Head h = head(i + k + ahead);
                qn[k] = S.t_op[h.one(mine_of(h))];
                rn[k] = S.t_op[h.two(mine_of(h))];
            }
#pragma unroll
            for (int k = 0; k < ahead; ++k) {
                if (i + k >= m) break;
                const Head h = head(i + k);
                const int t = mine_of(h);
                if (h.n <= nq) {
                    if (t < h.n) quad(q[k], r[k], [&]() { return h.two(t); }, t < h.ns);
                } else {
                    if (t < h.n) lane(q[k], r[k], [&]() { return h.two(t); }, t < h.ns);
                    for (int u = t + T; u < h.n; u += T)
                        lane(S.t_op[h.one(u)], S.t_op[h.two(u)], [&]() { return h.two(u); },
                             u < h.ns);
                }
                __syncthreads();
                if constexpr (LONG) {
                    const int nl = __builtin_amdgcn_readlane(longs, i + k);
                    const int ls = nl & 0xffff, all = ls + (nl >> 16);
                    for (int u = (int)threadIdx.x / kWave; u < all; u += T / kWave) {
                        const int x = u < ls ? u : h.ns + u - ls;
                        rest(tail_op(S.t_op[h.one(x)]).d, h.two(x), u < ls);
                    }
                    if (all > 0) __syncthreads();
                }
            }
#pragma unroll
            for (int k = 0; k < ahead; ++k) {
                q[k] = qn[k];
                r[k] = rn[k];
            }
        }
    }
}

// The tail's values in LDS: the four 16-byte rows of the slot records (W,
// then V or U) as separate arrays of TS, so that lanes on consecutive slots
// read consecutive 16-byte words (records of 64 bytes would put four lanes
// on each bank), then the nodes' pivot blocks and the rhs.
struct TailLds {
    double2* r;  // TS x 4 rows
    double* d;   // K x 4
    double* y;   // K x 2
    double* q;   // K: one over the pivot block's determinant
    int TS;
    __device__ __forceinline__ explicit TailLds(const DevSym& S)
        : r(reinterpret_cast<double2*>(pf_smem)),
          d(pf_smem + 8 * S.tail_slots),
          y(d + 4 * S.tail_nodes),
          q(y + 2 * S.tail_nodes),
          TS(S.tail_slots)
    {
    }
    // pivot block of node j and its inverse
    __device__ __forceinline__ void setD(int j, const Blk& v) const
    {
        bstore(d + 4 * j, v);
        q[j] = 1.0 / bdet(v);
    }
    // the row x of a block times D_j^-1
    __device__ __forceinline__ double2 over(const double2& x, int j) const
    {
        const Blk v = bload(d + 4 * j);
        const double i = q[j];
        return make_double2(fma(x.x, v.d, -(x.y * v.c)) * i, fma(x.y, v.a, -(x.x * v.b)) * i);
    }
    __device__ __forceinline__ Blk Dinv(int j) const
    {
        const Blk v = bload(d + 4 * j);
        const double i = q[j];
        return {v.d * i, -v.b * i, -v.c * i, v.a * i};
    }
    __device__ __forceinline__ Blk get(int row, int t) const
    {
        const double2 u = r[row * TS + t], v = r[(row + 1) * TS + t];
        return {u.x, u.y, v.x, v.y};
    }
    // W_t D_j^-1
    __device__ __forceinline__ Blk W_over(int t, int j) const
    {
        const double2 u = over(r[t], j), v = over(r[TS + t], j);
        return {u.x, u.y, v.x, v.y};
    }
    __device__ __forceinline__ void put(int row, int t, const Blk& v) const
    {
        r[row * TS + t] = make_double2(v.a, v.b);
        r[(row + 1) * TS + t] = make_double2(v.c, v.d);
    }
    __device__ __forceinline__ Blk W(int t) const { return get(0, t); }
    __device__ __forceinline__ Blk U(int t) const { return get(2, t); }
    __device__ __forceinline__ void setW(int t, const Blk& v) const { put(0, t, v); }
    __device__ __forceinline__ void setU(int t, const Blk& v) const { put(2, t, v); }
    __device__ __forceinline__ double2 yv(int j) const
    {
        return *reinterpret_cast<const double2*>(y + 2 * j);
    }
    __device__ __forceinline__ void sety(int j, double a, double b) const
    {
        *reinterpret_cast<double2*>(y + 2 * j) = make_double2(a, b);
    }
};

// Group sums of a block and, with rhs, of a 2-vector, all six interleaved.
__device__ __forceinline__ void gsum_blk(Blk& v, double& z0, double& z1, bool rhs, int g)
{
    if (rhs) {
        double t[6] = {v.a, v.b, v.c, v.d, z0, z1};
        gsum_n(t, g);
        v = {t[0], t[1], t[2], t[3]};
        z0 = t[4];
        z1 = t[5];
    } else {
        double t[4] = {v.a, v.b, v.c, v.d};
        gsum_n(t, g);
        v = {t[0], t[1], t[2], t[3]};
    }
}

// Left-looking block LDU of node record x (FactorizeGraphA, pull form):
//   D_j  = A_jj - sum_{i in R(j)} W_ji U_ij
//   W_kj = A_kj - sum_i W_ki U_ij,  V_jk = A_jk - sum_i W_ji U_ik  (k in S(j))
//   stored: LU[s] <- (W_kj, U_jk = D_j^-1 V_jk), and with STORE_D the D
//   section <- D_j^-1 (needed only by later solves with these factors).
// With FWD, also the forward substitution and normalisation of the rhs:
//   y_j = D_j^-1 (b_j - sum_{i in R(j)} W_ji y_i).
// Loads are issued in batches so that the chain of dependent requests per
// node stays short: the record's dependants first (diagonal inputs, rhs,
// the first two destinations' slot records, the first R indices), then R(j)
// four entries per lane at a time, then two destinations per step with both
// update chains in flight together.  Absent list entries, slots and update
// pairs are not loaded (a load no lane of the wavefront needs is skipped)
// and add nothing.
// SYM: a symmetric matrix (eq. 2 blockwise): only the lower blocks take
// updates and U_jk = D_j^-1 W_kj^T.
// x: the node's level-ordered index (for the zero-pivot marker s_bad).
template <class SRC, bool FWD, bool STORE_D, bool SYM = false>
__device__ __forceinline__ void factor_node(const DevSym& S, const SRC& src, int x,
                                            const NodeRec& rec, int lane, int g, const View& w,
                                            int64_t lu, const View& wr, int64_t rhs, int* s_bad)
{
    const int4 n0 = rec.a;
    const int4 n1 = rec.b;
    const int j = n0.x, bus = n0.y;
    const int r1 = n0.w, s1 = n1.y;
    const typename SRC::DiagIn din = src.diag_in(j, bus, n1.z);
    double2 bj = make_double2(0.0, 0.0);
    if constexpr (FWD) {
        if constexpr (SRC::kRhsInRecord) bj = din.f;
        else bj = wr.v2(rhs + 2 * (int64_t)j);
    }
    // Absent list entries are not loaded at all (each guarded load is skipped
    // when no lane of the wavefront needs it: the sweeps are bound by the
    // number of vector-memory instructions, not by bytes).
    int s = n1.x + lane;
    const int4 z4 = make_int4(0, 0, 0, 0);
    int4 sa = z4, sb = z4, sa2 = z4, sb2 = z4;
    if (s < s1) {
        sa = S.slot_info[2 * s];
        sb = S.slot_info[2 * s + 1];
    }
    if (s + g < s1) {
        sa2 = S.slot_info[2 * (s + g)];
        sb2 = S.slot_info[2 * (s + g) + 1];
    }
    int2 e[4];
    int r = n0.z + lane;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        e[k] = make_int2(0, 0);
        if (r + k * g < r1) e[k] = S.rl[r + k * g];
    }
    Blk ds = bzero();
    double z0 = 0.0, z1 = 0.0;
    for (; r < r1; r += 4 * g) {
        Blk wv[4], uv[4];
        double2 yi[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            wv[k] = bzero();
            uv[k] = bzero();
            yi[k] = make_double2(0.0, 0.0);
            if (r + k * g < r1) {
                wv[k] = w.blk(lu + 8 * (int64_t)e[k].y);
                uv[k] = w.blk(lu + 8 * (int64_t)e[k].y + 4);
                if (FWD) yi[k] = wr.v2(rhs + 2 * (int64_t)e[k].x);
            }
        }
        const int rn = r + 4 * g;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (rn + k * g < r1) e[k] = S.rl[rn + k * g];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (r + k * g < r1) {
                bmadd(ds, wv[k], uv[k]);
                if (FWD) mvadd(z0, z1, wv[k], yi[k].x, yi[k].y);
            }
        }
    }
    if (g > 1) {
        gsum_blk(ds, z0, z1, FWD, g);
    }
    const Blk Ajj = src.diag_of(din);
    bool ok;
    const Blk Di = binv({Ajj.a - ds.a, Ajj.b - ds.b, Ajj.c - ds.c, Ajj.d - ds.d}, ok);
    for (; s < s1; s += 2 * g) {
        const int s2 = s + g;
        const bool two = s2 < s1;
        const typename SRC::OffIn o1 = src.off_in(s, sa.y, sa.z, sa.w);
        typename SRC::OffIn o2{};
        if (two) o2 = src.off_in(s2, sa2.y, sa2.z, sa2.w);
        const int u0 = sb.x, u1 = sb.y, v0 = two ? sb2.x : 0, v1 = two ? sb2.y : 0;
        int2 p = make_int2(0, 0), q = make_int2(0, 0);
        if (u0 < u1) p = S.upd[u0];
        if (v0 < v1) q = S.upd[v0];
        const int sn = s + 2 * g;
        if (sn < s1) {
            sa = S.slot_info[2 * sn];
            sb = S.slot_info[2 * sn + 1];
        }
        if (sn + g < s1) {
            sa2 = S.slot_info[2 * (sn + g)];
            sb2 = S.slot_info[2 * (sn + g) + 1];
        }
        Blk Wk, Vk, Wk2, Vk2;
        src.off_of(din, o1, Wk, Vk);
        src.off_of(din, o2, Wk2, Vk2);
        apply_updates2<SYM>(S.upd, u0, u1, v0, v1, p, q, w, lu, Wk, Vk, Wk2, Vk2);
        w.put(lu + 8 * (int64_t)s, Wk);
        w.put(lu + 8 * (int64_t)s + 4, bmul(Di, SYM ? btrans(Wk) : Vk));
        if (two) {
            w.put(lu + 8 * (int64_t)s2, Wk2);
            w.put(lu + 8 * (int64_t)s2 + 4, bmul(Di, SYM ? btrans(Wk2) : Vk2));
        }
    }
    if (lane == 0) {
        if (!ok) mark_pivot(s_bad, x);
        if (STORE_D) w.put(4 * (int64_t)j, Di);
        if (FWD) {
            double y0 = 0.0, y1 = 0.0;
            mvadd(y0, y1, Di, bj.x - z0, bj.y - z1);
            wr.put2(rhs + 2 * (int64_t)j, make_double2(y0, y1));
        }
    }
}

// Local slot of clique pair (a, b), a < b: the clique's slots are numbered
// node by node, node a owning KC - a - 1 of them.
__device__ __forceinline__ int clique_slot(int c0, int KC, int a, int b)
{
    return c0 + a * (KC - 1) - (a * (a - 1)) / 2 + (b - a - 1);
}

// Right-looking factorisation of the upper levels below the tail in global
// memory, on values that have taken every update from below (W, V per slot, D
// and, with FWD, z): one thread per destination of a level's operation list
// (g_op), over the threads of every workgroup of the split, one barrier of the
// split per level.  Leaves the pivots and V as they are (not inverted, not
// normalised).  A thread's first two terms come from known places of the
// list: their indices are requested before the barrier that starts the level,
// then all their values together.
template <bool FWD, class P>
__device__ __forceinline__ void factor_ops(const P& par, const DevSym& S, const View& w,
                                           int64_t lu, const View& wr, int64_t rhs)
{
    const int T = wg_size();
    const int me = par.rank() * T + (int)threadIdx.x, all = par.size() * T;
    const int nl = S.tail_level - S.mid_level;
    struct Head {
        int op0, ns, nd, ns2, nd2;
        // position of destination index t's second operation
        __device__ __forceinline__ int two(int t) const
        {
            const bool slot = t < ns;
            const int k = slot ? t : t - ns;
            return k < (slot ? ns2 : nd2) ? op0 + nd + (slot ? 0 : ns2) + k : op0;
        }
    };
    struct Ops {
        int4 o, p;
        int no, np;  // offsets of the term after each, 0 = none
    };
    struct Val {
        Blk Wa, Va, Wb, Vb, D;
        double2 z;
    };
    auto fetch = [&](const Head& h, int t) {
        const int a = h.op0 + (t < h.nd ? t : 0), b = h.two(t);
        return Ops{S.g_op[a], S.g_op[b], S.g_next[a], S.g_next[b]};
    };
    auto load = [&](const int4& o, bool slot) {
        Val v;
        const int64_t ra = lu + 8 * (int64_t)o.y, rb = lu + 8 * (int64_t)o.z;
        v.D = w.blk(4 * (int64_t)o.w);
        v.Wa = w.blk(ra);
        v.Va = w.blk(ra + 4);
        if (slot) {
            v.Wb = w.blk(rb);
            v.Vb = w.blk(rb + 4);
        } else if (FWD) {
            v.z = wr.v2(rhs + 2 * (int64_t)o.w);
        }
        return v;
    };
    // all terms of a destination, the first two's values requested together
    auto terms = [&](const Ops& e, const Head& h, int t, bool slot, auto&& add) {
        const Val v = load(e.o, slot);
        if (!e.no) {
            add(v);
            return;
        }
        const Val u = load(e.p, slot);
        add(v);
        add(u);
        int at = h.two(t), nx = e.np;
        while (nx) {
            at += nx;
            const int4 o = S.g_op[at];
            nx = S.g_next[at];
            add(load(o, slot));
        }
    };
    for (int l0 = 0; l0 < nl; l0 += kWave) {
        const int m = nl - l0 < kWave ? nl - l0 : kWave;
        const int hl = (int)(threadIdx.x & (kWave - 1));
        const int4 ha = S.g_lev[2 * (l0 + (hl < m ? hl : m - 1))];
        const int4 hb = S.g_lev[2 * (l0 + (hl < m ? hl : m - 1)) + 1];
        // the table entry of a level, read where all lanes are active
        auto head = [&](int i) {
            const int k = i < m ? i : m - 1;
            return Head{__builtin_amdgcn_readlane(ha.x, k), __builtin_amdgcn_readlane(ha.y, k),
                        __builtin_amdgcn_readlane(ha.z, k), __builtin_amdgcn_readlane(hb.x, k),
                        __builtin_amdgcn_readlane(hb.y, k)};
        };
        Head h = head(0);
        Ops cur = fetch(h, me);
        for (int i = 0; i < m; ++i) {
            const Head hn = head(i + 1);
            for (int t = me; t < h.nd; t += all) {
                const Ops e = cur;
                if (t + all < h.nd) cur = fetch(h, t + all);
                if (e.o.x < 0) continue;
                bool ok;
                if (t < h.ns) {
                    const int64_t rd = lu + 8 * (int64_t)e.o.x;
                    Blk A = w.blk(rd), B = w.blk(rd + 4);
                    terms(e, h, t, true, [&](const Val& v) {
                        const Blk Di = binv(v.D, ok);
                        bmsub(A, v.Wa, bmul(Di, v.Vb));
                        bmsub(B, v.Wb, bmul(Di, v.Va));
                    });
                    w.put(rd, A);
                    w.put(rd + 4, B);
                } else {
                    const int64_t rd = 4 * (int64_t)e.o.x, zd = rhs + 2 * (int64_t)e.o.x;
                    Blk A = w.blk(rd);
                    double2 z = make_double2(0.0, 0.0);
                    if (FWD) z = wr.v2(zd);
                    terms(e, h, t, false, [&](const Val& v) {
                        const Blk Di = binv(v.D, ok);
                        bmsub(A, v.Wa, bmul(Di, v.Va));
                        if (FWD) {
                            double y0 = 0.0, y1 = 0.0;
                            mvadd(y0, y1, Di, v.z.x, v.z.y);
                            z.x = fma(-v.Wa.a, y0, fma(-v.Wa.b, y1, z.x));
                            z.y = fma(-v.Wa.c, y0, fma(-v.Wa.d, y1, z.y));
                        }
                    });
                    w.put(rd, A);
                    if (FWD) wr.put2(zd, z);
                }
            }
            h = hn;
            cur = fetch(h, me);
            par.sync();
        }
    }
}

// The rows of the upper levels below the tail normalised, after factor_ops:
// U_jk = D_j^-1 V_jk, y_j = D_j^-1 z_j and, with STORE_D, D_j^-1; kRowLanes
// lanes per node (of one wavefront, so that the pivot is read by all of them
// before it is replaced), nodes first, first + step, ....
constexpr int kRowLanes = 4;
template <bool FWD, bool STORE_D>
__device__ __forceinline__ void upper_rows(const DevSym& S, const View& w, int64_t lu,
                                           const View& wr, int64_t rhs, int* s_bad, int first,
                                           int step)
{
    const int x1 = S.level_ptr[S.mid_level];
    const int n = S.level_ptr[S.tail_level] - x1;
    const int lane = (int)threadIdx.x & (kRowLanes - 1);
    for (int i = first; i < n; i += step) {
        const int j = S.u_node[2 * i].x;
        const int4 b = S.u_node[2 * i + 1];
        bool ok;
        const Blk Di = binv(w.blk(4 * (int64_t)j), ok);
        double2 z = make_double2(0.0, 0.0);
        if (FWD) z = wr.v2(rhs + 2 * (int64_t)j);
        for (int t = b.z + lane; t < b.w; t += kRowLanes)
            w.put(lu + 8 * (int64_t)t + 4, bmul(Di, w.blk(lu + 8 * (int64_t)t + 4)));
        if (lane == 0) {
            if (!ok) mark_pivot(s_bad, x1 + i);
            if (STORE_D) w.put(4 * (int64_t)j, Di);
            if (FWD) {
                double y0 = 0.0, y1 = 0.0;
                mvadd(y0, y1, Di, z.x, z.y);
                wr.put2(rhs + 2 * (int64_t)j, make_double2(y0, y1));
            }
        }
    }
}

// The tail of the factorisation and, in a spread launch, the upper levels
// below it (from mid_level on).
// Phase A (all threads, no ordering): every diagonal, rhs entry and slot
//   there takes the updates of descendants below (global memory).
// Phase B: the levels upward, right-looking: once a level's pivots are
//   final, every block above that one of its nodes j updates (A_kl -= W_kj
//   D_j^-1 V_jl, the rhs with the diagonal) is one destination of the level's
//   operation list (t_op), the terms of a destination with several such nodes
//   in a fixed order; one barrier per level.  A level costs one short chain
//   (operands from LDS, the products, for a diagonal the determinant's
//   reciprocal) instead of a node's whole lower-neighbour list and a slot's
//   update list (up to 44 pairs) in one lane.  It is bound by the
//   instructions of that chain: on a level with few destinations a quad of
//   lanes shares one, a row of the result each (8 products per lane instead
//   of 32); with more than a quarter as many destinations as threads one
//   thread takes one, where further rounds of quads would cost more.
//   Measured per Newton step: 200 buses, 31 levels, 31 us left-looking, 22
//   us with one thread per destination, 20 us so; 10,000 buses, 256 cases,
//   56 levels and the updates from below, 237, 143 and 103 us.
// Phase C: all rows normalised at once (U_jk = D_j^-1 V_jk, y_j); the pivots
//   stay as they are in LDS.
// WRITE stores the tail's factors to global memory.
// With a Spread split, all workgroups share phase A for all upper levels, and
// then factorise those below the tail right-looking in global memory
// (factor_ops); the values lie in their own places there (D blocks, rhs
// entries, slot records), where workgroup 0 loads the tail from to run the
// rest, while the others normalise the rows below it and return.  A level
// costs one grid barrier and one short chain (an operation's values, the
// products) where the left-looking sweep walks a node's record, lists, blocks
// and update pairs: 4.5 against 8-14 us a level (one 10,000-bus case over 32
// workgroups, 19 levels).  One workgroup alone keeps the left-looking levels:
// there an operation's 19 scattered 16-byte accesses bound it, and a 2,000-bus
// batch of 1,024 took 2.41 instead of 1.72 ms.
template <class SRC, bool FWD, bool WRITE, class P = OneGroup>
__device__ __forceinline__ void upper_factor(const DevSym& S, const SRC& src, const View& w,
                                             int64_t lu, const View& wr, int64_t rhs, int* s_bad,
                                             const P& par = P{})
{
    const int K = S.tail_nodes, TS = S.tail_slots;
    const int nT = S.nlev - S.tail_level;
    const TailLds L(S);
    const int T = wg_size();
    // the items: all of the upper levels, or the tail's alone
    const int x0 = P::kSpread ? 0 : S.level_ptr[S.tail_level] - S.level_ptr[S.mid_level];
    const int y0 = P::kSpread ? 0 : S.u_slots - TS;
    const int UN = S.nn - S.level_ptr[S.mid_level] - x0, US = S.u_slots - y0;
    const int a0 = par.rank() * T + (int)threadIdx.x, as = par.size() * T;
    for (int it = a0; it < UN + US; it += as) {
        if (it < UN) {
            const int4 t0 = S.u_node[2 * (x0 + it)];
            const int4 t1 = S.u_node[2 * (x0 + it) + 1];
            const int r1 = P::kSpread ? t1.y : t0.w;
            Blk acc = src.diag(t0.x, t0.y, t0.z);
            double z0 = 0.0, z1 = 0.0;
            if constexpr (FWD) {
                double2 b;
                if constexpr (SRC::kRhsInRecord) b = src.rhs_at(t0.y);
                else b = wr.v2(rhs + 2 * (int64_t)t0.x);
                z0 = b.x;
                z1 = b.y;
            }
            // lower neighbours below the upper levels: four per step, their
            // blocks and y requested together, the next four indices in
            // flight (entries past the list's end are not loaded)
            if (t1.x < r1) {
                int2 e[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) e[k] = upd_at(S.u_rl, t1.x + k, r1);
                for (int r = t1.x; r < r1; r += 4) {
                    int2 nx[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) nx[k] = upd_at(S.u_rl, r + 4 + k, r1);
                    Blk wv[4], uv[4];
                    double2 yi[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        wv[k] = bzero();
                        uv[k] = bzero();
                        yi[k] = make_double2(0.0, 0.0);
                        if (r + k < r1) {
                            wv[k] = w.blk(lu + 8 * (int64_t)e[k].y);
                            uv[k] = w.blk(lu + 8 * (int64_t)e[k].y + 4);
                            if (FWD) yi[k] = wr.v2(rhs + 2 * (int64_t)e[k].x);
                        }
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (r + k < r1) {
                            bmsub(acc, wv[k], uv[k]);
                            if (FWD) {
                                z0 = fma(-wv[k].a, yi[k].x, fma(-wv[k].b, yi[k].y, z0));
                                z1 = fma(-wv[k].c, yi[k].x, fma(-wv[k].d, yi[k].y, z1));
                            }
                        }
                    }
#pragma unroll
                    for (int k = 0; k < 4; ++k) e[k] = nx[k];
                }
            }
            if constexpr (!P::kSpread) {
                L.setD(it, acc);
                L.sety(it, z0, z1);
            } else {
                w.put(4 * (int64_t)t0.x, acc);
                if (FWD) wr.put2(rhs + 2 * (int64_t)t0.x, make_double2(z0, z1));
            }
        } else {
            const int t = it - UN;
            const int4 a = S.u_slot[2 * (y0 + t)];
            const int4 b = S.u_slot[2 * (y0 + t) + 1];
            Blk Wk, Vk;
            src.off(a.x, a.y, a.z, a.w, b.x, Wk, Vk);
            apply_updates(S.u_upd, b.y, P::kSpread ? b.z : b.w, w, lu, Wk, Vk);
            if constexpr (!P::kSpread) {
                L.setW(t, Wk);
                L.setU(t, Vk);
            } else {
                w.put(lu + 8 * (int64_t)a.x, Wk);
                w.put(lu + 8 * (int64_t)a.x + 4, Vk);
            }
        }
    }
    if constexpr (P::kSpread) {
        par.sync();
        factor_ops<FWD>(par, S, w, lu, wr, rhs);
        const int g0 = K > 0 ? 1 : 0;  // workgroup 0 has the tail to do
        if (par.rank() >= g0)
            upper_rows<FWD, WRITE>(S, w, lu, wr, rhs, s_bad,
                                   ((par.rank() - g0) * T + (int)threadIdx.x) / kRowLanes,
                                   (par.size() - g0) * T / kRowLanes);
        if (par.rank() != 0) return;
        for (int it = threadIdx.x; it < K + TS; it += T) {
            if (it < K) {
                const int j = S.t_node[2 * it].x;
                L.setD(it, w.blk(4 * (int64_t)j));
                const double2 z = FWD ? wr.v2(rhs + 2 * (int64_t)j) : make_double2(0.0, 0.0);
                L.sety(it, z.x, z.y);
            } else {
                const int t = it - K;
                const int64_t sg = lu + 8 * (int64_t)S.t_slot[t].x;
                L.setW(t, w.blk(sg));
                L.setU(t, w.blk(sg + 4));
            }
        }
    }
    __syncthreads();
    if (K == 0) return;
    // A quad of lanes per destination, a row of the result each: lanes 0 and
    // 1 the rows of W_d -= W_a D_j^-1 V_b (or of the diagonal), lanes 2 and 3
    // those of V_d -= W_b D_j^-1 V_a (or the entries of z_d -= W_a D_j^-1
    // z_j), as a row of the left block times D_j^-1, then times the right
    // block.
    const int row = (int)threadIdx.x & 1;
    const bool hi = ((int)threadIdx.x & 2) != 0;
    // this lane's first entry of destination d
    auto target = [&](int d, bool slot) {
        return slot ? reinterpret_cast<double*>(L.r + (2 * hi + row) * TS + d)
                    : hi ? L.y + 2 * d + row : L.d + 4 * d + 2 * row;
    };
    auto take = [&](const TailOp& e, bool zrow, double& a0, double& a1) {
        const double2 l = L.r[row * TS + (hi ? e.b : e.a)];
        const double2* const right = zrow ? reinterpret_cast<const double2*>(L.y) + e.j
                                          : L.r + 2 * TS + (hi ? e.a : e.b);
        const double2 u = right[0], v = right[zrow ? 0 : TS];
        const double2 t = L.over(l, e.j);
        a0 = fma(-t.x, u.x, fma(-t.y, zrow ? v.y : v.x, a0));
        a1 = fma(-t.x, u.y, fma(-t.y, v.y, a1));
    };
    auto finish = [&](double* dst, int d, bool slot, double a0, double a1) {
        dst[0] = a0;
        if (slot || !hi) dst[1] = a1;
        if (!slot) {
            // the pivot's determinant from its two rows
            const double b0 = dpp_peer<0xB1>(a0), b1 = dpp_peer<0xB1>(a1);
            if (!hi && row == 0) L.q[d] = 1.0 / bdet({a0, a1, b0, b1});
        }
    };
    auto quad = [&](const uint2& q, const uint2& second, auto&& at2, bool slot) {
        const int d = tail_op(q).d;
        double* const dst = target(d, slot);
        double a0 = dst[0], a1 = dst[1];
        tail_terms(S, q, second, at2(), [&](const TailOp& e) { take(e, hi && !slot, a0, a1); });
        finish(dst, d, slot, a0, a1);
    };
    // A long destination's rest: a quad of the wavefront per operation, their
    // sums added up over the quads.
    auto rest = [&](int d, int at2, bool slot) {
        double a0 = 0.0, a1 = 0.0;
        tail_rest(S, at2, ((int)threadIdx.x & (kWave - 1)) >> 2, kWave / 4,
                  [&](const TailOp& e) { take(e, hi && !slot, a0, a1); });
        for (int k = 4; k < kWave; k *= 2) {
            a0 += __shfl_xor(a0, k, kWave);
            a1 += __shfl_xor(a1, k, kWave);
        }
        if (((int)threadIdx.x & (kWave - 1)) < 4) {
            double* const dst = target(d, slot);
            finish(dst, d, slot, dst[0] + a0, dst[1] + a1);
        }
    };
    // One thread per destination, one form for both kinds, so that a wavefront
    // holding both runs one path: A -= W_a D_j^-1 V_b with A = W_d or the
    // diagonal D_d, and B -= W_b D_j^-1 X with B = V_d, X = V_a, or (a = b)
    // B = z_d, X = z_j as the first column of a block.  The same operations in
    // the same order as a quad's: which of them a level takes depends on the
    // workgroup's size, the results (and a zero pivot's verdict) do not.
    auto lane = [&](const uint2& q, const uint2& second, auto&& at2, bool slot) {
        const int d = tail_op(q).d;
        double2* const a0 = slot ? L.r + d : reinterpret_cast<double2*>(L.d) + 2 * d;
        double2* const a1 = slot ? L.r + TS + d : a0 + 1;
        double2* const b0 = slot ? L.r + 2 * TS + d : reinterpret_cast<double2*>(L.y) + d;
        double2* const b1 = slot ? L.r + 3 * TS + d : b0;
        auto as_block = [&](const double2& u, const double2& v) {
            return Blk{u.x, slot ? u.y : 0.0, slot ? v.x : u.y, slot ? v.y : 0.0};
        };
        const double2 u = *a0, v = *a1;
        Blk A = {u.x, u.y, v.x, v.y};
        Blk B = as_block(*b0, *b1);
        tail_terms(S, q, second, at2(), [&](const TailOp& e) {
            const double2* const x0 =
                slot ? L.r + 2 * TS + e.a : reinterpret_cast<const double2*>(L.y) + e.j;
            const double2* const x1 = slot ? L.r + 3 * TS + e.a : x0;
            const Blk Vb = L.U(e.b), X = as_block(*x0, *x1);
            bmsub(A, L.W_over(e.a, e.j), Vb);
            bmsub(B, L.W_over(e.b, e.j), X);
        });
        *a0 = make_double2(A.a, A.b);
        *a1 = make_double2(A.c, A.d);
        *b0 = make_double2(B.a, slot ? B.b : B.c);
        if (slot) *b1 = make_double2(B.c, B.d);
        else L.q[d] = 1.0 / bdet(A);
    };
    // only a tail with long destinations takes the form that looks for them (a
    // path of 150 buses, no long ones: 356 us, in that form 366; 198 leaves on
    // one bus: 314 us walked one after the other, so 222)
    // A spread launch takes it always: the code of a second form there slowed
    // one 10,000-bus case by 1% (1,222 -> 1,234 us) and the 64 mixed grids as much.
    constexpr bool always = P::kSpread;
    if (always || S.tail_longs) for_tail_updates<true>(S, nT, quad, lane, rest);
    else if constexpr (!always) for_tail_updates<false>(S, nT, quad, lane, rest);
    for (int it = threadIdx.x; it < K + TS; it += blockDim.x) {
        if (it < K) {
            const Blk D = bload(L.d + 4 * it);
            bool ok;
            (void)binv(D, ok);
            if (!ok) mark_pivot(s_bad, S.level_ptr[S.tail_level] + it);
            if (FWD) {
                const double2 z = L.yv(it);
                const Blk Di = L.Dinv(it);
                double y0 = 0.0, y1 = 0.0;
                mvadd(y0, y1, Di, z.x, z.y);
                L.sety(it, y0, y1);
            }
        } else {
            const int t = it - K;
            L.setU(t, bmul(L.Dinv(S.t_slot[t].z), L.U(t)));
        }
    }
    __syncthreads();
    if (WRITE) {
        for (int t = threadIdx.x; t < TS; t += blockDim.x) {
            const int s = S.t_slot[t].x;
            w.put(lu + 8 * (int64_t)s, L.W(t));
            w.put(lu + 8 * (int64_t)s + 4, L.U(t));
        }
        for (int jl = threadIdx.x; jl < K; jl += blockDim.x) {
            const int j = S.t_node[2 * jl].x;
            w.put(4 * (int64_t)j, L.Dinv(jl));
            if (FWD) wr.put2(rhs + 2 * (int64_t)j, L.yv(jl));
        }
        __syncthreads();
    }
}

// Newton step of one bus: theta -= dtheta, |V| -= d|V| (PQ), new e + jf;
// the record's first 32 bytes (e, f, |V|, theta) are rewritten in one store.
__device__ __forceinline__ void apply_step_to(const View& w, int64_t rec, const Blk& r, bool pv,
                                              double x0, double x1)
{
    const double va = r.d - x0;
    const double vm = pv ? r.c : r.c - x1;
    double sn, cs;
    sincos(va, &sn, &cs);
    w.put(rec, {vm * cs, vm * sn, vm, va});
}

__device__ __forceinline__ void apply_step(const View& w, int64_t rec, bool pv, double x0,
                                           double x1)
{
    apply_step_to(w, rec, w.blk(rec), pv, x0, x1);
}

// Backward substitution of the tail from LDS: x_j = y_j - sum U_jk x_k.  The
// clique goes first, on the first wavefront alone, column-oriented (a node per
// lane in registers as far as the lanes go: 200 buses 136 -> 122 us): once x_a
// is final, y_k -= U_ka x_a for every clique node k below a.  Every node
// below the clique then takes the clique's terms, and the levels follow
// downward, column-oriented too: one thread per slot whose higher neighbour
// is on the level (each lower node has at most one of them).  The x of the
// tail nodes are written to the rhs (for the levels below) and, with UPDATE,
// applied to the bus records in one parallel pass at the end, so that no
// level waits for a bus-record load.  With xs (the solution vector in LDS by
// position, over the tail's own LDS; at most four tail nodes per thread) the
// x go there instead of the rhs: each thread takes its x into registers,
// and writes them after a barrier.
template <bool UPDATE>
__device__ __forceinline__ void tail_backward(const DevSym& S, const View& w, int64_t rhs,
                                              int64_t bus_off, PvMask type, double2* xs)
{
    const int K = S.tail_nodes, KC = S.tail_clique;
    const int nT = S.nlev - S.tail_level;
    const TailLds L(S);
    double* const sy = L.y;
    const int kf = K - KC;
    if (KC > 0) {
        const int c0 = S.t_node[2 * kf].w;
        if (KC <= kWave) {
            if (threadIdx.x < kWave) {
                const int k = threadIdx.x;
                double2 y = make_double2(0.0, 0.0);
                if (k < KC) y = L.yv(kf + k);
                auto column = [&](int a) {
                    return k < a ? L.U(clique_slot(c0, KC, k, a)) : bzero();
                };
                Blk U = column(KC - 1);
                for (int a = KC - 1; a > 0; --a) {
                    const Blk next = column(a - 1);
                    const double x0 = lane_value(y.x, a), x1 = lane_value(y.y, a);
                    if (k < a) {
                        y.x = fma(-U.a, x0, fma(-U.b, x1, y.x));
                        y.y = fma(-U.c, x0, fma(-U.d, x1, y.y));
                    }
                    U = next;
                }
                if (k < KC) L.sety(kf + k, y.x, y.y);
            }
        } else if (threadIdx.x < kWave) {
            for (int a = KC - 1; a > 0; --a) {
                const int ja = kf + a;
                const double2 x = L.yv(ja);
                for (int k = threadIdx.x; k < a; k += kWave) {
                    const int jk = kf + k;
                    const Blk U = L.U(clique_slot(c0, KC, k, a));
                    const double2 y = L.yv(jk);
                    L.sety(jk, fma(-U.a, x.x, fma(-U.b, x.y, y.x)),
                           fma(-U.c, x.x, fma(-U.d, x.y, y.y)));
                }
                wave_sync();
            }
        }
        __syncthreads();
        // the clique's terms of every node below it
        for (int jl = threadIdx.x; jl < kf; jl += blockDim.x) {
            const int t0 = S.t_node[2 * jl].w, t1 = S.t_node[2 * jl + 1].x;
            double2 y = L.yv(jl);
            bool more = true;
            for (int t = t1 - 1; more && t >= t0; t -= 4) {  // the clique's are the last ones
                int kk[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) kk[i] = S.t_slot[t - i >= t0 ? t - i : t0].y;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    more = more && t - i >= t0 && kk[i] >= kf;
                    if (more) {
                        const Blk U = L.U(t - i);
                        const double2 x = L.yv(kk[i]);
                        y.x = fma(-U.a, x.x, fma(-U.b, x.y, y.x));
                        y.y = fma(-U.c, x.x, fma(-U.d, x.y, y.y));
                    }
                }
            }
            L.sety(jl, y.x, y.y);
        }
        __syncthreads();
    }
    for_tail_ops<false, false>(S, nT - KC, [&](const uint2& q) {
        const TailOp o = tail_op(q);
        const Blk U = L.U(o.a);
        const double2 x = L.yv(o.b), y = L.yv(o.d);
        L.sety(o.d, fma(-U.a, x.x, fma(-U.b, x.y, y.x)),
               fma(-U.c, x.x, fma(-U.d, x.y, y.y)));
    }, [](int, int) {});
    if (xs) {
        double2 xr[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int jl = threadIdx.x + r * blockDim.x;
            xr[r] = jl < K ? make_double2(sy[2 * jl], sy[2 * jl + 1]) : make_double2(0.0, 0.0);
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int jl = threadIdx.x + r * blockDim.x;
            if (jl < K) {
                const int4 t0 = S.t_node[2 * jl];
                xs[t0.x] = xr[r];
                if (UPDATE)
                    apply_step(w, bus_off + 8 * (int64_t)t0.y, type(t0.y), xr[r].x, xr[r].y);
            }
        }
    } else {
        for (int jl = threadIdx.x; jl < K; jl += blockDim.x) {
            const int4 t0 = S.t_node[2 * jl];
            const double x0 = sy[2 * jl], x1 = sy[2 * jl + 1];
            w.put2(rhs + 2 * (int64_t)t0.x, make_double2(x0, x1));
            if (UPDATE) apply_step(w, bus_off + 8 * (int64_t)t0.y, type(t0.y), x0, x1);
        }
    }
    __syncthreads();
}

// Backward substitution of node record x: x_j = y_j - sum_{k in S(j)} U_jk x_k,
// four slots per lane at a time (next indices in flight), the node's own
// rhs entry and bus record requested first.
template <bool UPDATE>
__device__ __forceinline__ void back_node(const DevSym& S, const NodeRec& rec, int lane, int g,
                                          const View& w, int64_t lu, const View& wb,
                                          int64_t rhs, int64_t bus_off, PvMask type,
                                          double2* xs)
{
    const int4 n0 = rec.a;
    const int4 n1 = rec.b;
    const int s1 = n1.y;
    const double2 y = wb.v2(rhs + 2 * (int64_t)n0.x);
    const int64_t brec = bus_off + 8 * (int64_t)n0.y;
    Blk br = bzero();
    bool pv = false;
    if (UPDATE) {
        br = wb.blk(brec);
        pv = type(n0.y);
    }
    // absent entries are not loaded (skipped when no lane needs them)
    int s = n1.x + lane;
    int kk[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        kk[k] = 0;
        if (s + k * g < s1) kk[k] = S.Li[s + k * g];
    }
    double a0 = 0.0, a1 = 0.0;
    for (; s < s1; s += 4 * g) {
        Blk u[4];
        double2 xk[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            u[k] = bzero();
            xk[k] = make_double2(0.0, 0.0);
            if (s + k * g < s1) {
                u[k] = w.blk(lu + 8 * (int64_t)(s + k * g) + 4);
                xk[k] = xs ? xs[kk[k]] : wb.v2(rhs + 2 * (int64_t)kk[k]);
            }
        }
        const int sn = s + 4 * g;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (sn + k * g < s1) kk[k] = S.Li[sn + k * g];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (s + k * g < s1) mvadd(a0, a1, u[k], xk[k].x, xk[k].y);
    }
    if (g > 1) {
        gsum2(a0, a1, g);
    }
    if (lane == 0) {
        const double x0 = y.x - a0, x1 = y.y - a1;
        if (xs) xs[n0.x] = make_double2(x0, x1);
        else wb.put2(rhs + 2 * (int64_t)n0.x, make_double2(x0, x1));
        if (UPDATE) apply_step_to(wb, brec, br, pv, x0, x1);
    }
}

// Max over the workgroup with a NaN flag; every thread gets the result.
__device__ __forceinline__ double block_max(double v, int nan, int& any_nan)
{
    __shared__ double s_v[kMaxThreads / 64 + 1];
    __shared__ int s_n[kMaxThreads / 64 + 1];
    for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
    nan = __any(nan);
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_v[wv] = v;
        s_n[wv] = nan;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0;
        int fl = 0;
        for (int i = 0; i < (int)(blockDim.x + 63) / 64; ++i) {
            m = fmax(m, s_v[i]);
            fl |= s_n[i];
        }
        s_v[kMaxThreads / 64] = m;
        s_n[kMaxThreads / 64] = fl;
    }
    __syncthreads();
    const double r = s_v[kMaxThreads / 64];
    any_nan = s_n[kMaxThreads / 64];
    __syncthreads();
    return r;
}

struct NewtonArgs {
    const double* yval;
    int64_t y_stride;
    const int8_t* type;
    int64_t type_stride;
    const double* Psp;
    const double* Qsp;
    int64_t inj_stride;
    double* Vm;
    double* Va;
    int64_t v_stride;
    double* ws;
    int64_t ws_stride;
    double tol;
    int max_iter;
    int flags;
    int interleave;
    int B;
    int32_t* iters;
    double* norm;
    int32_t* status;
    int32_t* pivot;  // position of the first zero pivot, -1 if none (may be null)
};

// Arguments of the fused adjoint kernel (pf_adjoint).
struct AdjArgs {
    double* ws;  // pf_newton's workspace: factors of J at the solution
    int64_t ws_stride;
    int C;  // interleave of the workspace
    int B;
    const double* gVm;  // dL/d|V| [B][n] or null
    const double* gVa;  // dL/dtheta [B][n] or null
    int64_t gv_stride;
    const int8_t* type;
    int64_t type_stride;
    const int32_t* status;  // pf_newton's per-case status or null
    double* lam;            // out: adjoint vector [B][nn][2]
    int64_t lam_stride;
    double* gP;
    double* gQ;
    int64_t g_stride;
    // branch gradients in the same launch (gx null: none)
    const int32_t* from;
    const int32_t* to;
    const double* Vm;
    const double* Va;
    int64_t v_stride;
    const double* r;
    const double* x;
    int64_t branch_stride;
    double* gx;   // gx_mode 0: dL/dx [B][m]; 1: null here, per-case parts to the workspace
    int gx_mode;  // 0 per case, 1 summed over the cases (by k_adj_gx_sum)
};

struct CaseDesc {
    DevSym sym;
    int64_t bus_off, br_off, y_off, ws_off;
    // a batch of grids spread over more workgroups than cases: this case's
    // workgroup count, its grid-barrier words (doubles after ws_off) and the
    // first backward level left to its first workgroup
    int64_t sync_off;
    int32_t spread, back_lo;
};

// What the mismatch pass does with a bus's P, Q, F_P, F_Q: Newton stores all
// four in the second half of the bus record, in one store ...
struct MisNewton {
    const View& wb;
    int64_t bus_off;
    __device__ __forceinline__ double scale(int) const { return 1.0; }
    __device__ __forceinline__ void put(int i, int, double, double p, double q, double fp,
                                        double fq) const
    {
        wb.put(bus_off + 8 * (int64_t)i + 4, {p, q, fp, fq});
    }
};
// ... the fast decoupled iteration the right-hand side of its next half step,
// F_P / |V| or (second) F_Q / |V|, by position.
struct MisHalf {
    const double* vm;
    double* b;
    bool second;
    __device__ __forceinline__ double scale(int i) const { return vm[i]; }
    __device__ __forceinline__ void put(int, int pos, double v, double, double, double fp,
                                        double fq) const
    {
        b[pos] = (second ? fq : fp) / v;
    }
};

// Mismatch pass of one case: F = calculated - scheduled (F_Q = 0 at PV buses)
// and P + jQ, into out.  The thread's max |F| and NaN flag accumulate into mx
// and nan.  Buses are taken in bus
// order, NB per thread per step (blockDim apart), so that the admittance
// rows, row pointers, positions and scheduled injections of a wavefront are
// adjacent in memory; all loads of a step's buses are issued before any of
// them is summed.  The buses are first, first + stride, ... (the thread's
// index and count over the workgroups that share the case).
template <int NB, class EF, class OUT>
__device__ __forceinline__ void mismatch_pass(const DevSym& S, const double* yv, const EF& ef,
                                              const OUT& out, const PvMask& pvm,
                                              const double* Psp, const double* Qsp, double& mx,
                                              int& nan, int first, int stride)
{
    const int bd = stride;
    for (int i0 = first; i0 < S.n; i0 += NB * bd) {
        int ib[NB], pc[NB], q0[NB], q1[NB];
        bool has[NB], pv[NB];
        double sp[NB], sq[NB], sc[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            has[k] = i0 + k * bd < S.n;
            ib[k] = has[k] ? i0 + k * bd : i0;
            pc[k] = S.pos[ib[k]];
            q0[k] = S.yptr[ib[k]];
            q1[k] = S.yptr[ib[k] + 1];
            sp[k] = Psp[ib[k]];
            sq[k] = Qsp[ib[k]];
            sc[k] = out.scale(ib[k]);
        }
        double ve[NB], vf[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            ef.get(ib[k], ve[k], vf[k]);
            pv[k] = pvm(ib[k]);
        }
        int kk[NB][4];
        RowHead h[NB];
#pragma unroll
        for (int k = 0; k < NB; ++k) row_head_idx<EF>(S, yv, q0[k], q1[k], kk[k], h[k]);
#pragma unroll
        for (int k = 0; k < NB; ++k) row_head_v(ef, kk[k], h[k]);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            double p, q;
            row_finish(S, yv, ef, q0[k], q1[k], h[k], ve[k], vf[k], p, q);
            if (has[k] && pc[k] >= 0) {  // the slack is not a position
                const double fp = p - sp[k], fq = pv[k] ? 0.0 : q - sq[k];
                out.put(ib[k], pc[k], sc[k], p, q, fp, fq);
                nan |= (fp != fp) | (fq != fq);
                mx = fmax(mx, fmax(fabs(fp), fabs(fq)));
            }
        }
    }
}

}  // namespace
