// libpf fast decoupled power flow and branch flows (device code, kernels and
// their C ABI entry points).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <numeric>
#include <string>
#include <type_traits>
#include <vector>

#include "pf.h"
#include "pf_device.h"
#include "pf_host.h"

using namespace pf::abi;

namespace {

// ---------------------------------------------------------------------------
// Fast decoupled power flow (Sec. III names it beside NR; Table III times it),
// XB matrices: B' from branch reactances only, B'' = -Im(Y) of the full
// pi-model, both symmetric, so the paper's factorisation is LDL^T (eqs. 1-3)
// with scalar elements.  Per matrix: d section [fd_lu] then (w, u) per slot
// with w_kj = l_kj d_j and u_jk = l_kj; after factorisation d holds 1/d_j.
// B'' of a PV bus is the identity row and column, so its |V| never moves.
// ---------------------------------------------------------------------------

// Entries of B' and B'' from the branches [t0, t1) of an admittance entry's
// list, the first of them e0: one walk for both, four branches in flight (a bus
// with 200 branches: 65 us walked twice, 86 so and one load at a time, now 33;
// 2,000 ordinary buses 10.3 -> 7.6).
__device__ __forceinline__ double2 fd_entries(const DevSym& S, int t0, int t1, int e0, bool diag,
                                              const double* __restrict__ r,
                                              const double* __restrict__ x,
                                              const double* __restrict__ b)
{
    double v1 = 0.0, v2 = 0.0;
    auto add = [&](double rr, double xx, double bb) {
        const double bx = 1.0 / xx;
        const double bs = xx / (rr * rr + xx * xx);
        v1 += diag ? bx : -bx;
        v2 += diag ? bs - bb / 2.0 : -bs;
    };
    if (t0 < t1) add(r[e0], x[e0], b[e0]);
    int e[4];
    if (t0 + 1 < t1) {
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = t0 + 1 + k < t1 ? S.ybr[t0 + 1 + k] : e0;
    }
    for (int t = t0 + 1; t < t1; t += 4) {
        double rr[4], xx[4], bb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            rr[k] = r[e[k]];
            xx[k] = x[e[k]];
            bb[k] = b[e[k]];
        }
        if (t + 4 < t1) {
#pragma unroll
            for (int k = 0; k < 4; ++k) e[k] = t + 4 + k < t1 ? S.ybr[t + 4 + k] : e0;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (t + k < t1) add(rr[k], xx[k], bb[k]);
    }
    return make_double2(v1, v2);
}

// Left-looking LDL^T of one node (pull form, like factor_node with 1x1
// blocks and U = L^T):
//   d_j = a_jj - sum_{i in R(j)} w_ji u_ij,
//   w_kj = a_kj - sum_i w_ki u_ij (k in S(j)),  u_jk = w_kj / d_j.
// Bound by its chains of loads (list, then factor entries), so four terms are
// requested at a time, the next four's indices under them: both matrices of
// 384 cases of 2,000 buses 183 -> 155 us.  A wavefront without a second term
// takes the one (a radial grid of 2,000 buses 1,954 us four at a time, 1,792 so).
__device__ __forceinline__ void fd_factor_node(const DevSym& S, const NodeRec& rec, int lane,
                                               int g, double* m, int* s_bad)
{
    const int j = rec.a.x;
    double2* sl = reinterpret_cast<double2*>(m + S.fd_lu);
    double ds = 0.0;
    const int r0 = rec.a.z + lane, r1 = rec.a.w;
    if (!__any(r0 + g < r1)) {  // a radial grid's nodes: no lane has a second one
        if (r0 < r1) {
            const double2 wu = sl[S.rl[r0].y];
            ds = wu.x * wu.y;
        }
    } else {
        for (int r = r0; r < r1; r += 4 * g) {
            int at[4];
            double2 wu[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) at[k] = S.rl[r + k * g < r1 ? r + k * g : r].y;
#pragma unroll
            for (int k = 0; k < 4; ++k) wu[k] = sl[at[k]];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (r + k * g < r1) ds = fma(wu[k].x, wu[k].y, ds);
        }
    }
    if (g > 1) ds = gsum(ds, g);
    const double D = m[j] - ds;
    const bool ok = D != 0.0 && isfinite(D);
    const double Dinv = 1.0 / D;
    for (int s = rec.b.x + lane; s < rec.b.y; s += g) {
        const int4 b = S.slot_info[2 * s + 1];
        double W = sl[s].x;
        int2 p[4];
        if (b.x < b.y) {
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = S.upd[b.x + k < b.y ? b.x + k : b.x];
        }
        for (int u = b.x; u < b.y; u += 4) {
            double w[4], v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w[k] = sl[p[k].x].x;
                v[k] = sl[p[k].y].y;
            }
            const int un = u + 4 < b.y ? u + 4 : u;
#pragma unroll
            for (int k = 0; k < 4; ++k) p[k] = S.upd[un + k < b.y ? un + k : un];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (u + k < b.y) W = fma(-w[k], v[k], W);
        }
        sl[s] = make_double2(W, W * Dinv);
    }
    if (lane == 0) {
        m[j] = Dinv;
        if (!ok) *s_bad = 1;
    }
}

// Forward substitution and normalisation:
//   y_j = (1/d_j) (b_j - sum_{i in R(j)} w_ji y_i), levels [0, l1) upward.
// Four entries per lane per batch with the next batch's indices in flight;
// the node's own b_j and 1/d_j are requested first.  b holds the right-hand
// side and x the half step's work vector, both by position.
__device__ __forceinline__ void fd_forward(const DevSym& S, const double* m, const double* b,
                                           double* x, int l1)
{
    const double2* sl = reinterpret_cast<const double2*>(m + S.fd_lu);
    for_nodes(S, 0, l1, true, [&](int, const NodeRec& rec, int lane, int g) {
        const int j = rec.a.x, r1 = rec.a.w;
        const double bj = b[j];
        const double dj = m[j];
        int r = rec.a.z + lane;
        // absent entries are not loaded (skipped when no lane needs them)
        int2 e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            e[k] = make_int2(0, 0);
            if (r + k * g < r1) e[k] = S.rl[r + k * g];
        }
        double z = 0.0;
        for (; r < r1; r += 4 * g) {
            double w[4], y[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w[k] = 0.0;
                y[k] = 0.0;
                if (r + k * g < r1) {
                    w[k] = sl[e[k].y].x;
                    y[k] = x[e[k].x];
                }
            }
            const int rn = r + 4 * g;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (rn + k * g < r1) e[k] = S.rl[rn + k * g];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (r + k * g < r1) z = fma(w[k], y[k], z);
        }
        if (g > 1) z = gsum(z, g);
        if (lane == 0) x[j] = dj * (bj - z);
    });
}

// State of one case.  |V| and theta are updated in the caller's arrays; the
// workspace keeps (cos, sin) of theta per bus (the magnitude half step leaves
// them as they are) and (e, f) for the mismatch pass, which is copied to or
// made in LDS when it has room there.
struct FdState {
    double* Vm;
    double* Va;
    double2* cs;
    double2* ef;
};

// The half step of every bus from the solution x by position: theta -= x
// (ANGLE), else |V| -= x at PQ buses.  In bus order, as every array but x is
// then read and written contiguously (done with each node's substitution
// instead it put a bus record's load, the sine and the store at the end of
// every level).  The next bus's loads are in flight under the sine: taking
// several buses at once instead needs more registers than two workgroups per
// compute unit leave.
template <bool ANGLE, class E>
__device__ __forceinline__ void fd_half_step(const DevSym& S, const FdState& st,
                                             const PvMask& pv, const double* x, E&& put_ef)
{
    struct Bus {
        double vm, x;
        double2 t;  // theta, or (cos, sin)
    };
    const int T = wg_size(), n = S.n;
    auto load = [&](int i, int p) {
        Bus b{0.0, 0.0, make_double2(0.0, 0.0)};
        if (i < n) {
            b.vm = st.Vm[i];
            if (ANGLE) b.t.x = st.Va[i];
            else b.t = st.cs[i];
            if (p >= 0) b.x = x[p];
        }
        return b;
    };
    int i = fresh_thread();
    int p = i < n ? S.pos[i] : -1, pn = i + T < n ? S.pos[i + T] : -1;
    Bus b = load(i, p);
    while (i < n) {
        const int p2 = i + 2 * T < n ? S.pos[i + 2 * T] : -1;
        const Bus next = load(i + T, pn);
        double vm = b.vm;
        double2 cs = b.t;
        if (ANGLE) {
            double va = b.t.x;
            if (p >= 0) {  // the slack keeps its voltage
                va -= b.x;
                st.Va[i] = va;
            }
            sincos(va, &cs.y, &cs.x);
            st.cs[i] = cs;
        } else if (p >= 0 && !pv(i)) {
            vm -= b.x;
            st.Vm[i] = vm;
        }
        put_ef(i, make_double2(vm * cs.x, vm * cs.y));
        i += T;
        p = pn;
        pn = p2;
        b = next;
    }
}

// The top of the tree (the LDS tail's levels) of a factored matrix, copied
// into LDS once per launch: (w, u) per local slot, 1/d per local node.
struct FdTail {
    double2* wu;  // TS
    double* d;    // K
};

__device__ __forceinline__ void fd_tail_load(const DevSym& S, const double* m, const FdTail& t)
{
    const double2* sl = reinterpret_cast<const double2*>(m + S.fd_lu);
    for (int i = threadIdx.x; i < S.tail_slots; i += blockDim.x) t.wu[i] = sl[S.t_slot[i].x];
    for (int i = threadIdx.x; i < S.tail_nodes; i += blockDim.x) t.d[i] = m[S.t_node[2 * i].x];
}

// Forward substitution of the tail levels in LDS: each tail node first takes
// b_j and the terms of its descendants outside the
// tail (global lists, all nodes at once), then the tail levels go upward
// with the local lists.  y of the tail stays in sy for the backward sweep.
__device__ __forceinline__ void fd_forward_tail(const DevSym& S, const double* m, const FdTail& t,
                                                double* sy, const double* rhs, const double* x)
{
    const double2* sl = reinterpret_cast<const double2*>(m + S.fd_lu);
    for (int jl = threadIdx.x; jl < S.tail_nodes; jl += blockDim.x) {
        const int4 a = S.t_node[2 * jl], b = S.t_node[2 * jl + 1];
        double z = rhs[a.x];
        const int r1 = b.z;
        int r = b.y;
        int2 e[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) e[k] = S.t_rl[r + k < r1 ? r + k : 0];
        for (; r < r1; r += 4) {
            double w[4], y[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                w[k] = sl[e[k].y].x;
                y[k] = x[e[k].x];
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) e[k] = S.t_rl[r + 4 + k < r1 ? r + 4 + k : 0];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (r + k < r1) z = fma(-w[k], y[k], z);
        }
        sy[jl] = z;
    }
    __syncthreads();
    // the levels below the clique, right-looking: the diagonal operations of
    // the factorisation's lists carry the rhs terms z_k -= w_kj (z_j / d_j)
    const int nT = S.nlev - S.tail_level, KC = S.tail_clique;
    const int kf = S.tail_nodes - KC;
    auto one = [&](const uint2& q, const uint2& second, int at) {
        const int d = tail_op(q).d;
        double z = sy[d];
        tail_terms(S, q, second, at, [&](const TailOp& o) {
            z = fma(-t.wu[o.a].x, t.d[o.j] * sy[o.j], z);
        });
        sy[d] = z;
    };
    auto rest = [&](int d, int at) {
        const int lane = (int)threadIdx.x & (kWave - 1);
        double z = 0.0;
        tail_rest(S, at, lane, kWave, [&](const TailOp& o) {
            z = fma(-t.wu[o.a].x, t.d[o.j] * sy[o.j], z);
        });
        z = gsum(z, kWave);
        if (lane == 0) sy[d] += z;
    };
    if (S.tail_longs) for_tail_ops<true, true>(S, nT - KC, one, rest);
    else for_tail_ops<true, false>(S, nT - KC, one, rest);
    for (int jl = threadIdx.x; jl < kf; jl += blockDim.x) sy[jl] *= t.d[jl];
    if (KC > 0 && threadIdx.x < kWave) {
        // the clique (every node adjacent to all above it) column by column
        // on the first wavefront, without workgroup barriers; a node per lane
        // in registers, as far as the lanes go, the next column in flight
        const int c0 = S.t_node[2 * kf].w;
        if (KC <= kWave) {
            const int k = threadIdx.x;
            auto column = [&](int q) {
                return k > q && k < KC ? t.wu[clique_slot(c0, KC, q, k)].x : 0.0;
            };
            const double d = k < KC ? t.d[kf + k] : 0.0;
            double z = k < KC ? sy[kf + k] : 0.0, w = column(0);
            for (int q = 0; q < KC; ++q) {
                const double next = column(q + 1);
                const double yq = lane_value(d * z, q);
                if (k > q) z = fma(-w, yq, z);
                w = next;
            }
            if (k < KC) sy[kf + k] = d * z;
        } else {
            for (int q = 0; q < KC; ++q) {
                const double yq = t.d[kf + q] * sy[kf + q];
                for (int k = q + 1 + threadIdx.x; k < KC; k += kWave)
                    sy[kf + k] = fma(-t.wu[clique_slot(c0, KC, q, k)].x, yq, sy[kf + k]);
                if (threadIdx.x == 0) sy[kf + q] = yq;
                wave_sync();
            }
        }
    }
    __syncthreads();
}

// Backward substitution of the tail levels in LDS, downward; then each tail x
// goes to x for the levels below.
__device__ __forceinline__ void fd_backward_tail(const DevSym& S, const FdTail& t, double* sy,
                                                 double* x)
{
    const int nT = S.nlev - S.tail_level, KC = S.tail_clique;
    const int kf = S.tail_nodes - KC;
    if (KC > 0) {
        // the clique first, column by column on the first wavefront: once x_q
        // is final, y_k -= u_kq x_q for every clique node k below q; then the
        // clique's terms of every node below it
        if (threadIdx.x < kWave) {
            const int c0 = S.t_node[2 * kf].w;
            if (KC <= kWave) {
                const int k = threadIdx.x;
                auto column = [&](int q) {
                    return k < q ? t.wu[clique_slot(c0, KC, k, q)].y : 0.0;
                };
                double y = k < KC ? sy[kf + k] : 0.0, u = column(KC - 1);
                for (int q = KC - 1; q > 0; --q) {
                    const double next = column(q - 1);
                    const double xq = lane_value(y, q);
                    if (k < q) y = fma(-u, xq, y);
                    u = next;
                }
                if (k < KC) sy[kf + k] = y;
            } else {
                for (int q = KC - 1; q > 0; --q) {
                    const double xq = sy[kf + q];
                    for (int k = threadIdx.x; k < q; k += kWave)
                        sy[kf + k] = fma(-t.wu[clique_slot(c0, KC, k, q)].y, xq, sy[kf + k]);
                    wave_sync();
                }
            }
        }
        __syncthreads();
        for (int jl = threadIdx.x; jl < kf; jl += blockDim.x) {
            const int t0 = S.t_node[2 * jl].w, t1 = S.t_node[2 * jl + 1].x;
            double y = sy[jl];
            bool more = true;
            for (int q = t1 - 1; more && q >= t0; q -= 4) {  // the clique's are the last ones
                int kk[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) kk[i] = S.t_slot[q - i >= t0 ? q - i : t0].y;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    more = more && q - i >= t0 && kk[i] >= kf;
                    if (more) y = fma(-t.wu[q - i].y, sy[kk[i]], y);
                }
            }
            sy[jl] = y;
        }
        __syncthreads();
    }
    for_tail_ops<false, false>(S, nT - KC, [&](const uint2& q) {
        const TailOp o = tail_op(q);
        sy[o.d] = fma(-t.wu[o.a].y, sy[o.b], sy[o.d]);
    }, [](int, int) {});
    __syncthreads();
    for (int jl = threadIdx.x; jl < S.tail_nodes; jl += blockDim.x)
        x[S.t_node[2 * jl].x] = sy[jl];
    __syncthreads();
}

// Backward substitution x_j = y_j - sum_{k in S(j)} u_jk x_k, levels
// downward; four slots per lane per batch with the next batch's indices in
// flight.
__device__ __forceinline__ void fd_backward(const DevSym& S, const double* m, double* x, int l1)
{
    const double2* sl = reinterpret_cast<const double2*>(m + S.fd_lu);
    for_nodes(S, 0, l1, false, [&](int, const NodeRec& rec, int lane, int g) {
        const int s1 = rec.b.y;
        const double yj = x[rec.a.x];
        // absent entries are not loaded (skipped when no lane needs them)
        int s = rec.b.x + lane;
        int kk[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            kk[k] = 0;
            if (s + k * g < s1) kk[k] = S.Li[s + k * g];
        }
        double a = 0.0;
        for (; s < s1; s += 4 * g) {
            double u[4], xk[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                u[k] = 0.0;
                xk[k] = 0.0;
                if (s + k * g < s1) {
                    u[k] = sl[s + k * g].y;
                    xk[k] = x[kk[k]];
                }
            }
            const int sn = s + 4 * g;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (sn + k * g < s1) kk[k] = S.Li[sn + k * g];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (s + k * g < s1) a = fma(u[k], xk[k], a);
        }
        if (g > 1) a = gsum(a, g);
        if (lane == 0) x[rec.a.x] = yj - a;
    });
}

// What k_fdpf keeps in LDS besides the PV mask and the tails: nothing (FD_NONE,
// both matrices' tails), (e, f) per bus over the tail of one matrix at a time,
// which is loaded after each mismatch pass (FD_OVER), and in it too the work
// vector x of a half step (FD_OVER_X), or everything apart (FD_APART).
enum { FD_NONE, FD_OVER, FD_OVER_X, FD_APART };

// Offsets in doubles into the dynamic LDS (the PV mask at 0): (w, u) and 1/d
// of the two matrices' tails, the tail's y, x by position and (e, f) per bus.
struct FdLds {
    int32_t mode, wu1, d1, wu2, d2, y, x, ef;
};

// The fast decoupled iteration of one case (one workgroup): mismatch, angle
// half step with B', mismatch, magnitude half step with B'', until max|F| <
// tol; iters counts angle half steps and max_iter bounds them.
// Latency bounds it: a chain of some 60 barrier-separated steps per half step
// (levels, tail, mismatch) on one workgroup, so registers are held to what two
// workgroups per compute unit leave (128; with 156 a batch of 384 took two
// rounds), x and (e, f) are in LDS where they fit, and the sine is taken once
// per angle half step, in bus order.  Before -> after: 10,000 buses x 256
// cases 5.52 -> 3.40 ms, 2,000 buses x 384 outages 2.65 -> 1.58 ms (the whole
// screen), 3,001 buses alone 1.21 -> 0.97 ms.
template <int MODE>
__device__ void fdpf_case(const DevSym& S, const FdLds& L, const double* yv, const int8_t* type,
                          const double* Psp, const double* Qsp, double* Vm, double* Va,
                          double* ws, const double* m1, const double* m2, double tol,
                          int max_iter, int32_t* o_iters, double* o_norm, int32_t* o_status)
{
    uint32_t* fd_pv = reinterpret_cast<uint32_t*>(pf_smem);
    const FdTail t1{reinterpret_cast<double2*>(pf_smem + L.wu1), pf_smem + L.d1};
    const FdTail t2{reinterpret_cast<double2*>(pf_smem + L.wu2), pf_smem + L.d2};
    double* sy = pf_smem + L.y;
    const EFLds efs{reinterpret_cast<double2*>(pf_smem + L.ef)};
    constexpr bool efl = MODE != FD_NONE, shared = MODE == FD_OVER || MODE == FD_OVER_X;
    const bool tail = S.tail_nodes > 0;
    const int lg = tail ? S.tail_level : S.nlev;  // levels swept in global memory
    // workspace: (cos, sin) | (e, f) | b | x
    const FdState st{Vm, Va, reinterpret_cast<double2*>(ws),
                     reinterpret_cast<double2*>(ws) + S.n};
    double* const b = ws + 4 * (int64_t)S.n;
    double* const x = MODE >= FD_OVER_X ? pf_smem + L.x : b + S.nn;
    const EFLds efg{st.ef};
    if (tail && !shared) {
        fd_tail_load(S, m1, t1);
        fd_tail_load(S, m2, t2);
    }
    auto put_ef = [&](int i, double2 v) {
        if (!efl) st.ef[i] = v;
        else if (!shared) efs.s[i] = v;
    };
    for (int i = threadIdx.x; i < S.n; i += blockDim.x) {
        double sn, cs;
        const double vm = Vm[i], va = Va[i];
        sincos(va, &sn, &cs);
        st.cs[i] = make_double2(cs, sn);
        put_ef(i, make_double2(vm * cs, vm * sn));
    }
    pv_fill_at(fd_pv, S, type);
    __syncthreads();
    const PvMask pvm{fd_pv};
    int it = 0, half = 0, status = ST_NOT_CONVERGED;
    double nrm = 0.0;
    for (;;) {
        double mx = 0.0;
        int nan = 0;
        const MisHalf out{Vm, b, half != 0};
        if (shared) {
            // each thread's own buses of the half step (or of the start)
            for (int i = fresh_thread(); i < S.n; i += wg_size()) {
                const double2 cs = st.cs[i];
                const double vm = Vm[i];
                efs.s[i] = make_double2(vm * cs.x, vm * cs.y);
            }
            __syncthreads();
        }
        mismatch_pass<2>(S, yv, efl ? efs : efg, out, pvm, Psp, Qsp, mx, nan, fresh_thread(),
                         wg_size());
        int any_nan = 0;
        nrm = block_max(mx, nan, any_nan);
        if (any_nan || !isfinite(nrm)) {
            status = ST_NONFINITE;
            break;
        }
        if (nrm < tol) {
            status = ST_OK;
            break;
        }
        if (half == 0 && it >= max_iter) break;
        if (shared && tail) {
            fd_tail_load(S, half == 0 ? m1 : m2, t1);
            __syncthreads();
        }
        const double* m = half == 0 ? m1 : m2;
        const FdTail& t = half == 0 || shared ? t1 : t2;
        fd_forward(S, m, b, x, lg);
        if (tail) {
            fd_forward_tail(S, m, t, sy, b, x);
            fd_backward_tail(S, t, sy, x);
        }
        fd_backward(S, m, x, lg);
        if (half == 0) {
            fd_half_step<true>(S, st, pvm, x, put_ef);
            ++it;
        } else {
            fd_half_step<false>(S, st, pvm, x, put_ef);
        }
        __syncthreads();
        half ^= 1;
    }
    if (threadIdx.x == 0) {
        if (o_iters) *o_iters = it;
        if (o_norm) *o_norm = nrm;
        if (o_status) *o_status = status;
    }
}

}  // namespace


// Fast decoupled matrices of B cases: B' then B'' (fd_mat doubles each) in
// the scalar filled layout, lower and upper values equal.  A thread per
// diagonal entry, then one per slot: the chain of loads from the slot to its
// branches bounds it (a thread per node, slot after slot: 2,000 buses x 384
// cases 116 us, now 61).
__global__ void k_fd_matrices(DevSym S, int B, int per_case, int slots,
                              const double* __restrict__ r, const double* __restrict__ x,
                              const double* __restrict__ b,
                              int64_t bstride, const double* __restrict__ ysh,
                              int64_t sh_stride, const int8_t* __restrict__ type,
                              int64_t type_stride, double* __restrict__ mat, int64_t mstride)
{
    const int2 at = item_block(per_case, B);
    const int c = at.x, p = at.y + threadIdx.x;
    const int s = p - S.fd_lu;
    if (c < 0 || s >= slots) return;
    const bool diag = s < 0, pad = diag && p >= S.nn;  // padding of the d sections
    int q = -1, bj = 0, bk = 0;
    if (!diag) {
        const int4 a = S.slot_info[2 * s];
        q = a.z;
        bk = a.y;
        bj = S.slot_info[2 * s + 1].w;
    } else if (!pad) {
        q = S.ydiag[p];
        bj = S.perm[p];
    }
    const int t0 = q < 0 ? 0 : S.ybr_ptr[q], t1 = q < 0 ? 0 : S.ybr_ptr[q + 1];
    const int e0 = t0 < t1 ? S.ybr[t0] : 0;
    const double* rc = r + c * bstride;
    const double* xc = x + c * bstride;
    const double* bc = b + c * bstride;
    const int8_t* tc = type + c * type_stride;
    double* m1 = mat + c * mstride;
    double* m2 = m1 + S.fd_mat;
    const double2 v = fd_entries(S, t0, t1, e0, diag, rc, xc, bc);
    const bool pvj = tc[bj] == T_PV;
    if (diag) {
        // B'' = -Im(Y): the bus shunt's susceptance comes off the diagonal
        const double bsh = ysh && !pad ? ysh[c * sh_stride + 2 * (int64_t)bj + 1] : 0.0;
        m1[p] = pad ? 0.0 : v.x;
        m2[p] = pad ? 0.0 : pvj ? 1.0 : v.y - bsh;
    } else {
        const double w2 = pvj || tc[bk] == T_PV ? 0.0 : v.y;
        reinterpret_cast<double2*>(m1 + S.fd_lu)[s] = make_double2(v.x, v.x);
        reinterpret_cast<double2*>(m2 + S.fd_lu)[s] = make_double2(w2, w2);
    }
}

// In-place LDL^T of B' and B'' of case blockIdx.x, level by level.
// Two workgroups per case, one per matrix (B' and B'' are independent).  The
// status is set to OK by k_fill_status beforehand; a workgroup that meets a
// zero pivot stores ST_ZERO_PIVOT (both may, with the same value).
__global__ __launch_bounds__(kLevelThreads) void k_fd_factor(DevSym S, double* mat,
                                                             int64_t mstride, int32_t* status)
{
    __shared__ int s_bad;
    const int c = blockIdx.x >> 1, which = blockIdx.x & 1;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    double* m = mat + c * mstride + which * S.fd_mat;
    for_nodes(S, 0, S.nlev, true, [&](int, const NodeRec& rec, int lane, int g) {
        fd_factor_node(S, rec, lane, g, m, &s_bad);
    });
    __syncthreads();
    if (threadIdx.x == 0 && status && s_bad) status[c] = ST_ZERO_PIVOT;
}

__global__ void k_fill_status(int B, int32_t* status, int32_t v)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < B) status[c] = v;
}

template <int MODE>
__global__ __launch_bounds__(kLevelThreads, 4) void k_fdpf(DevSym S, FdLds L, NewtonArgs a,
                                                           const double* mat, int64_t mstride)
{
    const int c = blockIdx.x;
    const double* m1 = mat + c * mstride;
    fdpf_case<MODE>(S, L, a.yval + c * a.y_stride, a.type + c * a.type_stride,
                    a.Psp + c * a.inj_stride, a.Qsp + c * a.inj_stride, a.Vm + c * a.v_stride,
                    a.Va + c * a.v_stride, a.ws + c * a.ws_stride, m1, m1 + S.fd_mat, a.tol,
                    a.max_iter, a.iters ? a.iters + c : nullptr, a.norm ? a.norm + c : nullptr,
                    a.status ? a.status + c : nullptr);
}

// Branch flows (Sec. II-A: post-convergence, edge by edge): pi-model with
// series y = g + jb' = 1/(r + jx) and charging b,
//   S_ft = V_f conj((y + jb/2) V_f - y V_t)
//        = |V_f|^2 (g - j(b' + b/2)) - |V_f||V_t| e^{j d} (g - jb'),
// d = theta_f - theta_t, and the same from the other end with -d: one sine for
// both ends.  The outputs are not read here: stored past the caches, which
// leaves the voltages of a batch called again there.  The gathered voltages
// bound it, not the sines (one or two: the same 119 us at 10,000 buses x 512
// cases; several cases per thread: 141 and more): with a case's workgroups on
// one XCD 81 us; 63 us for the bytes.  Whole calls back to back: the same batch
// 146 -> 104 us, six batches in turn, none of whose voltages stay in the
// caches, 181 -> 133.
__global__ void k_branch_flows(int m, int B, int per_case, const int32_t* __restrict__ from,
                               const int32_t* __restrict__ to, const double* __restrict__ r,
                               const double* __restrict__ x, const double* __restrict__ b,
                               int64_t bstride, const double* __restrict__ Vm,
                               const double* __restrict__ Va, int64_t vstride, double* Pft,
                               double* Qft, double* Ptf, double* Qtf, int64_t ostride)
{
    const int2 at = item_block(per_case, B);
    const int c = at.x, e = at.y + threadIdx.x;
    if (c < 0 || e >= m) return;
    const int fb = from[e], tb = to[e];
    const double rr = r[c * bstride + e], xx = x[c * bstride + e], hb = b[c * bstride + e] / 2.0;
    const double* vm = Vm + c * vstride;
    const double* va = Va + c * vstride;
    const double vf = vm[fb], vt = vm[tb];
    double sn, cs;
    sincos(va[fb] - va[tb], &sn, &cs);
    const double den = rr * rr + xx * xx;
    const double g = rr / den, yb = -xx / den, bs = yb + hb;
    const double ff = vf * vf, tt = vt * vt, ft = vf * vt;
    const double gc = g * cs, gs = g * sn, bc = yb * cs, bn = yb * sn;
    const int64_t o = c * ostride + e;
    __builtin_nontemporal_store(ff * g - ft * (gc + bn), &Pft[o]);
    __builtin_nontemporal_store(-ff * bs - ft * (gs - bc), &Qft[o]);
    __builtin_nontemporal_store(tt * g - ft * (gc - bn), &Ptf[o]);
    __builtin_nontemporal_store(-tt * bs + ft * (gs + bc), &Qtf[o]);
}


namespace {

using FdKernel = void (*)(DevSym, FdLds, NewtonArgs, const double*, int64_t);
constexpr FdKernel kFdKernels[] = {&k_fdpf<FD_NONE>, &k_fdpf<FD_OVER>, &k_fdpf<FD_OVER_X>,
                                   &k_fdpf<FD_APART>};

// What the current device offers a launch: the dynamic LDS that any of the
// fast decoupled kernels may ask for, and its compute units.
struct FdDevice {
    int64_t dyn;
    int cus;
};
FdDevice fd_device()
{
    FdDevice d{lds_limit(kFdKernels[0]), compute_units()};
    for (FdKernel k : kFdKernels) d.dyn = std::min(d.dyn, lds_limit(k));
    return d;
}

// LDS of B cases (bytes into *bytes).  Everything apart, if the device can
// keep as many of the launch's workgroups resident as with less LDS (and it
// fits a budget that the caller set below the default, to leave room for
// other launches' workgroups); else (e, f) over the rest as far as the
// caller's budget has room for it; else (e, f) in the workspace.
FdLds fd_lds(const HostSym& h, int B, int threads, const FdDevice& dev, size_t* bytes)
{
    const int64_t mask = (((int64_t)pv_mask_bytes(h.n) + 15) / 16) * 2;
    const int64_t TS = h.tail_slots, K = h.tail_nodes, n = h.n, nn = h.nn;
    const int64_t K2 = (K + 1) & ~(int64_t)1, nn2 = (nn + 1) & ~(int64_t)1;
    const int64_t tails = 4 * TS + 3 * K2;  // both matrices' (w, u) | 1/d | 1/d | y
    const int64_t apart = mask + tails + nn2 + 2 * n;
    const int64_t less = mask + (h.ef_lds ? std::max((int64_t)h.ef_lds / 8, 2 * (TS + K)) : tails);
    // workgroups a compute unit gets, of those its registers have room for
    const int64_t want = std::min(((int64_t)B + dev.cus - 1) / dev.cus,
                                  std::max((int64_t)1, (int64_t)2 * kLevelThreads / threads));
    auto resident = [&](int64_t doubles) { return std::min(want, dev.dyn / (8 * doubles + 512)); };
    const bool fits =
        h.tail_budget >= kDefaultTailBudget || 8 * (apart - mask) <= h.tail_budget;
    const bool all = fits && resident(apart) > 0 && resident(apart) >= resident(less);
    FdLds L;
    L.wu1 = L.x = L.ef = (int32_t)mask;
    if (all || !h.ef_lds) {
        L.mode = all ? FD_APART : FD_NONE;
        L.wu2 = (int32_t)(mask + 2 * TS);
        L.d1 = (int32_t)(mask + 4 * TS);
        L.d2 = (int32_t)(L.d1 + K2);
        L.y = (int32_t)(L.d2 + K2);
        if (all) {
            L.x = (int32_t)(mask + tails);
            L.ef = (int32_t)(mask + tails + nn2);
        }
    } else {
        // x after one matrix's tail, within the (e, f) copy
        const bool in = 8 * (2 * (TS + K) + nn) <= h.ef_lds;
        L.mode = in ? FD_OVER_X : FD_OVER;
        L.wu2 = L.wu1;
        L.d1 = L.d2 = (int32_t)(mask + 2 * TS);
        L.y = (int32_t)(L.d1 + K);
        if (in) L.x = (int32_t)(L.y + K);
    }
    *bytes = 8 * (size_t)(all ? apart : less);
    return L;
}

}  // namespace

extern "C" {
int pf_fdpf_matrices(const pf_symbolic s, int B, const double* d_r, const double* d_x,
                     const double* d_b, int64_t branch_stride, const double* d_ysh,
                     int64_t ysh_stride, const int8_t* d_type, int64_t type_stride,
                     double* d_mat, int64_t mat_stride, void* stream)
{
    if (!ready(s, "pf_fdpf_matrices")) return PF_E_INVALID;
    if (B < 0 || B > 65535 || !d_r || !d_x || !d_b || !d_type || !d_mat || (mat_stride & 7) ||
        branch_stride < 0 || ysh_stride < 0)
        return fail(PF_E_INVALID, "pf_fdpf_matrices: bad arguments");
    if (d_ysh && (ysh_stride & 1 || (B > 1 && ysh_stride != 0 && ysh_stride < 2 * s->h.n)))
        return fail(PF_E_INVALID, "pf_fdpf_matrices: ysh_stride must be 0 or even and >= 2*n");
    if (reinterpret_cast<uintptr_t>(d_mat) & 15)
        return fail(PF_E_WORKSPACE, "pf_fdpf_matrices: d_mat must be 16-byte aligned");
    if (B > 1 && mat_stride < 2 * s->h.fd_mat())
        return fail(PF_E_WORKSPACE, "pf_fdpf_matrices: mat_stride < fd_mat_doubles");
    if (!shared_stride_ok(B, branch_stride, s->h.m) || !shared_stride_ok(B, type_stride, s->h.n))
        return fail(PF_E_WORKSPACE, "pf_fdpf_matrices: a stride is too small or negative");
    if (B == 0) return PF_OK;
    const int64_t slots = (int64_t)s->h.Li.size();
    int per_case = 0;
    const dim3 grid = item_grid(s->h.fd_lu() + slots, B, &per_case);
    hipLaunchKernelGGL(k_fd_matrices, grid, dim3(256), 0, as_stream(stream), s->h.dev, B, per_case,
                       (int)slots, d_r, d_x, d_b, branch_stride, d_ysh, ysh_stride, d_type,
                       type_stride, d_mat, mat_stride);
    return launch_check("pf_fdpf_matrices");
}

int pf_fdpf_factor(const pf_symbolic s, int B, double* d_mat, int64_t mat_stride,
                   int32_t* d_status, void* stream)
{
    if (!ready(s, "pf_fdpf_factor")) return PF_E_INVALID;
    if (B < 0 || !d_mat || (mat_stride & 7))
        return fail(PF_E_INVALID, "pf_fdpf_factor: bad arguments");
    if (reinterpret_cast<uintptr_t>(d_mat) & 15)
        return fail(PF_E_WORKSPACE, "pf_fdpf_factor: d_mat must be 16-byte aligned");
    if (B > 1 && mat_stride < 2 * s->h.fd_mat())
        return fail(PF_E_WORKSPACE, "pf_fdpf_factor: mat_stride < fd_mat_doubles");
    if (B == 0) return PF_OK;
    if (d_status)
        hipLaunchKernelGGL(k_fill_status, dim3((B + 255) / 256), dim3(256), 0, as_stream(stream),
                           B, d_status, (int32_t)ST_OK);
    hipLaunchKernelGGL(k_fd_factor, dim3(2 * B), dim3(launch_threads(s->h, B)), 0,
                       as_stream(stream), s->h.dev, d_mat, mat_stride, d_status);
    return launch_check("pf_fdpf_factor");
}

int pf_fdpf(const pf_symbolic s, int B, const double* d_yval, int64_t y_stride,
            const int8_t* d_type, int64_t type_stride, const double* d_Psp, const double* d_Qsp,
            int64_t inj_stride, double* d_Vm, double* d_Va, int64_t v_stride,
            const double* d_mat, int64_t mat_stride, double tol, int max_iter, double* d_ws,
            int64_t ws_stride, int32_t* d_iters, double* d_norm, int32_t* d_status,
            void* stream)
{
    if (!ready(s, "pf_fdpf")) return PF_E_INVALID;
    if (B < 0 || max_iter < 0 || !(tol >= 0.0) || !d_yval || !d_type || !d_Psp || !d_Qsp ||
        !d_Vm || !d_Va || !d_mat || !d_ws || (mat_stride & 7))
        return fail(PF_E_INVALID, "pf_fdpf: bad arguments");
    if (B > 1 && v_stride < s->h.n) return fail(PF_E_WORKSPACE, "pf_fdpf: v_stride too small");
    if (!shared_stride_ok(B, y_stride, 2 * (int64_t)s->h.ycol.size()) ||
        !shared_stride_ok(B, type_stride, s->h.n) || !shared_stride_ok(B, inj_stride, s->h.n) ||
        !shared_stride_ok(B, mat_stride, 2 * s->h.fd_mat()))
        return fail(PF_E_WORKSPACE, "pf_fdpf: a stride is too small or negative");
    if (ws_stride < s->h.fd_ws_doubles() || (ws_stride & 7))
        return fail(PF_E_WORKSPACE,
                    "pf_fdpf: ws_stride must be >= fd_ws_doubles, a multiple of 8");
    if ((reinterpret_cast<uintptr_t>(d_ws) & 15) || (reinterpret_cast<uintptr_t>(d_mat) & 15))
        return fail(PF_E_WORKSPACE, "pf_fdpf: d_ws and d_mat must be 16-byte aligned");
    if (B == 0) return PF_OK;
    NewtonArgs a{d_yval, y_stride, d_type, type_stride, d_Psp, d_Qsp, inj_stride, d_Vm, d_Va,
                 v_stride, d_ws, ws_stride, tol, max_iter, 0, 1, B, d_iters, d_norm, d_status};
    size_t lds = 0;
    const int threads = launch_threads(s->h, B);
    const FdLds L = fd_lds(s->h, B, threads, fd_device(), &lds);
    hipLaunchKernelGGL(kFdKernels[L.mode], dim3(B), dim3(threads), lds, as_stream(stream),
                       s->h.dev, L, a, d_mat, mat_stride);
    return launch_check("pf_fdpf");
}

int pf_branch_flows(const pf_symbolic s, int B, const double* d_r, const double* d_x,
                    const double* d_b, int64_t branch_stride, const double* d_Vm,
                    const double* d_Va, int64_t v_stride, double* d_Pft, double* d_Qft,
                    double* d_Ptf, double* d_Qtf, int64_t out_stride, void* stream)
{
    if (!ready(s, "pf_branch_flows")) return PF_E_INVALID;
    if (B < 0 || B > 65535 || !d_r || !d_x || !d_b || !d_Vm || !d_Va || !d_Pft || !d_Qft ||
        !d_Ptf || !d_Qtf)
        return fail(PF_E_INVALID, "pf_branch_flows: bad arguments");
    if (B > 1 && (v_stride < s->h.n || out_stride < s->h.m))
        return fail(PF_E_WORKSPACE, "pf_branch_flows: stride too small");
    if (!shared_stride_ok(B, branch_stride, s->h.m))
        return fail(PF_E_WORKSPACE, "pf_branch_flows: branch_stride too small or negative");
    if (B == 0 || s->h.m == 0) return PF_OK;
    int per_case = 0;
    const dim3 grid = item_grid(s->h.m, B, &per_case);
    hipLaunchKernelGGL(k_branch_flows, grid, dim3(256), 0, as_stream(stream), s->h.m, B, per_case,
                       s->d_from,
                       s->d_to, d_r, d_x, d_b, branch_stride, d_Vm, d_Va, v_stride, d_Pft, d_Qft,
                       d_Ptf, d_Qtf, out_stride);
    return launch_check("pf_branch_flows");
}

}  // extern "C"
