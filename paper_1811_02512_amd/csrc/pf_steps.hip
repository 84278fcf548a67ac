// libpf: the Jacobian and its factorisation as calls of their own (kernels and
// their C ABI entry points), also the state estimator's factorisation.
#include <hip/hip_runtime.h>

#include "pf.h"
#include "pf_device.h"
#include "pf_host.h"

using namespace pf::abi;

namespace {

// Jacobian assembly straight from polar voltages (standalone kernel).
struct AsmPolar {
    const DevSym* S;
    const double* yv;
    const int8_t* type;
    const double* Vm;
    EFPolar ef;
    __device__ __forceinline__ Blk diag(int j) const
    {
        const int bus = S->perm[j];
        const double2 y = reinterpret_cast<const double2*>(yv)[S->ydiag[j]];
        double p, q;
        injection(*S, yv, ef, bus, p, q);
        return jac_diag(y.x, y.y, p, q, Vm[bus], type[bus] == T_PV);
    }
    __device__ __forceinline__ void off(int s, Blk& lo, Blk& up) const
    {
        const int4 a = S->slot_info[2 * s], b = S->slot_info[2 * s + 1];
        const int ylo = a.z;
        if (ylo < 0) {
            lo = bzero();
            up = bzero();
            return;
        }
        const int bj = b.w, bk = a.y;
        double ej, fj, ek, fk;
        ef.get(bj, ej, fj);
        ef.get(bk, ek, fk);
        const bool pj = type[bj] == T_PV, pk = type[bk] == T_PV;
        const double2 yl = reinterpret_cast<const double2*>(yv)[ylo];
        const double2 yu = reinterpret_cast<const double2*>(yv)[a.w];
        lo = jac_off(yl.x, yl.y, ek, fk, ej, fj, Vm[bj], pk, pj);
        up = jac_off(yu.x, yu.y, ej, fj, ek, fk, Vm[bk], pj, pk);
    }
};

}  // namespace

// Jacobian blocks of one case (item_block): a thread per diagonal block, then
// one per slot, so that a case's sines and chains of loads run side by side
// (with a node's slots in one thread, 5,003 buses x 48 cases took 44 us, now
// 36).  The diagonal section's padding is zeroed.
__global__ void k_jacobian(DevSym S, const double* yval, int64_t y_stride, const int8_t* type,
                           int64_t type_stride, const double* Vm, const double* Va,
                           int64_t v_stride, double* vals, int64_t vals_stride, int C, int slots,
                           int B, int per_case)
{
    const int2 at = item_block(per_case, B);
    const int t = at.y + threadIdx.x;
    const int c = at.x;
    if (c < 0) return;
    const EFPolar ef{Vm + c * v_stride, Va + c * v_stride};
    const AsmPolar A{&S, yval + c * y_stride, type + c * type_stride, Vm + c * v_stride, ef};
    const View w = case_view(vals, vals_stride, C, c);
    const int64_t lu = S.lu_off;
    if (t < S.nn) {
        w.put(4 * (int64_t)t, A.diag(t));
    } else if (t - S.nn < slots) {
        const int s = t - S.nn;
        Blk lo, up;
        A.off(s, lo, up);
        w.put(lu + 8 * (int64_t)s, lo);
        w.put(lu + 8 * (int64_t)s + 4, up);
    } else if (t - S.nn - slots < lu / 4 - S.nn) {
        w.put(4 * (int64_t)(t - slots), bzero());
    }
}

// SYM: a symmetric matrix; the levels below the LDS tail update the lower
// blocks only (the tail runs the general LDU, exact for it too).
template <bool SYM>
__global__ __launch_bounds__(kLevelThreads) void k_factor(DevSym S, double* vals,
                                                        int64_t vals_stride, int C, int B,
                                                        int32_t* status, int32_t* pivot)
{
    __shared__ int s_bad;
    const int c = case_of_block(blockIdx.x, C, B);
    if (c < 0) return;
    const View w = case_view(vals, vals_stride, C, c);
    const int64_t lu = S.lu_off;
    if (threadIdx.x == 0) s_bad = kNoPivot;
    __syncthreads();
    const SrcLoadT<SYM> src{w, lu};
    for_nodes(S, 0, S.tail_level, true, [&](int x, const NodeRec& r, int lane, int g) {
        factor_node<SrcLoadT<SYM>, false, true, SYM>(S, src, x, r, lane, g, w, lu, w, 0, &s_bad);
    });
    if (S.tail_nodes > 0) upper_factor<SrcLoadT<SYM>, false, true>(S, src, w, lu, w, 0, &s_bad);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (status) status[c] = s_bad != kNoPivot ? ST_ZERO_PIVOT : ST_OK;
        if (pivot) pivot[c] = s_bad == kNoPivot ? -1 : S.level_nodes[s_bad];
    }
}

namespace pf {
namespace abi {

// The level-scheduled factorisation of B matrices (sym: symmetric ones).
void factor_launch(const HostSym& h, int B, double* vals, int64_t stride, int C,
                   int32_t* status, int32_t* pivot, hipStream_t st, bool sym)
{
    (void)lds_limit(sym ? &k_factor<true> : &k_factor<false>);
    if (sym)
        hipLaunchKernelGGL(k_factor<true>, dim3(grid_blocks(B, C)), dim3(launch_threads(h, B)),
                           h.tail_lds, st, h.dev, vals, stride, C, B, status, pivot);
    else
        hipLaunchKernelGGL(k_factor<false>, dim3(grid_blocks(B, C)), dim3(launch_threads(h, B)),
                           h.tail_lds, st, h.dev, vals, stride, C, B, status, pivot);
}

}  // namespace abi
}  // namespace pf

extern "C" {
int pf_jacobian(const pf_symbolic s, int B, const double* d_yval, int64_t y_stride,
                const int8_t* d_type, int64_t type_stride, const double* d_Vm, const double* d_Va,
                int64_t v_stride, double* d_vals, int64_t vals_stride, int vals_interleave,
                void* stream)
{
    if (!ready(s, "pf_jacobian")) return PF_E_INVALID;
    if (B < 0 || B > 65535 || !d_yval || !d_type || !d_Vm || !d_Va || !d_vals ||
        !valid_interleave(vals_interleave) || (vals_stride & 7))
        return fail(PF_E_INVALID, "pf_jacobian: bad arguments");
    if (B > 1 && vals_stride < s->h.vals_doubles())
        return fail(PF_E_WORKSPACE, "pf_jacobian: vals_stride < vals_doubles");
    if (!shared_stride_ok(B, y_stride, 2 * (int64_t)s->h.ycol.size()) ||
        !shared_stride_ok(B, type_stride, s->h.n) || v_stride < 0 ||
        (B > 1 && v_stride < s->h.n))
        return fail(PF_E_WORKSPACE, "pf_jacobian: a stride is too small or negative");
    if (B == 0 || s->h.nn == 0) return PF_OK;
    const int64_t slots = (int64_t)s->h.Li.size();
    int per_case = 0;
    const dim3 grid = item_grid(s->h.lu_off() / 4 + slots, B, &per_case);
    hipLaunchKernelGGL(k_jacobian, grid, dim3(256), 0, as_stream(stream), s->h.dev, d_yval,
                       y_stride, d_type, type_stride, d_Vm, d_Va, v_stride, d_vals, vals_stride,
                       vals_interleave, (int)slots, B, per_case);
    return launch_check("pf_jacobian");
}

int pf_factor(const pf_symbolic s, int B, double* d_vals, int64_t vals_stride,
              int vals_interleave, int32_t* d_status, int32_t* d_pivot, void* stream)
{
    if (!ready(s, "pf_factor")) return PF_E_INVALID;
    if (B < 0 || !d_vals || !valid_interleave(vals_interleave) || (vals_stride & 7))
        return fail(PF_E_INVALID, "pf_factor: bad arguments");
    if (B > 1 && vals_stride < s->h.vals_doubles())
        return fail(PF_E_WORKSPACE, "pf_factor: vals_stride < vals_doubles");
    if (B == 0) return PF_OK;
    factor_launch(s->h, B, d_vals, vals_stride, vals_interleave, d_status, d_pivot,
                  as_stream(stream), false);
    return launch_check("pf_factor");
}

}  // extern "C"
