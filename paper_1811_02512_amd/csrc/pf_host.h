// libpf host-side internals shared by the C ABI files: the symbolic handle and
// the argument / error / launch-shape helpers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "pf.h"
#include "pf_internal.h"

struct pf_symbolic_s {
    pf::HostSym h;
    const int32_t* d_from = nullptr;  // device copies of the branch ends
    const int32_t* d_to = nullptr;
};

namespace pf {
namespace abi {

// Thread-local message of the last failed call (pf_last_error).
extern thread_local std::string g_err;

// Records msg as the thread's last error and returns code.
int fail(int code, const std::string& msg);
int hip_check(hipError_t e, const char* what);
int launch_check(const char* what);
// The current device: compute units (1 if unknown) and the dynamic LDS a launch
// of `kernel` may ask for there, raised at the first question to what the
// device has beside the kernel's static LDS; the default limit where that is
// refused.  Kept per device and kernel, safe from several threads; errors of
// the queries are cleared, so that no launch check reports them.
int compute_units();
int64_t lds_limit(const void* kernel);
template <class K>
int64_t lds_limit(K* kernel)
{
    return lds_limit(reinterpret_cast<const void*>(kernel));
}
// Workgroup size of the level-scheduled kernels: the symbolic's setting, or
// by batch size.
int launch_threads(const pf::HostSym& h, int B);
// Grid of a per-item kernel (an item: a bus, a branch, a slot; 256 threads per
// workgroup) over B cases, and the workgroups per case it hands to the kernel
// (item_block): one dimension, a case on one XCD, from eight cases on where
// three quarters of the XCDs' turns are taken.  Below that the last turn's
// idle XCDs cost more than the shared fetches save.  Admittances, Jacobian and
// fast decoupled matrices of 10,000 buses (us), so / two-dimensional: 6 cases
// 16, 17, 11 / 15, 16, 10; 9 cases 22, 25, 17 / 18, 22, 15; 12 cases 23, 26, 17 /
// 23, 27, 19; 14 cases 23, 26, 18 / 26, 30, 21; 18 cases 28, 34, 26 / 30, 36,
// 27; 33 cases 38, 51, 38 / 46, 57, 50.
inline dim3 item_grid(int64_t items, int B, int* per_case)
{
    const int64_t nb = (items + 255) / 256, full = ((int64_t)B + 7) / 8 * 8, lin = nb * full;
    // (under 2^32 threads)
    const bool xcd = B >= 8 && 3 * full <= 4 * (int64_t)B && lin < (int64_t)1 << 23;
    *per_case = xcd ? (int)nb : 0;
    return xcd ? dim3((unsigned)lin) : dim3((unsigned)nb, B);
}
// Builds the upper levels' lists for the next upload, whole where a launch is
// to spread the grid (what is on the device stays as it is).
int upper_lists(pf::HostSym& h, bool whole, const char* fn);
// Blocks for B cases in groups of C placed one XCD round apart.
int grid_blocks(int B, int C);
bool valid_interleave(int C);
// Interleave pf_newton uses for B cases.
int newton_interleave(const pf::HostSym& h, int B);
// A symbolic that is non-null and uploaded (else records the error).
bool ready(const pf_symbolic s, const char* fn);
inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }
// A per-case stride of an input that the cases may also share: 0 (one array
// for all cases) or, with more than one case, at least one row.
inline bool shared_stride_ok(int B, int64_t stride, int64_t row)
{
    return stride >= 0 && (stride == 0 || B <= 1 || stride >= row);
}
// Branch gradients (and, with bus, the injection gradients) of B cases from
// their adjoint vectors (pf_adjoint_params, pf_adjoint).
int adjoint_branch_launch(const pf_symbolic s, int B, const double* d_lam, int64_t lam_stride,
                          const int8_t* d_type, int64_t type_stride, const double* d_Vm,
                          const double* d_Va, int64_t v_stride, const double* d_r,
                          const double* d_x, int64_t branch_stride, const int32_t* d_status,
                          double* d_gP, double* d_gQ, int64_t g_stride, double* d_gx,
                          int gx_mode, void* stream, bool bus);
// The level-scheduled factorisation of B matrices (sym: symmetric ones).
void factor_launch(const pf::HostSym& h, int B, double* vals, int64_t stride, int C,
                   int32_t* status, int32_t* pivot, hipStream_t st, bool sym);

}  // namespace abi
}  // namespace pf
