// S3: mask = |v| > tau, ascending index list and its length (Alg. 1 line 3; S_t of Eq. 5 with the strict
// comparison Alg. 1 uses).  One workgroup of 16 waves per task.  Each wave owns a contiguous slice of
// the channels: pass 1 keeps and counts wave ballots, an LDS prefix over the 16 wave totals gives every
// wave its base offset, pass 2 writes each selected channel at base + (selected channels before it), which keeps
// the list ascending without any sort.
#include "floe_dev.h"
#include "launch.h"
#include "select_task.h"

namespace floe {

__global__ __launch_bounds__(1024) void select_kernel(const float* __restrict__ v, int f, const float* __restrict__ tau,
                                                      int32_t* __restrict__ idx, int32_t* __restrict__ count, int pad) {
    const int task = blockIdx.x;
    select_task(v + (size_t)task * f, f, tau[task], idx + (size_t)task * f, count + task, pad != 0);
}

hipError_t launch_select(const float* v, int f, int n_tasks, const float* tau, int32_t* idx, int32_t* count,
                         hipStream_t stream, bool pad) {
    if (n_tasks == 0) return hipSuccess;
    select_kernel<<<dim3(n_tasks), dim3(1024), 0, stream>>>(v, f, tau, idx, count, pad);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void pad_list_kernel(int32_t* __restrict__ idx, long long n) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) idx[i] = -1;
}

hipError_t launch_pad_list(int32_t* idx, int f, int n_tasks, hipStream_t stream) {
    const long long n = (long long)n_tasks * f, blocks = (n + 255) / 256;
    if (n == 0) return hipSuccess;
    if (blocks > 0x7fffffffll) return hipErrorInvalidValue;
    pad_list_kernel<<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(idx, n);
    return hipGetLastError();
}

}  // namespace floe
