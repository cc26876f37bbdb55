// eg_batched.hip -- the label pass for a batch of fields.
//
// Every kernel here covers all fields of the batch in one launch: the grid's
// y dimension is the field, x strides over that field's items.  Stage (d)
// of a batch runs the stage (d) kernels with the batch field selector.
#include "eg_internal.h"

namespace eg {

constexpr int kBatchBlocksPerField = 48;

__device__ __forceinline__ uint32_t rd(const uint32_t* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256) void k_binit(const BatchPlan* __restrict__ plan)
{
    const BatchField& F = plan->fields[blockIdx.x];
    const int t = threadIdx.x;
    if (t < C_SLOTS) F.ta.ctr[t] = 0;
    if (t < EG_H_SLOTS) F.arc.header[t] = 0;
    if (blockIdx.x == 0 && t < C_SLOTS) plan->bctr[t] = 0;
}

// ------------------------------------------------------------------ labels

// Both exit-list kernels take four consecutive entries per thread (one 16-byte
// access, four independent gathers or chains in flight), as the single-field
// kernels do: every workspace is 256-byte aligned (eg_batch_plan checks it).
__global__ __launch_bounds__(256) void k_bexit_init(const BatchPlan* __restrict__ plan)
{
    const BatchField F = plan->fields[blockIdx.y];  // a copy: loop loads cannot alias it
    const uint32_t req = rd(&F.ta.ctr[C_NEXIT]);
    const uint32_t n = req < F.ta.cap_exit ? req : F.ta.cap_exit;
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    const int32_t* lab = F.ta.lab;
    const uint32_t nq = n >> 2;
    const uint4* e4 = reinterpret_cast<const uint4*>(F.ta.exits);
    int4* r4 = reinterpret_cast<int4*>(F.exres);
    for (uint32_t q = t; q < nq; q += stride) {
        const uint4 e = e4[q];
        r4[q] = make_int4(lab[e.x], lab[e.y], lab[e.z], lab[e.w]);
    }
    if (t < (n & 3u)) F.exres[(nq << 2) + t] = lab[F.ta.exits[(nq << 2) + t]];
}

__global__ __launch_bounds__(256) void k_bexit_jump(const BatchPlan* __restrict__ plan)
{
    const BatchField F = plan->fields[blockIdx.y];  // a copy: loop loads cannot alias it
    const uint32_t req = rd(&F.ta.ctr[C_NEXIT]);
    const uint32_t n = req < F.ta.cap_exit ? req : F.ta.cap_exit;
    const int hops = plan->tuning.hops;
    const int sweeps = sweeps_for(plan->tuning, F.N);
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    bool open = sweep(F.exres, n, F.ta.lab, F.exres, F.N, hops, t, stride, false);
    for (int k = 1; __ballot(open) != 0 && k < sweeps; ++k)
        open = sweep(F.exres, n, F.ta.lab, F.exres, F.N, hops, t, stride, true);
    if (__ballot(open) != 0 && __lane_id() == 0) atomicOr(&plan->bctr[C_OPEN], 1u);
}

hipError_t launch_batched_init(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s)
{
    hipLaunchKernelGGL(k_binit, dim3(hplan.count), dim3(256), 0, s, dplan);
    return hipGetLastError();
}

hipError_t launch_batched_rest(const BatchPlan* dplan, const BatchPlan& hplan, hipStream_t s)
{
    const dim3 grid(kBatchBlocksPerField, hplan.count);
    hipLaunchKernelGGL(k_bexit_init, grid, dim3(256), 0, s, dplan);
    hipLaunchKernelGGL(k_bexit_jump, grid, dim3(256), 0, s, dplan);
    const hipError_t e = launch_final_tiled_batched(dplan, hplan, s);
    if (e != hipSuccess) return e;
    return launch_arcs_batched(dplan, hplan, s);
}

}  // namespace eg
