// eg_batched.hip -- the label pass for a batch of fields.
//
// Every kernel here covers all fields of the batch in one launch: the grid's
// y dimension is the field, x strides over that field's items.  Stage (d)
// of a batch runs the stage (d) kernels with the batch field selector.
#include "eg_internal.h"

namespace eg {

constexpr int kBatchBlocksPerField = 48;  // a multiple of the exit list's regions
constexpr int kBatchRestBlocks = 64;      // a power of two

__global__ __launch_bounds__(256) void k_binit(const BatchPlan* __restrict__ plan)
{
    const BatchField& F = plan->fields[blockIdx.x];
    const int t = threadIdx.x;
    if (t < C_SLOTS) F.ta.ctr[t] = 0;
    if (t < kRegions) F.ta.claims[kRegionStride * t] = 0;
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
    exit_first(exit_part(F.ta.claims, F.ta.cap_region, F.ta.regions, blockIdx.x, gridDim.x), F.ta.exits, F.exres,
               F.ta.lab);
}

__global__ __launch_bounds__(256) void k_bexit_jump(const BatchPlan* __restrict__ plan)
{
    const BatchField F = plan->fields[blockIdx.y];  // a copy: loop loads cannot alias it
    const ExitPart p = exit_part(F.ta.claims, F.ta.cap_region, F.ta.regions, blockIdx.x, gridDim.x);
    const int hops = plan->tuning.hops;
    const bool capped = plan->capped != 0;
    const int sweeps = capped ? min(sweeps_for(plan->tuning, F.N), kCappedSweeps) : sweeps_for(plan->tuning, F.N);
    const int32_t* lab = F.ta.lab;
    int32_t* res = F.exres;
    int32_t* part = res + p.at;
    bool open = sweep(part, p.n, lab, res, F.N, hops, p.t, p.stride, false);
    for (int k = 1; __ballot(open) != 0 && k < sweeps; ++k)
        open = sweep(part, p.n, lab, res, F.N, hops, p.t, p.stride, true);
    if (__ballot(open) != 0 && __lane_id() == 0) atomicOr(&plan->bctr[capped ? C_CODES : C_OPEN], 1u);
}

// What the tile-ordered pass left open where lists are capped.
__global__ __launch_bounds__(256) void k_bcodes_rest(const BatchPlan* __restrict__ plan)
{
    if (plan->bctr[C_CODES] == 0) return;
    const BatchField F = plan->fields[blockIdx.y];
    codes_rest(F.ta.lab, F.exres, F.N, plan->tuning.hops, sweeps_for(plan->tuning, F.N), blockIdx.x, gridDim.x,
               F.ta.ctr, &plan->bctr[C_OPEN]);
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
    if (hplan.capped) {
        const dim3 rest(kBatchRestBlocks, hplan.count);
        hipLaunchKernelGGL(k_bcodes_rest, rest, dim3(256), 0, s, dplan);
    }
    return launch_arcs_batched(dplan, hplan, s);
}

}  // namespace eg
