// The replica step's kernels: alone and over the members of a batch.
#include <hip/hip_runtime.h>

#include "fs_kernels.hpp"
#include "fs_reps.hpp"

namespace fsk {

template <int STORAGE, int LGW>
__global__ __launch_bounds__(REPS_TPB, reps_waves(LGW)) void reps_kernel(StepArgs a)
{
    __shared__ RepsShared<LGW> s;
    // (the first and only argument)
    reps_body<STORAGE, LGW>((ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr(), a.step_off, s, blockIdx.x, gridDim.x);
}

// Every member of a batch that runs the replica step with groups of 2^LGW
// chunks: member m owns the workgroups [first[m], first[m + 1]).
template <int STORAGE, int LGW>
__global__ __launch_bounds__(REPS_TPB, reps_waves(LGW)) void reps_batch_kernel(const StepArgs* __restrict__ table,
                                                              const uint32_t* __restrict__ first, uint32_t members,
                                                              uint32_t step_off)
{
    __shared__ RepsShared<LGW> s;
    const uint32_t m = owner_of(first, members, blockIdx.x);
    reps_body<STORAGE, LGW>((ArgsPtr)(unsigned long long)(table + m), step_off, s, blockIdx.x - first[m],
                            first[m + 1] - first[m]);
}

template <int S>
const void* reps_sel(int lgW, bool batch)
{
    switch (lgW) {
    case 2: return batch ? (const void*)&reps_batch_kernel<S, 2> : (const void*)&reps_kernel<S, 2>;
    case 3: return batch ? (const void*)&reps_batch_kernel<S, 3> : (const void*)&reps_kernel<S, 3>;
    case 4: return batch ? (const void*)&reps_batch_kernel<S, 4> : (const void*)&reps_kernel<S, 4>;
    default: return nullptr;
    }
}

const void* reps_kernel_fn(int storage, int lgW, bool batch)
{
    return storage == 0 ? reps_sel<0>(lgW, batch) : reps_sel<1>(lgW, batch);
}

} // namespace fsk
