// The replica step's kernels: alone and over the members of a batch.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fs_kernels.hpp"
#include "fs_reps.hpp"

namespace fsk {

template <int STORAGE, int LGW>
__global__ __launch_bounds__(REPS_TPB, 4) void reps_kernel(StepArgs a)
{
    __shared__ RepsShared<LGW> s;
    reps_body<STORAGE, LGW>(a, s, blockIdx.x, gridDim.x);
}

// Every member of a batch that runs the replica step with groups of 2^LGW
// chunks: member m owns the workgroups [first[m], first[m + 1]).
template <int STORAGE, int LGW>
__global__ __launch_bounds__(REPS_TPB, 4) void reps_batch_kernel(const StepArgs* __restrict__ table,
                                                              const uint32_t* __restrict__ first, uint32_t members,
                                                              uint32_t step_off)
{
    __shared__ RepsShared<LGW> s;
    const uint32_t m = owner_of(first, members, blockIdx.x);
    StepArgs a = table[m];
    a.step_off = step_off;
    reps_body<STORAGE, LGW>(a, s, blockIdx.x - first[m], first[m + 1] - first[m]);
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

// Exact counts of every replica added into base[R][4] (zeroed before): the
// counts the replica step's transitions are added to.
template <int STORAGE>
__global__ __launch_bounds__(WG) void count_all_kernel(const void* state_v, uint32_t total, int32_t lgR, uint32_t* base)
{
    using state_t = typename Store<STORAGE>::state_t;
    const state_t* state = (const state_t*)state_v;
    __shared__ uint32_t s[4 * 64];
    const uint32_t C = 4u << lgR, rm = (1u << lgR) - 1u;
    for (uint32_t i = threadIdx.x; i < C; i += WG) s[i] = 0;
    __syncthreads();
    for (uint32_t u = blockIdx.x * WG + threadIdx.x; u < total; u += gridDim.x * WG)
        atomicAdd(&s[(u & rm) * 4u + (uint32_t)state[u]], 1u); // LDS
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < C; i += WG)
        if (s[i]) atomicAdd(&base[i], s[i]);
}

hipError_t launch_count_all(int storage, const void* state, uint32_t total, int32_t lgR, uint32_t* base, hipStream_t s)
{
    hipError_t e = launch_clear_u32(base, (size_t)4 << lgR, s);
    if (e != hipSuccess) return e;
    const uint32_t g = std::max(1u, std::min((total + WG * 16u - 1u) / (WG * 16u), 1024u));
    if (storage == 0)
        hipLaunchKernelGGL(count_all_kernel<0>, dim3(g), dim3(WG), 0, s, state, total, lgR, base);
    else
        hipLaunchKernelGGL(count_all_kernel<1>, dim3(g), dim3(WG), 0, s, state, total, lgR, base);
    return hipGetLastError();
}

} // namespace fsk
