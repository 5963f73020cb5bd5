// ea_group.hip -- per-class kernels of the walker-interleaved LDS engine
// (ea_group.hpp: Gaussian couplings; ea_groupbits.hpp: +-1).
#include "ea_group.hpp"
#include "ea_groupbits.hpp"

namespace ea {

// VAR only separates the symbol of the one-sample-per-launch comparator.
template <int L, int JK, int VAR>
__global__ void __launch_bounds__(GROUP_MAX_THREADS, 4) group_sweep_kernel(SweepArgs A)
{
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int code = A.items[blockIdx.x];
    const SampleDev d = sample_of_item(A.samples, code >> 1);
    if constexpr (JK == 0) run_group_item<L>(A, d, code & 1, smem);
    else run_group_bits_item<L>(A, d, code & 1, smem, whole_block());
}

#define EA_GROUP(Lv)                                                 \
    template __global__ void group_sweep_kernel<Lv, 0, 0>(SweepArgs); \
    template __global__ void group_sweep_kernel<Lv, 1, 0>(SweepArgs); \
    template __global__ void group_sweep_kernel<Lv, 0, 1>(SweepArgs); \
    template __global__ void group_sweep_kernel<Lv, 1, 1>(SweepArgs);
EA_GROUP(2)
EA_GROUP(4)
EA_GROUP(6)
EA_GROUP(8)
EA_GROUP(10)
EA_GROUP(12)
EA_GROUP(14)
EA_GROUP(16)
#undef EA_GROUP

}  // namespace ea
