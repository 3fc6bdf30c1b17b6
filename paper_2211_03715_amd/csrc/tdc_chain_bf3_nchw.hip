// Instances of the bf16-part CHAIN kernel for NCHW activations read four bytes at a time.
#include "tdc_chain_bf3_kernel.h"

hipError_t tdc_launch_chain_bf3_nchw(const TdcChainBf3Args &a, int nb2, int pb, int mb1, dim3 grid, size_t lds, hipStream_t s, bool prepare_only)
{
    return tdc_launch_chain_bf3_lay<TDC_LAY_NCHW>(a, nb2, pb, mb1, grid, lds, s, prepare_only);
}
