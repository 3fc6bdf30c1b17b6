// Weight re-layout in three bf16 parts (tdc_bf3.h, layout: tdc_internal.h), for the layers that run CHAIN or the dense tiles in them.
#include "tdc_bf3.h"
#include "tdc_internal.h"

namespace {

// The largest magnitudes below 2^126 of RANGE_BLOCKS parts of each of up to three weight tensors, behind their packed parts.
constexpr int RANGE_BLOCKS = TDC_PACKED3_TAIL / 4;
struct RangeArgs {
    const float *w[3];
    size_t n[3];
    float *largest[3];
};
__global__ void pack3_range_kernel(RangeArgs a)
{
    const float *__restrict__ w = a.w[blockIdx.y];
    const size_t n = a.n[blockIdx.y];
    float m = 0.f;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const float v = fabsf(w[i]);
        if (v < TDC_BIG) m = fmaxf(m, v);
    }
    __shared__ float part[256];
    part[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s; s >>= 1) {
        if ((int)threadIdx.x < s) part[threadIdx.x] = fmaxf(part[threadIdx.x], part[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) a.largest[blockIdx.y][blockIdx.x] = part[0];
}

// One thread per pair of components of the three-part layout: e = ((mb*S + step)*64 + lane)*4 + pair.  weight(kg, k, m) is
// the value of k-group kg's contraction index k (0..15) and output channel m, zero past the end of either.  A tensor whose
// largest weight is outside 2^-100 .. 2^14 is kept raw altogether (tdc_bf3.h).
template <class Weight>
__device__ __forceinline__ void pack3(size_t e, int KG, unsigned *__restrict__ out, const float *__restrict__ largest, Weight weight)
{
    float top = 0.f;
    for (int i = 0; i < RANGE_BLOCKS; ++i) top = fmaxf(top, largest[i]);
    const float least = top < 0x1p-100f || top > 0x1p14f ? INFINITY : 0.f;
    const int S = (KG + 1) / 2;
    const int pair = (int)(e & 3), lane = (int)((e >> 2) & 63);
    const size_t blk = e >> 8;
    const int step = (int)(blk % S), mb = (int)(blk / S);
    const int kg = 2 * step + (pair >> 1), m = 16 * mb + (lane & 15), k = 4 * (lane >> 4) + 2 * (pair & 1);
    unsigned p[3];
    tdc_split2_raw(kg < KG ? weight(kg, k, m) : 0.f, kg < KG ? weight(kg, k + 1, m) : 0.f, least, p[0], p[1], p[2]);
    for (int i = 0; i < 3; ++i) out[(blk * 3 + i) * 256 + lane * 4 + pair] = p[i];
}

__global__ void pack3_core_kernel(TdcDims d, const float *__restrict__ core, unsigned *__restrict__ out, const float *__restrict__ largest, size_t total)
{
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    pack3(e, d.K * d.K * d.NB1, out, largest, [&](int kg, int k, int m) {
        const int tap = kg / d.NB1, r = tap / d.K, s = tap % d.K, d1 = 16 * (kg % d.NB1) + k;
        return d1 < d.R1 && m < d.R2 ? core[(((size_t)d1 * d.R2 + m) * d.K + r) * d.K + s] : 0.f;
    });
}

// U_in [C][R1] and U_out [R2][N]: w[k][m], `rows` x `cols`
__global__ void pack3_matrix_kernel(int rows, int cols, const float *__restrict__ w, unsigned *__restrict__ out, const float *__restrict__ largest, size_t total)
{
    const size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    pack3(e, (rows + 15) / 16, out, largest, [&](int kg, int k, int m) {
        return 16 * kg + k < rows && m < cols ? w[(size_t)(16 * kg + k) * cols + m] : 0.f;
    });
}

float *pack3_largest(void *packed, size_t bytes) { return reinterpret_cast<float *>(static_cast<char *>(packed) + bytes); }

}  // namespace

hipError_t tdc_launch_pack3(const TdcDims &d, hipStream_t s, const float *U_in, const float *core, const float *U_out,
                            void *uin_p3, void *core_p3, void *uout_p3)
{
    const int T = 256;
    const size_t b1 = tdc_packed3_bytes(d.NB1, d.KG1), b2 = tdc_packed3_bytes(d.NB2, d.K * d.K * d.NB1), b3 = tdc_packed3_bytes(d.NB3, d.NB2);
    const RangeArgs r = {{U_in, core, U_out},
                         {(size_t)d.C * d.R1, (size_t)d.R1 * d.R2 * d.K * d.K, (size_t)d.R2 * d.N},
                         {pack3_largest(uin_p3, b1), pack3_largest(core_p3, b2), pack3_largest(uout_p3, b3)}};
    hipLaunchKernelGGL(pack3_range_kernel, dim3(RANGE_BLOCKS, 3), dim3(256), 0, s, r);
    const size_t n1 = b1 / 12, n2 = b2 / 12, n3 = b3 / 12;
    hipLaunchKernelGGL(pack3_matrix_kernel, dim3((unsigned)((n1 + T - 1) / T)), dim3(T), 0, s, d.C, d.R1, U_in, (unsigned *)uin_p3, r.largest[0], n1);
    hipLaunchKernelGGL(pack3_matrix_kernel, dim3((unsigned)((n3 + T - 1) / T)), dim3(T), 0, s, d.R2, d.N, U_out, (unsigned *)uout_p3, r.largest[2], n3);
    hipLaunchKernelGGL(pack3_core_kernel, dim3((unsigned)((n2 + T - 1) / T)), dim3(T), 0, s, d, core, (unsigned *)core_p3, r.largest[1], n2);
    return hipGetLastError();
}

hipError_t tdc_launch_pack3_core(const TdcDims &d, hipStream_t s, const float *core, void *core_p3)
{
    const int T = 256;
    const size_t bytes = tdc_packed3_bytes(d.NB2, d.K * d.K * d.NB1), n = bytes / 12;
    const RangeArgs r = {{core}, {(size_t)d.R1 * d.R2 * d.K * d.K}, {pack3_largest(core_p3, bytes)}};
    hipLaunchKernelGGL(pack3_range_kernel, dim3(RANGE_BLOCKS), dim3(256), 0, s, r);
    hipLaunchKernelGGL(pack3_core_kernel, dim3((unsigned)((n + T - 1) / T)), dim3(T), 0, s, d, core, (unsigned *)core_p3, r.largest[0], n);
    return hipGetLastError();
}
