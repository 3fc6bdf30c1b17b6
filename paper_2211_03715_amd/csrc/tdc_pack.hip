// Weight re-layout kernels: caller layouts -> the frag-major packed layout of tdc_internal.h.
// The paper (section 5.2) converts its core weights to a coalescing-friendly layout once,
// offline; this is the same step for this library's MFMA operand order.
#include <algorithm>

#include "tdc_split.h"
#include "tdc_internal.h"

size_t tdc_packed_floats_uin(const TdcDims &d) { return (size_t)d.NB1 * d.KG1 * 256; }
size_t tdc_packed_floats_core(const TdcDims &d) { return (size_t)d.NB2 * d.K * d.K * d.NB1 * 256; }
size_t tdc_packed_floats_uout(const TdcDims &d) { return (size_t)d.NB3 * d.NB2 * 256; }

namespace {

// e = ((mb*KG + kg)*64 + lane)*4 + j  ->  k = 16*kg + 4*(lane/16) + j, m = 16*mb + lane%16
__device__ __forceinline__ void unpack_index(size_t e, int kgroups, int &mb, int &kg, int &k16, int &m)
{
    const int j = (int)(e & 3);
    const int lane = (int)((e >> 2) & 63);
    const size_t blk = e >> 8;
    kg = (int)(blk % kgroups);
    mb = (int)(blk / kgroups);
    k16 = 4 * (lane >> 4) + j;
    m = 16 * mb + (lane & 15);
}

__global__ void pack_uin_kernel(TdcDims d, const float *__restrict__ U_in, float *__restrict__ out, size_t total)
{
    size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    int mb, kg, k16, m;
    unpack_index(e, d.KG1, mb, kg, k16, m);
    if (d.s1_runs) k16 = 4 * (k16 & 3) + (k16 >> 2);      // component j of lane group g holds channel 4*j + g
    const int c = 16 * kg + k16;
    out[e] = (c < d.C && m < d.R1) ? U_in[(size_t)c * d.R1 + m] : 0.f;
}

__global__ void pack_core_kernel(TdcDims d, const float *__restrict__ core, float *__restrict__ out, size_t total)
{
    size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    int mb, kg, k16, m;
    unpack_index(e, d.K * d.K * d.NB1, mb, kg, k16, m);
    const int tap = kg / d.NB1;              // r*K + s
    const int d1 = 16 * (kg % d.NB1) + k16;
    const int r = tap / d.K, s = tap % d.K;
    out[e] = (d1 < d.R1 && m < d.R2) ? core[(((size_t)d1 * d.R2 + m) * d.K + r) * d.K + s] : 0.f;
}

// ---- parts (tdc_split.h)
//
// Output channel m of a weight tensor is scaled by 2^scale[m], its largest weight to 2^13 .. 2^14; rows of the core by the inverse of U_in's
// scales before that.  A channel that has weights from 2^10 on beside others that the scaling takes below 2^-13 (three parts: 2^-1), where
// parts lose bits, is kept in fp32 alone: its parts are NaN.  Smaller weights beside ordinary ones only lose what is below the
// rounding of their channel's sums, or else those are watched (tdc_split.h).

// One weight tensor w[row][col][tap] -- the contraction runs over rows and taps -- and where things go.
struct SplitTensor {
    const float *w;
    int rows, cols, KK, NBk, NBm, KG;      // NBk, KG: k-groups per tap and in all
    unsigned *parts;
    int *exponents;
    float *raw;
    int *top, *low, *most, *odd;           // of each channel's weights the largest and smallest exponent, the largest before ranks
                                           // are scaled, and whether one is no number, TDC_SPLIT_CHUNKS shares
    bool last;                             // U_out, W
    // The core: U_in [rows_before][rows], whose columns are scaled each by its own power of two.  A row is scaled by the inverse,
    // so that z1 holds all ranks at one size, and what size the ranks have between the two factors makes no difference.
    const float *before;
    int rows_before;
};
constexpr int SPLIT_NONE = 100000, SPLIT_TOP = 13;

// channels without a finite weight that is not zero take 0
__device__ __forceinline__ int split_scale(int top) { return top == -SPLIT_NONE ? 0 : SPLIT_TOP - top; }
__device__ __forceinline__ bool split_counts(float w) { return w != 0.f && fabsf(w) < INFINITY; }

// over a workgroup of 256
__device__ __forceinline__ int split_block_max(int v)
{
    __shared__ int part[256];
    __syncthreads();
    part[threadIdx.x] = v;
    __syncthreads();
    for (int s = 128; s; s >>= 1) {
        if ((int)threadIdx.x < s) part[threadIdx.x] = max(part[threadIdx.x], part[threadIdx.x + s]);
        __syncthreads();
    }
    return part[0];
}
// the largest of a channel's shares, by the 16 lanes that have one each
__device__ __forceinline__ int split_share_max(int v)
{
    for (int s = 8; s; s >>= 1) v = max(v, __shfl_xor(v, s));
    return v;
}

// the scale of column m of the tensor before, by a wavefront
__device__ __forceinline__ int split_scale_before(const SplitTensor &t, int m)
{
    int top = -SPLIT_NONE;
    for (int row = threadIdx.x & 63; row < t.rows_before; row += 64) {
        const float w = t.before[(size_t)row * t.rows + m];
        if (split_counts(w)) top = max(top, ilogbf(w));
    }
    for (int s = 32; s; s >>= 1) top = max(top, __shfl_xor(top, s));
    return split_scale(top);
}

// the ranges of 64 output channels' weights among one share of the rows
__device__ __forceinline__ void split_range(const SplitTensor &t, int block)
{
    __shared__ int top4[256], low4[256], most4[256], odd4[256];
    const int share = block % TDC_SPLIT_CHUNKS, m = block / TDC_SPLIT_CHUNKS * 64 + (threadIdx.x & 63);
    int top = -SPLIT_NONE, low = SPLIT_NONE, most = -SPLIT_NONE, odd = 0;
    for (int row = share + TDC_SPLIT_CHUNKS * (threadIdx.x >> 6); row < t.rows; row += 4 * TDC_SPLIT_CHUNKS) {
        const int undo = t.before ? split_scale_before(t, row) : 0;
        const float *__restrict__ w = t.w + ((size_t)row * t.cols + m) * t.KK;
        for (int i = 0; i < (m < t.cols ? t.KK : 0); ++i) {
            odd |= !(fabsf(w[i]) < INFINITY);
            if (split_counts(w[i])) {
                const int e = ilogbf(w[i]);
                top = max(top, e - undo);
                low = min(low, e - undo);
                most = max(most, e);
            }
        }
    }
    top4[threadIdx.x] = top;
    low4[threadIdx.x] = low;
    most4[threadIdx.x] = most;
    odd4[threadIdx.x] = odd;
    __syncthreads();
    if (threadIdx.x < 64 && m < 16 * t.NBm) {
        const auto max4 = [](const int *p) { return max(max(p[0], p[64]), max(p[128], p[192])); };
        const int at = share * 16 * t.NBm + m, *q = low4 + threadIdx.x;
        t.top[at] = max4(top4 + threadIdx.x);
        t.most[at] = max4(most4 + threadIdx.x);
        t.odd[at] = max4(odd4 + threadIdx.x);
        t.low[at] = min(min(q[0], q[64]), min(q[128], q[192]));
    }
}

struct SplitArgs {
    SplitTensor t[3];
    int n;                                 // 3: U_in, core, U_out; 1: W
};
__global__ void split_range_kernel(SplitArgs a)
{
    if (a.n == 3 && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) a.t[0].exponents[0] = 0;
    if ((int)blockIdx.x < (a.t[blockIdx.y].NBm + 3) / 4 * TDC_SPLIT_CHUNKS) split_range(a.t[blockIdx.y], blockIdx.x);
}

// One thread per pair of components: e = ((mb*S + step)*64 + lane)*4 + pair, one workgroup per block and step.  Exponents: W: the
// channel's; U_in: none, its scales are the core's rows', but in the first place whether a weight of the layer is no number or not in
// parts; core: what takes a channel to the scale of the largest; U_out: the channel's and that scale together.
template <int NP>
__global__ void split_pack_kernel(SplitArgs a)
{
    static_assert(TDC_SPLIT_CHUNKS == 16, "a share to each of 16 lanes");
    const SplitTensor &t = a.t[blockIdx.y];
    const int S = (t.KG + 1) / 2;
    if ((int)blockIdx.x >= t.NBm * S) return;
    const int pair = (int)(threadIdx.x & 3), lane = (int)(threadIdx.x >> 2);
    const size_t blk = blockIdx.x;
    const int step = (int)(blk % S), mb = (int)(blk / S);
    __shared__ int scales[16], wides[16], undo[2][16];
    {   // 16 channels, 16 shares of each
        const int share = threadIdx.x & 15, c = threadIdx.x >> 4, at = share * 16 * t.NBm + 16 * mb + c;
        const int top = split_share_max(t.top[at]), low = -split_share_max(-t.low[at]), most = split_share_max(t.most[at]), odd = split_share_max(t.odd[at]);
        const bool empty = top == -SPLIT_NONE, wide = !empty && most >= 10 && top - low > SPLIT_TOP - tdc_lowest_weight(NP);
        if (share == 0) {
            scales[c] = empty ? SPLIT_NONE : split_scale(top);
            wides[c] = wide;
            if (a.n == 3 && step == 0 && (wide || odd)) atomicOr(a.t[0].exponents, 1);
        }
        if (t.before)
            for (int h = 0; h < 2; ++h) {
                const int kg = 2 * step + h, row = 16 * (kg % t.NBk) + c;
                const int v = split_share_max(kg < t.KG && row < t.rows ? a.t[0].top[share * 16 * a.t[0].NBm + row] : -SPLIT_NONE);
                if (share == 0) undo[h][c] = split_scale(v);
            }
    }
    __syncthreads();
    const int kg = 2 * step + (pair >> 1), m = 16 * mb + (lane & 15), k = 4 * (lane >> 4) + 2 * (pair & 1);
    const int scale = scales[lane & 15];
    const bool wide = wides[lane & 15], empty = scale == SPLIT_NONE;
    const int tap = kg / t.NBk, row = 16 * (kg - tap * t.NBk) + k;
    float v[2], scaled[2];
    for (int i = 0; i < 2; ++i) {
        const bool there = kg < t.KG && row + i < t.rows;
        v[i] = there && m < t.cols ? t.w[((size_t)(row + i) * t.cols + m) * t.KK + tap] : 0.f;
        scaled[i] = ldexpf(v[i], (empty ? 0 : scale) - (t.before ? undo[pair >> 1][k + i] : 0));
        if (wide) scaled[i] = NAN;
        if (t.last && empty && v[i] == 0.f) scaled[i] = there ? ((row + i) % 2 ? 0x1p12f : 0x1p13f) : 0.f;       // see TDC_EMPTY
    }
    unsigned p[NP];
    tdc_split2<NP, tdc_lift_weights(NP)>(scaled[0], scaled[1], TdcScale(0), p);
    for (int i = 0; i < NP; ++i) t.parts[(blk * NP + i) * 256 + lane * 4 + pair] = p[i];
    if (kg < t.KG) {
        float *raw = t.raw + (((size_t)mb * t.KG + kg) * 64 + lane) * 4 + 2 * (pair & 1);
        raw[0] = v[0];
        raw[1] = v[1];
    }
    if (step || (a.n == 3 && blockIdx.y == 0)) return;
    int lowest = 0;                                    // the scale of the core's largest channel
    if (a.n == 3) {
        const SplitTensor &c = a.t[1];
        int top = -SPLIT_NONE;
        for (int i = threadIdx.x; i < 16 * c.NBm * TDC_SPLIT_CHUNKS; i += 256) top = max(top, c.top[i]);
        lowest = split_scale(split_block_max(top));
    }
    if (threadIdx.x < 16) {
        const int sc = scales[threadIdx.x];
        t.exponents[16 * mb + threadIdx.x] = wides[threadIdx.x] ? TDC_WIDE : sc == SPLIT_NONE ? (t.last ? TDC_EMPTY : 0) : t.last ? sc + lowest : lowest - sc;
    }
}

__global__ void pack_uout_kernel(TdcDims d, const float *__restrict__ U_out, float *__restrict__ out, size_t total)
{
    size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    int mb, kg, k16, m;
    unpack_index(e, d.NB2, mb, kg, k16, m);
    const int d2 = 16 * kg + k16;
    out[e] = (d2 < d.R2 && m < d.N) ? U_out[(size_t)d2 * d.N + m] : 0.f;
}

// Wm[d1][n][r][s] = sum_d2 core[d1][d2][r][s] * U_out[d2][n]: stage 3 folded into the core.
__global__ void merge_core_uout_kernel(TdcDims d, const float *__restrict__ core, const float *__restrict__ U_out,
                                       float *__restrict__ wm, size_t total)
{
    size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= total) return;
    const int KK = d.K * d.K;
    const int tap = (int)(e % KK);
    const int n = (int)((e / KK) % d.N);
    const int d1 = (int)(e / ((size_t)KK * d.N));
    float acc = 0.f;
    for (int d2 = 0; d2 < d.R2; ++d2) acc += core[((size_t)d1 * d.R2 + d2) * KK + tap] * U_out[(size_t)d2 * d.N + n];
    wm[e] = acc;
}

}  // namespace

hipError_t tdc_launch_pack_merged(const TdcDims &d, hipStream_t s, const float *U_in, const float *core,
                                  const float *U_out, float *uin_p, float *wm, float *wm_p)
{
    const int T = 256;
    const size_t n1 = tdc_packed_floats_uin(d), nm = (size_t)d.R1 * d.N * d.K * d.K;
    hipLaunchKernelGGL(pack_uin_kernel, dim3((unsigned)((n1 + T - 1) / T)), dim3(T), 0, s, d, U_in, uin_p, n1);
    hipLaunchKernelGGL(merge_core_uout_kernel, dim3((unsigned)((nm + T - 1) / T)), dim3(T), 0, s, d, core, U_out, wm, nm);
    TdcDims m = d;          // the merged kernel is a core tensor with R2 = N
    m.R2 = d.N;
    m.NB2 = d.NB3;
    const size_t n2 = tdc_packed_floats_core(m);
    hipLaunchKernelGGL(pack_core_kernel, dim3((unsigned)((n2 + T - 1) / T)), dim3(T), 0, s, m, wm, wm_p, n2);
    return hipGetLastError();
}

hipError_t tdc_launch_pack(const TdcDims &d, hipStream_t s, const float *U_in, const float *core,
                           const float *U_out, float *uin_p, float *core_p, float *uout_p)
{
    const int T = 256;
    size_t n1 = tdc_packed_floats_uin(d), n2 = tdc_packed_floats_core(d), n3 = tdc_packed_floats_uout(d);
    hipLaunchKernelGGL(pack_uin_kernel, dim3((unsigned)((n1 + T - 1) / T)), dim3(T), 0, s, d, U_in, uin_p, n1);
    hipLaunchKernelGGL(pack_core_kernel, dim3((unsigned)((n2 + T - 1) / T)), dim3(T), 0, s, d, core, core_p, n2);
    hipLaunchKernelGGL(pack_uout_kernel, dim3((unsigned)((n3 + T - 1) / T)), dim3(T), 0, s, d, U_out, uout_p, n3);
    return hipGetLastError();
}

hipError_t tdc_launch_pack_core(const TdcDims &d, hipStream_t s, const float *core, float *core_p)
{
    const int T = 256;
    const size_t n2 = tdc_packed_floats_core(d);
    hipLaunchKernelGGL(pack_core_kernel, dim3((unsigned)((n2 + T - 1) / T)), dim3(T), 0, s, d, core, core_p, n2);
    return hipGetLastError();
}

static SplitTensor split_tensor(int parts, const float *w, int rows, int cols, int K, void *out, bool last)
{
    SplitTensor t;
    t.w = w; t.rows = rows; t.cols = cols; t.KK = K * K;
    t.NBk = (rows + 15) / 16; t.NBm = (cols + 15) / 16; t.KG = t.KK * t.NBk;
    t.parts = (unsigned *)out;
    t.exponents = (int *)((char *)out + tdc_split_bytes(parts, t.NBm, t.KG));
    t.raw = (float *)(t.exponents + 16 * t.NBm);
    t.top = (int *)(t.raw + (size_t)t.NBm * t.KG * 256);
    t.low = t.top + 16 * t.NBm * TDC_SPLIT_CHUNKS;
    t.most = t.low + 16 * t.NBm * TDC_SPLIT_CHUNKS;
    t.odd = t.most + 16 * t.NBm * TDC_SPLIT_CHUNKS;
    t.last = last;
    t.before = nullptr;
    t.rows_before = 0;
    return t;
}

static hipError_t launch_split(int parts, hipStream_t s, const SplitArgs &a)
{
    size_t ranges = 0, packs = 0;
    for (int i = 0; i < a.n; ++i) {
        ranges = std::max(ranges, (size_t)(a.t[i].NBm + 3) / 4 * TDC_SPLIT_CHUNKS);
        packs = std::max(packs, (size_t)a.t[i].NBm * ((a.t[i].KG + 1) / 2));
    }
    hipLaunchKernelGGL(split_range_kernel, dim3((unsigned)ranges, a.n), dim3(256), 0, s, a);
    hipLaunchKernelGGL(parts == 2 ? split_pack_kernel<2> : split_pack_kernel<3>, dim3((unsigned)packs, a.n), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t tdc_launch_split_core(const TdcDims &d, int parts, hipStream_t s, const float *core, void *core_sp)
{
    SplitArgs a = {};
    a.n = 1;
    a.t[0] = split_tensor(parts, core, d.R1, d.R2, d.K, core_sp, true);
    return launch_split(parts, s, a);
}

hipError_t tdc_launch_split_layer(const TdcDims &d, hipStream_t s, const float *U_in, const float *core, const float *U_out,
                                  void *uin_sp, void *core_sp, void *uout_sp)
{
    SplitArgs a = {};
    a.n = 3;
    a.t[0] = split_tensor(2, U_in, d.C, d.R1, 1, uin_sp, false);
    a.t[1] = split_tensor(2, core, d.R1, d.R2, d.K, core_sp, false);
    a.t[1].before = U_in;
    a.t[1].rows_before = d.C;
    a.t[2] = split_tensor(2, U_out, d.R2, d.N, 1, uout_sp, true);
    return launch_split(2, s, a);
}
