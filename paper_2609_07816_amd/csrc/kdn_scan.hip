// Chunk bookkeeping and the log-depth carry of the variance chain (arXiv 2609.07816, App.
// "Hardware-Efficient Chunkwise Algorithm", Sec. "Chunkwise Gain Computation", eq.
// chunk-gain-carry), shared by the forward and the gain scan.
//
// The variance recurrence of every (sequence, head, channel) is a product of 2x2 Moebius
// matrices acting on z = [n; d] (p = n / d). Given each chunk's summary M_bar_m (the product of
// its token matrices, later on the left), the state entering chunk m is
//   z_in_m = M_bar_{m-1} ... M_bar_0 z_0,   z_0 = [p_0; 1],
// an exclusive scan with an associative operator, 64 chunks per step (longer sequences carry step
// to step): one variance per head (isotropic) as a Kogge-Stone scan inside one wavefront, log2(64) =
// 6 rounds; one per channel (diagonal) as a tree of products of four.
#include "kdn_device.h"

namespace kdn {
namespace {

__global__ void chunk_table_kernel(const int32_t* __restrict__ cu, int N, int ntok, int ch,
                                   int maxch, int32_t* __restrict__ choff)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int acc = 0;
    for (int n = 0; n < N; ++n) {
        choff[n] = acc;
        const int t0 = min(max(cu[n], 0), ntok), t1 = min(max(cu[n + 1], t0), ntok);
        acc = min(acc + (t1 - t0 + ch - 1) / ch, maxch);
    }
    choff[N] = acc;
}

__device__ __forceinline__ float4 shfl_up4(float4 x, int off)
{
    return make_float4(__shfl_up(x.x, off, 64), __shfl_up(x.y, off, 64),
                       __shfl_up(x.z, off, 64), __shfl_up(x.w, off, 64));
}

// Diagonal: 16 channels per workgroup, a tree of three levels over 64 chunks per step: four chunks in
// each of 16 segments (a thread's loads, a row of 16 channels being 256 contiguous bytes), four
// segments in each wavefront, four wavefronts. A thread applies the wavefronts before its own, the
// segments before its own, and replays its chunks. Bound by the latency of one load and of that
// chain. A wavefront per channel with a lane per chunk (16-byte reads H d_k apart, 6 shuffle rounds)
// took 51 us for 2,100 chunks of 32 packed sequences (16 heads, d128) against 21 us, and 6.0 against
// 5.5 us for 4 x 64 chunks; two levels, 16 segments in order, 22 and 5.6 us.
constexpr int CPB = 16, NSEG = 16, SEGC = 4;
__global__ __launch_bounds__(CPB * NSEG) void carry_scan_diag_kernel(
    const float4* __restrict__ summ, const float* __restrict__ P0, ChunkMap cm, int ch, int H,
    int nchan, float2* __restrict__ carry, float* __restrict__ P_T)
{
    constexpr int NWV = CPB * NSEG / 64, SPW = 64 / CPB;  // wavefronts, segments in each
    __shared__ float4 seg[NSEG][CPB], s_wave[NWV][CPB];
    __shared__ float2 s_in[CPB];
    const int n = blockIdx.x / H, h = blockIdx.x % H;
    const int cl = threadIdx.x % CPB, sg = threadIdx.x / CPB;
    const int w = sg / SPW, sw = sg % SPW;  // wavefront, segment within it
    const int c = CPB * blockIdx.y + cl;
    int t0, t1;
    seq_span(cm, n, t0, t1);
    const int nchs = (t1 - t0 + ch - 1) / ch;
    const int g0 = cm.cu ? cm.choff[n] : n * ((cm.T + ch - 1) / ch);
    const int nch = max(0, min(nchs, cm.maxch - g0));
    const size_t pidx = ((size_t)n * H + h) * nchan + c;
    if (nch == 0) {  // an empty sequence keeps its initial variances
        if (P_T && sg == 0) P_T[pidx] = P0 ? P0[pidx] : 1.f;
        return;
    }
    const size_t base = ((size_t)g0 * H + h) * nchan + c, stride = (size_t)H * nchan;
    float2 zin = make_float2(P0 ? P0[pidx] : 1.f, 1.f);  // z_0 = [p_0; 1]
    for (int b0 = 0; b0 < nch; b0 += NSEG * SEGC) {
        const int m0 = b0 + SEGC * sg;
        float4 x[SEGC];
#pragma unroll
        for (int i = 0; i < SEGC; ++i) {
            x[i] = make_float4(1.f, 0.f, 0.f, 1.f);
            if (m0 + i < nch) x[i] = summ[base + (size_t)(m0 + i) * stride];
        }
        float4 p = x[0];
#pragma unroll
        for (int i = 1; i < SEGC; ++i) p = mat_mul(x[i], p);
        seg[sg][cl] = p;
        __syncthreads();
        if (sw == 0) {  // the product of the wavefront's segments
#pragma unroll
            for (int q = 1; q < SPW; ++q) p = mat_mul(seg[sg + q][cl], p);
            s_wave[w][cl] = p;
        }
        __syncthreads();
        float2 z = zin;
#pragma unroll
        for (int q = 0; q < NWV - 1; ++q) {
            const float2 y = mat_vec(s_wave[q][cl], z);
            z = q < w ? y : z;
        }
#pragma unroll
        for (int q = 0; q < SPW - 1; ++q) {
            const float2 y = mat_vec(seg[SPW * w + q][cl], z);
            z = q < sw ? y : z;
        }
#pragma unroll
        for (int i = 0; i < SEGC; ++i) {
            if (m0 + i < nch) {
                carry[base + (size_t)(m0 + i) * stride] = z;
                z = mat_vec(x[i], z);
            }
        }
        if (sg == NSEG - 1) s_in[cl] = z;  // after the step's last chunk (it fills every segment)
        __syncthreads();
        zin = s_in[cl];
    }
}

// Isotropic: one wavefront per (sequence, head), its lanes are chunks. Grid N * H.
__global__ __launch_bounds__(64) void carry_scan_iso_kernel(const float4* __restrict__ summ,
                                                         const float* __restrict__ P0,
                                                         ChunkMap cm, int ch, int H,
                                                         float2* __restrict__ carry,
                                                         float* __restrict__ P_T)
{
    const int n = blockIdx.x / H, h = blockIdx.x % H;
    if (n >= cm.N) return;
    const int lane = threadIdx.x;
    int t0, t1;
    seq_span(cm, n, t0, t1);
    const int nchs = (t1 - t0 + ch - 1) / ch;
    const int g0 = cm.cu ? cm.choff[n] : n * ((cm.T + ch - 1) / ch);
    const int nch = max(0, min(nchs, cm.maxch - g0));
    const size_t pidx = (size_t)n * H + h;
    if (nch == 0) {  // an empty sequence keeps its initial variances
        if (P_T && lane == 0) P_T[pidx] = P0 ? P0[pidx] : 1.f;
        return;
    }
    float cn = P0 ? P0[pidx] : 1.f, cd = 1.f;  // z_0 = [p_0; 1]
    for (int b0 = 0; b0 < nch; b0 += 64) {
        const int m = b0 + lane;
        float4 x = make_float4(1.f, 0.f, 0.f, 1.f);
        if (m < nch) x = summ[(size_t)(g0 + m) * H + h];
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {  // inclusive prefix, later chunks on the left
            const float4 y = shfl_up4(x, off);
            if (lane >= off) x = mat_mul(x, y);
        }
        float zn = fmaf(x.x, cn, x.y * cd), zd = fmaf(x.z, cn, x.w * cd);  // after chunk m
        rescale2(zn, zd);
        float en = __shfl_up(zn, 1, 64), ed = __shfl_up(zd, 1, 64);       // before chunk m
        if (lane == 0) {
            en = cn;
            ed = cd;
        }
        if (m < nch) carry[(size_t)(g0 + m) * H + h] = make_float2(en, ed);
        const int lastl = min(63, nch - 1 - b0);
        cn = __shfl(zn, lastl, 64);
        cd = __shfl(zd, lastl, 64);
    }
}

__global__ __launch_bounds__(1024) void order_kernel(const int32_t* __restrict__ cu, int N,
                                                     int ntok, int32_t* __restrict__ order)
{
    __shared__ int32_t len[ORDER_MAX];
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
        const int t0 = min(max(cu[i], 0), ntok), t1 = min(max(cu[i + 1], t0), ntok);
        len[i] = t1 - t0;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < N; i += blockDim.x) {
        const int li = len[i];
        int rank = 0;
        for (int j = 0; j < N; ++j) {
            const int lj = len[j];
            rank += (lj > li) || (lj == li && j < i);
        }
        order[rank] = i;
    }
}

}  // namespace

hipError_t launch_chunk_table(const int32_t* cu, int N, int ntok, int ch, int maxch,
                              int32_t* choff, hipStream_t st)
{
    hipLaunchKernelGGL(chunk_table_kernel, dim3(1), dim3(1), 0, st, cu, N, ntok, ch, maxch,
                       choff);
    return hipGetLastError();
}

hipError_t launch_carry_scan(const float4* summ, const float* P0, const ChunkMap& cm, int ch,
                             int H, int nchan, float2* carry, float* P_T, hipStream_t st)
{
    if (nchan == 1)
        hipLaunchKernelGGL(carry_scan_iso_kernel, dim3((unsigned)(cm.N * H)), dim3(64), 0, st, summ,
                           P0, cm, ch, H, carry, P_T);
    else  // nchan = d_k, a multiple of 16
        hipLaunchKernelGGL(carry_scan_diag_kernel,
                           dim3((unsigned)(cm.N * H), (unsigned)(nchan / CPB)), dim3(CPB * NSEG), 0,
                           st, summ, P0, cm, ch, H, nchan, carry, P_T);
    return hipGetLastError();
}

hipError_t launch_order(const int32_t* cu, int N, int ntok, int32_t* order, hipStream_t st)
{
    if (N > ORDER_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(order_kernel, dim3(1), dim3(1024), 0, st, cu, N, ntok, order);
    return hipGetLastError();
}

}  // namespace kdn
