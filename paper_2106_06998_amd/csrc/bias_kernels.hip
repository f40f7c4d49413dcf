// Bias gradient of a convolution layer: db[m] = sum_{b,oy,ox} dY[b,m,oy,ox], in fp32, rounded once to the storage type.
// One streaming read of dY; bound by HBM.  Planes: a workgroup sums a piece of one channel's values (the channel's planes over
// the batch counted as one run of vectors, S pieces so that about two workgroups per compute unit are resident); channels-last:
// a workgroup sums a run of pixels, its threads along the channels.  S > 1: the pieces are added in order afterwards, so that
// the result does not depend on timing, in the launch of the weight gradient's second pass or in one of their own.
#include <algorithm>

#include "common.h"
#include "launch.h"

namespace xc {

namespace {

template <int DT> struct BiasElem { typedef uint16_t t; };
template <> struct BiasElem<XCONV_F32> { typedef float t; };

template <int DT> __device__ inline float bias_val(typename BiasElem<DT>::t v)
{
    if constexpr (DT == XCONV_F32) return v;
    else return st16_to_f32<DT>(v);
}
template <int DT> __device__ inline void bias_put(void *out, int c, float v)
{
    if constexpr (DT == XCONV_F32) static_cast<float *>(out)[c] = v;
    else static_cast<uint16_t *>(out)[c] = f32_to_st16<DT>(v);
}
// sum of the values of a 16-byte vector
template <int DT> __device__ inline float vec_sum(const uint4 &v)
{
    if constexpr (DT == XCONV_F32) {
        return (__uint_as_float(v.x) + __uint_as_float(v.y)) + (__uint_as_float(v.z) + __uint_as_float(v.w));
    } else {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) s += st16_to_f32<DT>((uint16_t)(w[i] & 0xffffu)) + st16_to_f32<DT>((uint16_t)(w[i] >> 16));
        return s;
    }
}

// planes.  HWv: vectors (VEC) or values per plane; piece s of a channel: vectors [s * len, (s + 1) * len) of its B * HWv
template <int DT, bool VEC>
__global__ __launch_bounds__(kThreads) void bias_planes_kernel(const void *dY, float *part, void *db, int B, int C, int HWv, long long len)
{
    typedef typename BiasElem<DT>::t elem_t;
    __shared__ float red[kThreads / 64];
    const int tid = threadIdx.x, c = blockIdx.x;
    const long long total = (long long)B * HWv, i0 = blockIdx.y * len, i1 = std::min(i0 + len, total);
    constexpr int U = 8;                          // loads in flight per thread
    float acc[U];
#pragma unroll
    for (int u = 0; u < U; ++u) acc[u] = 0.f;
    // (image, vector) of the thread's next value, advanced without divisions
    long long i = i0 + tid;
    long long b = i / HWv;
    int p = (int)(i - b * HWv);
    const int sb = kThreads / HWv, sp = kThreads - sb * HWv;
    while (i < i1) {
        uint4 v[U];
        elem_t e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool on = i < i1;
            const size_t at = ((size_t)(on ? b : 0) * C + c) * HWv + (on ? p : 0);
            if constexpr (VEC) v[u] = on ? static_cast<const uint4 *>(dY)[at] : uint4{0, 0, 0, 0};
            else e[u] = on ? static_cast<const elem_t *>(dY)[at] : elem_t(0);
            i += kThreads;
            b += sb;
            p += sp;
            if (p >= HWv) { p -= HWv; ++b; }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if constexpr (VEC) acc[u] += vec_sum<DT>(v[u]);
            else acc[u] += bias_val<DT>(e[u]);
        }
    }
    float s = ((acc[0] + acc[1]) + (acc[2] + acc[3])) + ((acc[4] + acc[5]) + (acc[6] + acc[7]));
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
    if ((tid & 63) == 0) red[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
        const float t = (red[0] + red[1]) + (red[2] + red[3]);
        if (part) part[(size_t)blockIdx.y * C + c] = t;
        else bias_put<DT>(db, c, t);
    }
}

// channels-last.  A workgroup takes CB channels (CV threads along them, V channels each) of a run of pixels
template <int DT, int V>
__global__ __launch_bounds__(kThreads) void bias_nhwc_kernel(const void *dY, float *part, void *db, long long npix, int C, int CV, long long len)
{
    typedef typename BiasElem<DT>::t elem_t;
    __shared__ float red[kThreads * V];
    const int tid = threadIdx.x, rows = kThreads / CV, row = tid / CV, cv = tid - row * CV;
    const int c0 = (blockIdx.x * CV + cv) * V;
    const long long p0 = blockIdx.y * len, p1 = std::min(p0 + len, npix);
    float acc[V];
#pragma unroll
    for (int v = 0; v < V; ++v) acc[v] = 0.f;
    if (row < rows && c0 < C) {
        constexpr int U = 4;
        for (long long p = p0 + row; p < p1; p += (long long)rows * U) {
            if constexpr (V > 1) {
                uint4 x[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const long long q = p + (long long)u * rows;
                    x[u] = q < p1 ? *reinterpret_cast<const uint4 *>(static_cast<const elem_t *>(dY) + (size_t)q * C + c0) : uint4{0, 0, 0, 0};
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    elem_t e[V];
                    __builtin_memcpy(e, &x[u], 16);
#pragma unroll
                    for (int v = 0; v < V; ++v) acc[v] += bias_val<DT>(e[v]);
                }
            } else {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const long long q = p + (long long)u * rows;
                    acc[0] += q < p1 ? bias_val<DT>(static_cast<const elem_t *>(dY)[(size_t)q * C + c0]) : 0.f;
                }
            }
        }
    }
#pragma unroll
    for (int v = 0; v < V; ++v) red[tid * V + v] = acc[v];
    __syncthreads();
    for (int i = tid; i < CV * V; i += kThreads) {
        const int c = blockIdx.x * CV * V + i;
        if (c >= C) continue;
        float s = 0.f;
        for (int r = 0; r < rows; ++r) s += red[r * CV * V + i];
        if (part) part[(size_t)blockIdx.y * C + c] = s;
        else bias_put<DT>(db, c, s);
    }
}

// pieces of a channel's values (planes) or of the pixels (channels-last): enough workgroups for two per compute unit, pieces
// of at least 32 KB
int bias_pieces(long long bytes, int groups)
{
    const long long most = std::max<long long>(1, bytes / (32 * 1024));
    return (int)std::max<long long>(1, std::min<long long>(std::min<long long>(most, 1024), 512 / std::max(1, groups)));
}

template <int DT>
hipError_t launch_bias_dt(const void *dY, float *part, void *db, int B, int C, int HW, bool nhwc, hipStream_t st, SideJobs *J)
{
    constexpr int V = DT == XCONV_F32 ? 4 : 8, ES = DT == XCONV_F32 ? 4 : 2;
    const bool al = (reinterpret_cast<uintptr_t>(dY) & 15u) == 0;
    int S;
    if (nhwc) {
        const long long npix = (long long)B * HW;
        const bool vec = al && C % V == 0;
        const int cv = std::min(kThreads, vec ? C / V : C), groups = ceil_div(vec ? C / V : C, cv);
        S = bias_pieces(npix * C * ES / groups, groups);
        const long long len = (npix + S - 1) / S;
        if (vec) hipLaunchKernelGGL((bias_nhwc_kernel<DT, V>), dim3(groups, S), dim3(kThreads), 0, st, dY, S > 1 ? part : nullptr, db, npix, C, cv, len);
        else hipLaunchKernelGGL((bias_nhwc_kernel<DT, 1>), dim3(groups, S), dim3(kThreads), 0, st, dY, S > 1 ? part : nullptr, db, npix, C, cv, len);
    } else {
        const bool vec = al && HW % V == 0;
        const int hwv = vec ? HW / V : HW;
        S = bias_pieces((long long)B * HW * ES, C);
        const long long len = ((long long)B * hwv + S - 1) / S;
        if (vec) hipLaunchKernelGGL((bias_planes_kernel<DT, true>), dim3(C, S), dim3(kThreads), 0, st, dY, S > 1 ? part : nullptr, db, B, C, hwv, len);
        else hipLaunchKernelGGL((bias_planes_kernel<DT, false>), dim3(C, S), dim3(kThreads), 0, st, dY, S > 1 ? part : nullptr, db, B, C, hwv, len);
    }
    hipError_t e = hipGetLastError();
    if (S == 1 || e != hipSuccess) return e;
    SideJobs alone{};
    SideJobs &q = J ? *J : alone;
    q.part = part; q.db = db; q.C = C; q.S = S; q.dtype = DT;
    q.total += C;
    return J ? hipSuccess : launch_side_jobs(alone, st);
}

}  // namespace

size_t bias_ws_bytes(int C) { return (size_t)C * 1024 * sizeof(float); }

hipError_t launch_bias_grad(int dtype, const void *dY, float *part, void *db, int B, int C, int HW, bool nhwc, hipStream_t st, SideJobs *J)
{
    if (dtype == XCONV_F32) return launch_bias_dt<XCONV_F32>(dY, part, db, B, C, HW, nhwc, st, J);
    if (dtype == XCONV_BF16) return launch_bias_dt<XCONV_BF16>(dY, part, db, B, C, HW, nhwc, st, J);
    return launch_bias_dt<XCONV_F16>(dY, part, db, B, C, HW, nhwc, st, J);
}

}  // namespace xc
