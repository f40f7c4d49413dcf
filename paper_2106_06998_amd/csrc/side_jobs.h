// Device side of SideJobs (common.h).
#pragma once
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace xc {

// Fragment i of a class: weights in the order [block of 32 output channels][chunk][tap][k-step][lane] of 16 bytes (a chunk =
// kConvUnits / 2 k-steps of channels, or all of them for resident patches); zero beyond the channels.  Floats are split: three
// times 64 lanes of 16 bytes a fragment, chunks of kConvUnitsSplit / 2 k-steps.
template <int ES, class SJ> __device__ inline void pack_fragment(const SJ &J, const PackClass &S, int i, int lane)
{
    constexpr int UE = 8, KS = (ES == 4 ? kConvUnitsSplit : kConvUnits) / 2;
    const int taps = S.kH * S.kW, nks = (J.Cin + 2 * UE - 1) / (2 * UE), nk = taps * nks;
    const int cks = J.res ? nks : KS;                         // k-steps of a full chunk
    const int mb = i / nk, k = i - mb * nk;
    const int ck = k / (taps * cks), r = k - ck * taps * cks;
    const int per = min(cks, nks - ck * cks), tap = r / per, s = r - tap * per;
    const int ky = tap / S.kW, kx = tap - ky * S.kW;
    const int co = mb * 32 + (lane & 31), u = 2 * (ck * cks + s) + (lane >> 5);
    const int c0 = u * UE;
    typedef typename std::conditional<ES == 4, float, uint16_t>::type elem_t;
    const elem_t *src = static_cast<const elem_t *>(J.w) + (size_t)co * J.w_sco + (S.ky0 + ky * S.kys) * J.kWfull + S.kx0 + kx * S.kxs;
    elem_t v[UE];
#pragma unroll
    for (int e = 0; e < UE; ++e) v[e] = co < J.Cout && c0 + e < J.Cin ? src[(size_t)(c0 + e) * J.w_sci] : elem_t(0);
    uint4 *out = static_cast<uint4 *>(J.packed) + S.w0 + (size_t)i * (ES == 4 ? kSplit * 64 : 64) + lane;
    if constexpr (ES == 4) {
        uint4 p[kSplit];
        split8_packed(v, p);
#pragma unroll
        for (int q = 0; q < kSplit; ++q) out[q * 64] = p[q];
    } else {
        *out = uint4{v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16), v[4] | ((uint32_t)v[5] << 16), v[6] | ((uint32_t)v[7] << 16)};
    }
}

// one wave adds the S pieces of channel c in a fixed order: lanes take the pieces lane, lane + 64, ...
template <class SJ> __device__ inline void bias_sum_channel(const SJ &J, int c, int lane)
{
    float s = 0.f;
    for (int i = lane; i < J.S; i += 64) s += J.part[(size_t)i * J.C + c];
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o);
    if (lane != 0) return;
    if (J.dtype == XCONV_F32) static_cast<float *>(J.db)[c] = s;
    else static_cast<uint16_t *>(J.db)[c] = J.dtype == XCONV_BF16 ? f32_to_st16<XCONV_BF16>(s) : f32_to_st16<XCONV_F16>(s);
}

// workgroup wg of nwg, of THREADS threads.  ES: bytes per element where the carrying kernel knows them, else 0
template <int ES, int THREADS, class SJ> __device__ inline void side_jobs(const SJ &J, int wg, int nwg)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(wg * (THREADS / 64) + (int)(threadIdx.x >> 6));
    for (int i = wave; i < J.total; i += nwg * (THREADS / 64)) {
        int q = i, c = 0;
        while (c < J.nsub && q >= J.sub[c].n) q -= J.sub[c++].n;
        if (c == J.nsub) bias_sum_channel(J, q, lane);
        else if (ES == 4 || (ES == 0 && J.es == 4)) pack_fragment<4>(J, J.sub[c], q, lane);
        else pack_fragment<2>(J, J.sub[c], q, lane);
    }
}

// In a kernel that may carry jobs (an empty pack or one SideJobs): does those of this workgroup, if it is one of theirs; number
// and count of the kernel's own workgroups along the grid
template <int ES, int THREADS> __device__ inline bool do_side_jobs(const SideJobs &J)
{
    if ((int)blockIdx.x >= J.groups) return false;
    if (blockIdx.y == 0) side_jobs<ES, THREADS>(J, blockIdx.x, J.groups);
    return true;
}
__device__ inline unsigned own_group() { return blockIdx.x; }
__device__ inline unsigned own_groups() { return gridDim.x; }
__device__ inline unsigned own_group(const SideJobs &J) { return blockIdx.x - J.groups; }
__device__ inline unsigned own_groups(const SideJobs &J) { return gridDim.x - J.groups; }

// workgroups that carry the jobs; a multiple of 8 keeps the dies of the others (xcd_block)
template <int THREADS, class SJ> inline int side_groups(const SJ *J)
{
    if (!J || J->total <= 0) return 0;
    const int n = (J->total + THREADS / 64 - 1) / (THREADS / 64);
    return (std::min(n, 1024) + 7) / 8 * 8;
}

}  // namespace xc
