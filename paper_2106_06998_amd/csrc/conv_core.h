// Forward convolution and exact input gradient of the layer (Sec. 2: XConv leaves the forward pass and
// the backpropagation through the layer exact; Algorithm 1 forward step 1 and the gradient with respect
// to the input):
//
//   forward      Y[b,m,oy,ox]  = sum_{n,ky,kx} W[m,n,ky,kx] X[b,n, oy*sh+ky-ph, ox*sw+kx-pw]
//   input grad   dX[b,n,iy,ix] = sum_{m,ky,kx} W[m,n,ky,kx] dY[b,m,oy,ox],  oy*sh+ky-ph = iy, ox*sw+kx-pw = ix
//
// Both are implicit GEMMs out[co, p] = sum_{tap, ci} W[co, ci, tap] * in[ci, src(p, tap)].  The input gradient of a
// strided layer is split by the remainder of the output position modulo the stride: each class is an ordinary
// unit-stride convolution with the taps that reach it (ConvSub), so no product with a structural zero is formed.
//
// Work split.  A workgroup of 4 waves owns TM = 32*MT*WM output channels x TN = 32*NT*(4/WM) output positions; a wave
// 32*MT x 32*NT of them as 32x32 accumulator tiles.  Positions are counted along strips of SW columns, row after row and
// image after image, so that small images fill a tile and wide ones give tiles of several short rows (a small halo).
// The input patch of a tile (its rows and columns with the halo, zero outside the image) is staged into LDS as
// [unit][position] (a unit = 16 bytes of channels: 8 at 16-bit storage, 4 at fp32) and serves all kernel taps from there:
// a tap only shifts the position a lane reads, so the input is read from memory about once instead of once per tap.
//   RES   all channels of the patch are resident: one staging phase, one barrier, then taps and channels without another
//         (up to kConvResident channels; the workgroups that share a compute unit cover each other's staging).  The
//         products of an output are summed tap by tap and, within a tap, by ascending channel.
//   !RES  chunks of kConvUnits units: the next chunk's patch is on its way through registers while the current one is multiplied
//         (two LDS buffers, one barrier per chunk).
// Floats with packed weights (conv_split) are multiplied on the 16-bit matrix cores, as sums of three bf16 numbers (split8, common.h): a
// patch holds three units for the one of the 16-bit types, split once as they are staged, the packed weights three fragments.  Six
// products of 32 cycles then do the work of eight fp32 ones of 64; they take 12 registers a fragment and twice the accumulators, which leaves
// room for one block of 32 channels a wave.  128 x 64 -> 64 channels 3x3 32x32: 98 -> 58 us (fp32 matrix instructions -> here), 64 x
// 256 -> 256 channels 28x28 521 -> 327, 8 x 64 -> 64 channels 256x256 321 -> 204, and the sums are three times closer to 64 bits.  A tile with
// sums that the pieces do not hold (split8) computes those on the fp32 instructions, from the same packed weights.
// Strided layers keep the patch columns split by their remainder modulo the stride, so that the lanes' reads stay consecutive.
// Weights come packed in fragment order (pack_fragment, one coalesced kilobyte per fragment, read through the L1 by
// every wave) or, without a workspace, are gathered from [C_out, C_in, kH, kW] through LDS, a group of k-steps at a time; patches are
// then chunks, as many units of one as there are channels for.
#pragma once
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "launch.h"

namespace xc {

namespace {

typedef float f32x16c __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4c __attribute__((ext_vector_type(4)));

// one 16-byte fragment pair: 32x32x16 at 16-bit storage, four 32x32x2 at fp32 (lanes 0-31 hold the first unit of a k-step,
// lanes 32-63 the second)
template <int DT> __device__ inline f32x16c conv_mma(const u32x4c &a, const u32x4c &b, f32x16c c)
{
    if constexpr (DT == XCONV_F32) {
#pragma unroll
        for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[e]), __uint_as_float(b[e]), c, 0, 0, 0);
        return c;
    } else if constexpr (DT == XCONV_BF16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    } else {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    }
}

// round to nearest even on the conversion instructions of the chip
template <int DT> __device__ inline uint16_t conv_round(float f)
{
    if constexpr (DT == XCONV_BF16) return __builtin_bit_cast(uint16_t, (__bf16)f);
    else return f32_to_f16_rne(f);
}

template <int DT> struct ConvElem { typedef uint16_t t; static constexpr int UE = 8, ES = 2; };
template <> struct ConvElem<XCONV_F32> { typedef float t; static constexpr int UE = 4, ES = 4; };

// channel (within a step) of element e of unit u.  fp32 products run two channels at a time, one from each unit of a k-step:
// with the even channels in one unit and the odd ones in the other they come in ascending order.  Channels-last tensors are
// read as whole units of four consecutive channels instead.
template <int UE, bool IL> __device__ inline int conv_unit_channel(int u, int e) { return IL ? (u >> 1) * 2 * UE + 2 * e + (u & 1) : u * UE + e; }

constexpr uint32_t kConvOob = 0x80000000u;   // byte offset past every buffer descriptor: the load returns zero

}  // namespace

// VEC: how a staging task reads `in`: 0 element by element (any strides), 1 pairs of columns (16-bit planes of even width),
//      2 whole units (channels-last, channels a multiple of the unit).
// SWAP: output positions in the rows of the accumulator tile (channels-last output: lanes along the channels), else in its columns.
// NC: most classes in one launch (above one, an index into the argument struct that is not a constant makes the compiler load every
//      argument where it is used: a launch of one class does without).
// PACKED: weights in fragment order; else GW waves along the output channels (P.WM).  BIG: 64-bit addresses (tensors beyond a 2 GiB buffer descriptor).
template <int DT, int VEC, bool SWAP, int MT, int NT, bool PACKED, bool BIG, bool RES, int NC, int GW>
__global__ __launch_bounds__(kThreads, conv_occupancy(MT, NT, conv_split(DT, PACKED), PACKED)) void conv_kernel(const ConvArgs<NC> P)
{
    typedef typename ConvElem<DT>::t elem_t;
    constexpr bool SPL = conv_split(DT, PACKED);                 // floats as three bf16 numbers each
    constexpr int NP = SPL ? kSplit : 1, CU = SPL ? kConvUnitsSplit : kConvUnits;   // pieces of a unit, units of a chunk
    constexpr int UE = SPL ? 8 : ConvElem<DT>::UE, ES = ConvElem<DT>::ES;
    constexpr int KS = CU / 2, CK = CU * UE;                     // k-steps and channels of a chunk (!RES)
    constexpr bool IL = DT == XCONV_F32 && !SPL && VEC != 2;     // units of a pair hold the even and the odd channels (conv_unit_channel)
    constexpr int VW = VEC == 1 ? 2 : 1;                         // columns per staging task
    constexpr int RW = VEC == 2 && !SPL ? 4 : UE;                // registers per staging task
    constexpr int G = (!RES ? (SPL ? 16 : 32) : SPL && MT * NT == 1 ? 32 : 64) / RW;           // staging tasks of a thread in flight

    extern __shared__ uint4 conv_lds[];
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    int id = xcd_block(blockIdx.x, gridDim.x);
    if (id >= P.nwg) return;
    int cls = 0;
    if constexpr (NC > 1) {
        // a tile of each class in turn: they read the same rows of `in` and write the same cache lines of `out`, which one L2 then
        // fetches once and puts together
        cls = id % P.nsub;
        id /= P.nsub;
        if (id >= P.sub[cls].wgs) return;
    }
    const ConvSub &S = P.sub[cls];
    int mtile, strip, tile;
    P.dNMT.divmod(id, id, mtile);
    S.dTPS.divmod(id, strip, tile);

    const int WN = 4 / P.WM, wm = wave % P.WM, wn = wave / P.WM;
    const int TN = 32 * NT * WN;
    const int npp_max = S.NPPmax;
    const int nks = (P.Cin + 2 * UE - 1) / (2 * UE);                            // k-steps of all channels
    const int NU = RES ? 2 * nks : PACKED ? CU : std::min(2 * nks, kConvUnits);   // units of a staged patch
    uint4 *patch = conv_lds;                                                    // [1 or 2][NU][NP][NPOS]
    const int patch_units = (RES || (!PACKED && nks <= KS) ? 1 : 2) * NU * NP * S.NPOS;
    uint2 *ptab = reinterpret_cast<uint2 *>(conv_lds + patch_units);             // [NPPmax] {source byte offset, LDS positions}
    uint2 *otab = ptab + npp_max;                                               // [TN] {output offset, LDS position of tap (0, 0)}
    uint4 *stab = conv_lds + patch_units + (npp_max + TN + 1) / 2;           // PACKED: LDS offsets of the k-steps' fragments, two lists
    uint2 *gtab = reinterpret_cast<uint2 *>(stab);                              // !PACKED: per k-step {LDS offset | step of its tap, weight offset}, two lists

    // ---- the tile: positions q0 .. q0 + TU - 1 of this strip (TU < TN where the patch of TN would not fit into LDS), rows R0 .. R1 counted over the batch
    const int TU = S.TU, NR = P.B * S.Ho;
    int R0, x0, b0, oyA;
    S.dSW.divmod(tile * TU, R0, x0);       // tile * TU below 2^31 (host)
    int R1 = R0 + S.dSW.div(x0 + TU - 1);
    R1 = R1 < NR - 1 ? R1 : NR - 1;
    S.dHo.divmod(R0, b0, oyA);
    const int b1 = S.dHo.div(R1);
    const int NPR = (R1 - R0) * S.sth + (b1 - b0) * (S.kH - S.sth) + S.kH;      // staged rows of this tile
    const int xs = strip * S.SW * P.sw - S.pw;                                  // source column of patch column `xa`
    const int xa = VW == 2 ? (xs & 1) : 0;
    const int npp = NPR * S.PWv;

    {
        for (int pp = tid; pp < npp; pp += kThreads) {
            int prow, pc, bi, l;
            S.dPWv.divmod(pp, prow, pc);
            S.dHV.divmod(oyA * S.sth + prow, bi, l);
            const int c = pc * VW;
            const int iy = (S.kH >= P.sh ? l : (l / S.kH) * P.sh + l % S.kH) - S.ph;
            const int ix = xs - xa + (S.kW >= P.sw ? c : (c / S.kW) * P.sw + c % S.kW);
            const bool ok = b0 + bi < P.B && (unsigned)iy < (unsigned)P.Hi && (unsigned)ix < (unsigned)P.Wi;
            const uint32_t off = (uint32_t)bi * (uint32_t)P.in_sb + (uint32_t)iy * (uint32_t)P.in_sy + (uint32_t)ix * (uint32_t)P.in_sx;
            int p0 = prow * S.PWs + c, p1 = p0 + 1;
            if (S.stw != 1) {
                p0 = prow * S.PWs + (c % S.stw) * S.PH + c / S.stw;
                p1 = prow * S.PWs + ((c + 1) % S.stw) * S.PH + (c + 1) / S.stw;
            }
            ptab[pp] = uint2{ok ? (BIG ? off : off * ES) : (BIG ? 0xffffffffu : kConvOob), (uint32_t)p0 | ((uint32_t)p1 << 16)};
        }
        for (int n = tid; n < TN; n += kThreads) {
            int dr, x, bi, oy;
            S.dSW.divmod(x0 + n, dr, x);
            const int row = R0 + dr, ox = strip * S.SW + x;
            S.dHo.divmod(oyA + dr, bi, oy);
            const bool in_batch = row < NR && n < TU, ok = in_batch && ox < S.Wo;
            const uint32_t off = (uint32_t)bi * (uint32_t)P.out_sb + (uint32_t)(S.oy0 + oy * P.osy) * (uint32_t)P.out_sy +
                                 (uint32_t)(S.ox0 + ox * P.osx) * (uint32_t)P.out_sx;
            const int pr = dr * S.sth + bi * (S.kH - S.sth);
            otab[n] = uint2{ok ? (BIG ? off : off * ES) : (BIG ? 0xffffffffu : kConvOob), (uint32_t)(in_batch ? pr * S.PWs + x : 0)};
        }
    }
    const int taps = S.kH * S.kW;
    const int nck = RES ? 1 : (P.Cin + CK - 1) / CK;
    auto tap_offset = [&](int ky, int kx) {
        const int cy = P.rev ? S.kH - 1 - ky : ky, cx = (P.rev ? S.kW - 1 - kx : kx) + xa;
        return cy * S.PWs + (S.stw == 1 ? cx : (cx % S.stw) * S.PH + cx / S.stw);
    };
    // Byte offset of k-step i's fragment from that of the first tap's first: list 0 for a resident patch or a full chunk, list 1
    // for the last chunk.  One 16-byte read serves four steps, so the loop over the steps has no index arithmetic of its own.
    const int nks_last = RES ? nks : nks - (nck - 1) * KS;
    const int n_full = taps * (RES ? nks : KS), n_last = taps * nks_last;
    const int cap0 = !PACKED && nck > 1 ? (n_full + 7) / 8 * 8 : 0, cap1 = (n_last + 7) / 8 * 8;   // !PACKED: entries of the lists, whole groups
    uint4 *alds = stab + (cap0 + cap1) / 2;                                     // !PACKED: [2][steps of a group][MT * WM][64] weight fragments
    if constexpr (!PACKED) {
        for (int i = tid; i < cap0 + cap1; i += kThreads) {
            const int list = i >= cap0 ? 1 : 0, k = i - list * cap0, ks = k / taps, tap = k - ks * taps;
            int ky, kx;
            S.dkW.divmod(tap, ky, kx);
            gtab[i] = ks < (list ? nks_last : KS) ? uint2{(uint32_t)((tap_offset(ky, kx) + 2 * ks * S.NPOS) * 16 + ks),
                                                  (uint32_t)((S.ky0 + ky * S.kys) * P.kWfull + S.kx0 + kx * S.kxs + ks * 2 * UE * P.w_sci)}
                                          : uint2{0, kConvOob};
        }
    }
    if constexpr (PACKED) {
        int *t = reinterpret_cast<int *>(stab);
        const int cap = conv_step_list(taps, RES ? nks : KS) * 4;
        for (int i = tid; i < (RES ? cap : 2 * cap); i += kThreads) {
            const int list = i >= cap ? 1 : 0, k = i - list * cap;
            int tap, ks, ky, kx;
            (list ? P.dksl : P.dks).divmod(k, tap, ks);
            S.dkW.divmod(tap, ky, kx);
            t[i] = tap < taps ? (tap_offset(ky, kx) + 2 * ks * NP * S.NPOS) * 16 : 0;
        }
    }
    __syncthreads();

    const elem_t *in_b = static_cast<const elem_t *>(P.in) + (size_t)b0 * P.in_sb;
    const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(in_b), 0, (int)kConvOob, 0x00020000);

    // ---- staging: task t = (unit, position); a phase of a chunk is G tasks of every thread
    const int ntask = npp * NU;
    const float rnpp = frcp(VEC == 2 ? NU : npp);
    uint32_t sr[G][RW];
    auto split = [&](int t, int &u, int &pp) {
        if constexpr (VEC == 2) fast_divmod(t, NU, rnpp, pp, u);
        else fast_divmod(t, npp, rnpp, u, pp);
    };
    auto stage_load = [&](int c0, int phase) {
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int t = tid + kThreads * (phase * G + i);
            if (t < ntask) {
                int u, pp;
                split(t, u, pp);
                const uint32_t off = ptab[pp].x;
                if constexpr (BIG) {
                    const elem_t *src = in_b + (size_t)off;
#pragma unroll
                    for (int e = 0; e < UE; ++e) {
                        const int c = c0 + conv_unit_channel<UE, IL>(u, e);
                        elem_t v = elem_t(0);
                        if (off != 0xffffffffu && c < P.Cin) v = src[(size_t)c * (size_t)P.in_sc];
                        sr[i][e] = ES == 4 ? __builtin_bit_cast(uint32_t, (float)v) : (uint32_t)v;
                    }
                } else if constexpr (VEC == 2 && SPL) {
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const uint32_t vo = c0 + u * UE + 4 * q < P.Cin ? off + (uint32_t)u * 32u + 16u * q : kConvOob;
                        const u32x4c v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)vo, c0 * ES, 0);
#pragma unroll
                        for (int e = 0; e < 4; ++e) sr[i][4 * q + e] = v[e];
                    }
                } else if constexpr (VEC == 2) {
                    const uint32_t vo = c0 + u * UE < P.Cin ? off + (uint32_t)u * 16u : kConvOob;
                    const u32x4c v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)vo, c0 * ES, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) sr[i][e] = v[e];
                } else {
                    const uint32_t cs = (uint32_t)P.in_sc * ES;             // bytes from a channel to the next
                    const int cu = conv_unit_channel<UE, IL>(u, 0), left = P.Cin - c0 - cu;
                    uint32_t first = (uint32_t)cu * cs;
                    // (a multiply-add has 64 bits and reads a neighbour of `off`, which may be on its way from memory: waits between the loads,
                    // C2's products 64.1 us for 62.9)
                    if constexpr (SPL) asm("" : "+v"(first));
                    const uint32_t vo = off + first;
                    constexpr int step = IL ? 2 : 1;
                    auto load = [&](auto part) {
#pragma unroll
                        for (int e = 0; e < UE; ++e) {
                            const int v = (int)(!decltype(part)::value || e * step < left ? vo : kConvOob), so = (int)((uint32_t)(c0 + e * step) * cs);
                            if constexpr (VEC == 1 || ES == 4) sr[i][e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, v, so, 0);
                            else sr[i][e] = __builtin_amdgcn_raw_buffer_load_b16(rsrc, v, so, 0);
                        }
                    };
                    if (c0 + NU * UE <= P.Cin) load(std::false_type{});
                    else load(std::true_type{});
                }
            }
        }
    };
    auto stage_write = [&](int buf, int phase) {
        uint4 *dst = patch + (size_t)buf * NU * NP * S.NPOS;
#pragma unroll
        for (int i = 0; i < G; ++i) {
            const int t = tid + kThreads * (phase * G + i);
            if (t < ntask) {
                int u, pp;
                split(t, u, pp);
                const uint32_t pos = ptab[pp].y;
                uint4 *d = dst + (size_t)u * NP * S.NPOS;
                if constexpr (SPL) {
                    float v[8];
                    uint4 piece[kSplit];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = __uint_as_float(sr[i][e]);
                    split8(v, piece);
#pragma unroll
                    for (int q = 0; q < kSplit; ++q) d[q * S.NPOS + (pos & 0xffffu)] = piece[q];
                } else if constexpr (VEC == 1) {
                    uint32_t rows[8][1];
                    uint4 cols[2];
#pragma unroll
                    for (int e = 0; e < 8; ++e) rows[e][0] = sr[i][e];
                    transpose_rows8<1>(rows, cols);
                    d[pos & 0xffffu] = cols[0];
                    d[pos >> 16] = cols[1];
                } else if constexpr (VEC == 2 || ES == 4) {
                    d[pos & 0xffffu] = uint4{sr[i][0], sr[i][1], sr[i][2], sr[i][3]};
                } else {
                    d[pos & 0xffffu] = uint4{sr[i][0] | (sr[i][1] << 16), sr[i][2] | (sr[i][3] << 16), sr[i][4] | (sr[i][5] << 16),
                                             sr[i][6] | (sr[i][7] << 16)};
                }
            }
        }
    };
    const int nphase = (ntask + kThreads * G - 1) / (kThreads * G);

    // split floats: the products h*h in a sum of their own, so that the five smaller ones do not round it (sums of 576 terms are off
    // by 1.3e-7 of their norm; 4.2e-7 on the fp32 matrix instructions)
    constexpr int NS = SPL ? 2 : 1;
    f32x16c accs[NS][MT][NT];
    auto &acc = accs[0];
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 16; ++e) accs[q][mt][nt][e] = 0.f;

    const int co_w = (mtile * P.WM + wm) * (32 * MT);    // first output channel of this wave
    int pos[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) pos[nt] = ((int)otab[(wn * NT + nt) * 32 + l32].y + h * NP * S.NPOS) * 16;   // bytes

    // ---- packed weight fragments: one kilobyte per k-step and 32 output channels, in the order of the k-steps
    const int nk = taps * nks;
    const char *apk[MT];
    if constexpr (PACKED) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            int mb = co_w / 32 + mt;
            mb = mb < P.NMB ? mb : P.NMB - 1;
            apk[mt] = static_cast<const char *>(P.wp) + ((size_t)S.w0 + (size_t)mb * nk * (64 * NP)) * 16;
        }
    }
    const uint32_t lane16 = (uint32_t)lane * 16u;
    // Without packed weights the workgroup gathers the fragments of a group of k-steps through LDS, one barrier each, the elements
    // of the next group on their way in registers.  A group has as many steps as 4096 (fp32: 2048) elements make, 16 (8) for each
    // thread: 8 for a tile of 32 output channels, 2 for 128.  The steps of a chunk run through the kernel offsets of one pair of
    // units, then of the next: the weights of a channel lie next to each other, and a layer of few channels fills its groups with
    // several offsets.  (A group per kernel offset, for chunks of kConvUnits units whatever the channels: 3 -> 64 channels 7x7 at
    // stride 4, 224x224, batch 16, bf16, took 1970 us, now 43; 16 -> 16 channels 3x3, 32x32, batch 4, fp32, 21 us, now 9.8.)
    constexpr int NEL = PACKED ? 1 : kConvGatherM * CK / kThreads;
    elem_t wg[NEL];
    const elem_t *wraw = static_cast<const elem_t *>(P.w);
    constexpr int TMW = 32 * MT * GW, KG = std::max(1, KS * kConvGatherM / TMW), SG = std::min(KS, KG);   // output channels of the tile, k-steps of a group and of a block
    const int co_t = mtile * TMW;
    const bool along = !P.rev;    // lanes along the inner channel index of the weights: the contraction channels, or (input gradient) the output channels
    // element i of a thread: output channel gc + i * gcs of the tile or, the other way round, channel gk + i * gks of the group's
    // steps; both divide 32 and 2 * UE, so that an offset is the thread's own plus one of the element.  Channels past the last of
    // the outer index lie behind the end of the weights, where the descriptor ends; those of the inner one are masked
    const int gk = along ? tid & (KG * 2 * UE - 1) : tid / TMW, gc = along ? tid / (KG * 2 * UE) : tid & (TMW - 1);
    constexpr int gks = kThreads / TMW, gcs = kThreads / (KG * 2 * UE);
    const uint32_t gw = ((uint32_t)(along ? gk % (2 * UE) : gk) * (uint32_t)P.w_sci + (uint32_t)gc * (uint32_t)P.w_sco) * ES;
    const int gd = ((along ? gk / (2 * UE) : 0) * MT * GW * 64 + (IL ? gk & 1 : gk / UE % 2) * 32 + gc / 32 * 64 + gc % 32) * UE +
                   (IL ? gk % (2 * UE) / 2 : gk % UE);
    auto gather_load = [&](const uint2 *list, int c0, int g) {
        const size_t first = (size_t)c0 * P.w_sci + (size_t)co_t * P.w_sco, all = std::max((size_t)P.w_sci * P.Cin, (size_t)P.w_sco * P.Cout);
        const auto wsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<elem_t *>(wraw + first), 0,
                                                            (int)std::min((all - first) * ES, (size_t)kConvOob - 1), 0x00020000);
        auto load = [&](uint32_t off) -> elem_t {
            if constexpr (ES == 4) return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(wsrc, (int)off, 0, 0));
            else return (elem_t)__builtin_amdgcn_raw_buffer_load_b16(wsrc, (int)off, 0, 0);
        };
        if (along) {
            const uint2 e = list[g * KG + gk / (2 * UE)];
            const bool on = e.y != kConvOob && c0 + (int)(e.x & 15u) * 2 * UE + gk % (2 * UE) < P.Cin;
            const uint32_t off = on ? gw + e.y * ES : kConvOob;
#pragma unroll
            for (int i = 0; i < NEL; ++i) wg[i] = load(off + (uint32_t)(i * gcs) * (uint32_t)P.w_sco * ES);
        } else {
            const uint32_t off = co_t + gc < P.Cout ? gw : kConvOob;
#pragma unroll
            for (int i = 0; i < NEL; ++i) {
                const uint32_t o = (uint32_t)__builtin_amdgcn_readfirstlane((int)list[g * KG + i * gks / (2 * UE)].y);
                wg[i] = load(o == kConvOob ? kConvOob : off + (o + (uint32_t)(i * gks % (2 * UE)) * (uint32_t)P.w_sci) * ES);
            }
        }
    };
    auto gather_write = [&](int buf) {
        elem_t *d = reinterpret_cast<elem_t *>(alds + buf * KG * MT * GW * 64) + gd;
        if (along) {
#pragma unroll
            for (int i = 0; i < NEL; ++i) d[(i * gcs / 32 * 64 + i * gcs % 32) * UE] = wg[i];
        } else {
#pragma unroll
            for (int i = 0; i < NEL; ++i) {
                constexpr int W = 2 * UE;
                const int x = i * gks % W;
                d[(i * gks / W * MT * GW * 64 + (IL ? 0 : x / UE) * 32) * UE + (IL ? x / 2 : x % UE)] = wg[i];
            }
        }
    };
    // ---- k-steps.  Weights are requested kAhead k-steps ahead (they come from the L2), patch fragments one step ahead, both in
    // front of the step's matrix instructions (sched_barrier: left alone, the compiler reads each fragment right before its
    // use and waits).  Four steps make a block (two of split floats, six products of each tile and three times the registers a step,
    // but for the smallest tile), so that the rings are indexed by constants.
    constexpr int kRing = SPL && !(RES && MT * NT == 1) ? 2 : 4, kAhead = kRing - 1;
    static_assert(KS % kRing == 0 || RES, "a full chunk is whole blocks");
    u32x4c a[kRing][MT][NP], b[2][NT][NP];
    auto load_a = [&](auto slot) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
#pragma unroll
            for (int q = 0; q < NP; ++q) a[decltype(slot)::value][mt][q] = *reinterpret_cast<const u32x4c *>(apk[mt] + lane16 + 1024 * q);
            apk[mt] += 1024 * NP;
        }
    };
    const char *patch_b = reinterpret_cast<const char *>(patch);
    const int piece = S.NPOS * 16;
    auto load_b = [&](auto slot, int off) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int q = 0; q < NP; ++q) b[decltype(slot)::value][nt][q] = *reinterpret_cast<const u32x4c *>(patch_b + (pos[nt] + off + q * piece));
    };
    auto multiply = [&](auto as, auto bs) {
#pragma unroll
        for (int p = 0; p < (SPL ? kSplitProducts : 1); ++p)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const u32x4c &av = a[decltype(as)::value][mt][SPL ? kSplitA[p] : 0], &bv = b[decltype(bs)::value][nt][SPL ? kSplitB[p] : 0];
                    constexpr int T = SPL ? XCONV_BF16 : DT;
                    f32x16c &c = accs[SPL && kSplitA[p] + kSplitB[p] > 0 ? 1 : 0][mt][nt];
                    c = SWAP ? conv_mma<T>(bv, av, c) : conv_mma<T>(av, bv, c);
                }
    };
    auto step = [&](auto jc, int next_off) {
        constexpr int j = decltype(jc)::value;
        load_b(std::integral_constant<int, (j + 1) & 1>{}, next_off);
        load_a(std::integral_constant<int, (j + kAhead) % kRing>{});
        // 16-bit chunks of the larger tiles: behind each matrix instruction a read of a fragment, a request for weights and two vector
        // instructions (addresses), which it hides (products of C5, rocprofv3: 260 -> 249 us); elsewhere they all go in front
        constexpr bool spread = !SPL && !RES && PACKED && DT != XCONV_F32 && MT * NT >= 4;
        if constexpr (!spread) __builtin_amdgcn_sched_barrier(0);
        multiply(std::integral_constant<int, j>{}, std::integral_constant<int, j & 1>{});
        if constexpr (spread) {
#pragma unroll
            for (int m = 0; m < MT * NT; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 2, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // blocks b0 .. b1-1 of a list, and the rest of n steps behind the last whole block when `tail`
    typedef std::conditional_t<kRing == 4, int4, int2> offsets_t;
    offsets_t so;
    auto first_block = [&](const uint4 *list, int base) {
        so = reinterpret_cast<const offsets_t *>(list)[0];
        load_b(std::integral_constant<int, 0>{}, base + so.x);
    };
    auto run_blocks = [&](const uint4 *list, int base, int blk0, int blk1) {
        for (int i = blk0; i < blk1; ++i) {
            const offsets_t sn = reinterpret_cast<const offsets_t *>(list)[i + 1];
            step(std::integral_constant<int, 0>{}, base + so.y);
            if constexpr (kRing == 4) {
                step(std::integral_constant<int, 1>{}, base + so.z);
                step(std::integral_constant<int, 2>{}, base + so.w);
            }
            step(std::integral_constant<int, kRing - 1>{}, base + sn.x);
            so = sn;
        }
    };
    auto run_tail = [&](int base, int left) {
        if (left > 0) step(std::integral_constant<int, 0>{}, base + so.y);
        if constexpr (kRing == 4) {
            if (left > 1) step(std::integral_constant<int, 1>{}, base + so.z);
            if (left > 2) step(std::integral_constant<int, 2>{}, base + so.w);
        }
    };

    if (nck > 0) {
        if constexpr (PACKED) {
            // Chunks: in the order of the steps, since loads complete in order and what the loop waits for counts those behind it.
            // (A resident patch is waited for in front of its loop, and its loads had better not queue behind these: the input
            // gradient of 256 -> 64 channels 1x1 56x56, batch 64, bf16 took 44 us with the order kept, 42 without.)
            load_a(std::integral_constant<int, 0>{});
            if constexpr (!RES) __builtin_amdgcn_sched_barrier(0);
            if constexpr (kAhead > 1) {
                load_a(std::integral_constant<int, 1>{});
                if constexpr (!RES) __builtin_amdgcn_sched_barrier(0);
                load_a(std::integral_constant<int, 2>{});
                if constexpr (!RES) __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            gather_load(nck > 1 ? gtab : gtab + cap0, 0, 0);
            gather_write(0);
        }
        for (int ph = 0; ph < nphase; ++ph) {
            stage_load(0, ph);
            stage_write(0, ph);
            // vmcnt(0): for the compiler, a branch of stage_write that is not taken leaves loads in flight, whose registers it waits for
            // between the loads of the next phase (C2's products 66.4 us without this wait, 62.9 with it)
            if constexpr (SPL) __builtin_amdgcn_s_waitcnt(0x0f70);
        }
        __syncthreads();
        if constexpr (RES) {
            first_block(stab, 0);
            run_blocks(stab, 0, 0, n_full / kRing);
            run_tail(0, n_full % kRing);
        } else if constexpr (PACKED) {
            const uint4 *list1 = stab + conv_step_list(taps, KS);
            for (int ck = 0; ck < nck; ++ck) {
                const bool more = ck + 1 < nck;
                const uint4 *list = more ? stab : list1;
                const int nblk = (more ? n_full : n_last) / kRing, base = (ck & 1) * NU * NP * S.NPOS * 16;
                first_block(list, base);
                for (int ph = 0; ph < nphase; ++ph) {
                    if (more) stage_load((ck + 1) * CK, ph);
                    run_blocks(list, base, nblk * ph / nphase, nblk * (ph + 1) / nphase);
                    if (more) stage_write((ck + 1) & 1, ph);
                }
                __syncthreads();
            }
            // behind the loop: with a path from the tail back into the blocks (a ring that is one or two steps further), the
            // compiler would have every block wait for all but the last step's weights
            run_tail(((nck - 1) & 1) * NU * NP * S.NPOS * 16, n_last % kRing);
        } else {
            int abuf = 0;
            for (int ck = 0; ck < nck; ++ck) {
                const int c0 = ck * CK;
                const bool more = ck + 1 < nck;
                const int base = (ck & 1) * NU * S.NPOS * 16, n = more ? n_full : n_last, ng = (n + KG - 1) / KG;
                const uint2 *list = more ? gtab : gtab + cap0;
                int g = 0;
                for (int ph = 0; ph < nphase; ++ph) {
                    if (more) stage_load(c0 + CK, ph);
                    for (const int gend = ng * (ph + 1) / nphase; g < gend; ++g) {
                        const bool next = g + 1 < ng || more;
                        if (g + 1 < ng) gather_load(list, c0, g + 1);
                        else if (more) gather_load(ck + 2 < nck ? gtab : gtab + cap0, c0 + CK, 0);
                        for (int q = 0; q < KG; q += SG) {
                            const int left = n - (g * KG + q);      // (a step past the last has weights of zero, but the patch may hold infinities)
                            const uint2 *l = list + g * KG + q;
                            const u32x4c *af = reinterpret_cast<const u32x4c *>(alds) + ((abuf * KG + q) * GW + wm) * MT * 64 + lane;
#pragma unroll
                            for (int j = 0; j < SG; ++j)
#pragma unroll
                                for (int mt = 0; mt < MT; ++mt) a[j][mt][0] = af[(j * GW * MT + mt) * 64];
                            auto off = [&](int j) { return base + (int)(l[j].x & ~15u); };
                            load_b(std::integral_constant<int, 0>{}, off(0));
                            load_b(std::integral_constant<int, 1>{}, off(1));
                            if (left > 0) multiply(std::integral_constant<int, 0>{}, std::integral_constant<int, 0>{});
                            if constexpr (SG > 2) load_b(std::integral_constant<int, 0>{}, off(2));
                            if (left > 1) multiply(std::integral_constant<int, 1>{}, std::integral_constant<int, 1>{});
                            if constexpr (SG > 2) {
                                load_b(std::integral_constant<int, 1>{}, off(3));
                                if (left > 2) multiply(std::integral_constant<int, 2>{}, std::integral_constant<int, 0>{});
                                if (left > 3) multiply(std::integral_constant<int, 3>{}, std::integral_constant<int, 1>{});
                            }
                        }
                        abuf ^= 1;
                        if (next) gather_write(abuf);
                        __syncthreads();
                    }
                    if (more) stage_write((ck + 1) & 1, ph);
                }
                __syncthreads();
            }
        }
    }

    uint32_t again = 0;          // split floats: a bit for each sum that has to be computed again
    if constexpr (SPL) {
        // The sums, scaled back.  One that is no finite number, with a factor or a sum beyond what the pieces hold (split8), is computed
        // once more on the fp32 matrix instructions: the tile's patch again, as floats, and the packed weights put together again.  So are sums
        // of one or two products, which round so seldom that what a product leaves out shows (largest error, in terms of the products: 1.4 times that
        // of fp32; with three 0.93, with 64 0.33).  The waves vote behind their stores, where they have nothing else to wait for; what
        // they stored is then stored again.
        static_assert(MT * NT <= 2, "one bit for each sum");
        float odd_sum = 0.f;       // NaN as soon as one of them is not finite
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                acc[0][nt][e] = (acc[0][nt][e] + accs[NS - 1][0][nt][e]) * kSplitUnscale;
                odd_sum = fmaf(acc[0][nt][e], 0.f, odd_sum);
            }
        again = taps * P.Cin <= 2 ? 0xffffffffu : 0u;
        if (odd_sum != 0.f) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    // (positions that are not stored may have read what was never staged)
                    const int n = (wn * NT + nt) * 32 + (SWAP ? 8 * (e / 4) + 4 * h + e % 4 : l32);
                    if (otab[n].x != kConvOob && !(fabsf(acc[0][nt][e]) < __builtin_inff())) again |= 1u << (nt * 16 + e);
                }
        }
    }

    // ---- accumulator tile: lane l holds column l % 32 and rows 8*(i/4) + 4*(l/32) + i%4, rounded once to the storage type.
    // The bias is added to the rounded product, in fp32, and the sum rounded again: what a separate addition gives, bit for
    // bit (a sum rounded once falls on the other side of zero now and then, which a ReLU behind the layer would show).
    elem_t *out_b = static_cast<elem_t *>(P.out) + (size_t)b0 * P.out_sb;
    const elem_t *bias = static_cast<const elem_t *>(P.bias);
    auto bias_of = [&](int co) {
        if (co >= P.Cout) return 0.f;
        if constexpr (ES == 4) return bias[co];
        else return st16_to_f32<DT>(bias[co]);
    };
    auto add_bias = [](float v, float bv) {
        if constexpr (ES == 4) return v + bv;
        else return st16_to_f32<DT>(conv_round<DT>(v)) + bv;
    };
    auto stored = [](float v) -> elem_t {
        if constexpr (ES == 4) return v;
        else return conv_round<DT>(v);
    };
    // byte offsets in a 2 GiB descriptor: per lane the position and its first channel, per register a scalar
    const auto orsrc = __builtin_amdgcn_make_buffer_rsrc(out_b, 0, (int)kConvOob, 0x00020000);
    const uint32_t cs = (uint32_t)P.out_sc * ES;
    const uint32_t odd = (uint32_t)lane & 1u;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        const int cb = co_w + mt * 32;          // channels cb .. cb + 31
        if (cb >= P.Cout) break;
        const bool full = cb + 32 <= P.Cout;
        if (bias) {
            float bv[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) bv[i] = bias_of(SWAP ? cb + l32 : cb + 8 * (i / 4) + 4 * h + i % 4);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mt][nt][i] = add_bias(acc[mt][nt][i], bv[i]);
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if constexpr (BIG) {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int r = 8 * (i / 4) + 4 * h + i % 4, co = cb + (SWAP ? l32 : r);
                    const uint32_t off = otab[(wn * NT + nt) * 32 + (SWAP ? r : l32)].x;
                    if (off != 0xffffffffu && co < P.Cout) out_b[(size_t)off + (size_t)co * (size_t)P.out_sc] = stored(acc[mt][nt][i]);
                }
            } else if (ES == 2 && P.pair) {
                // neighbouring lanes exchange halves: the even one stores two neighbours of register i, the odd one of register i + 1
                const uint32_t sel = odd ? 0x03020706u : 0x05040100u;
                auto both = [&](int i) {
                    const uint32_t p = (uint32_t)stored(acc[mt][nt][i]) | ((uint32_t)stored(acc[mt][nt][i + 1]) << 16);
                    const uint32_t q = (uint32_t)__builtin_amdgcn_mov_dpp((int)p, 0xB1, 0xF, 0xF, true);    // lane ^ 1
                    return __builtin_amdgcn_perm(q, p, sel);
                };
                if constexpr (SWAP) {
                    const uint32_t lo = (uint32_t)(l32 & ~1) * 2u;
                    const bool on = cb + l32 < P.Cout;
#pragma unroll
                    for (int i = 0; i < 16; i += 2) {
                        const uint2 *e = otab + (wn * NT + nt) * 32 + 8 * (i / 4) + 4 * h + i % 4;
                        const uint32_t off = e[odd].x;
                        __builtin_amdgcn_raw_buffer_store_b32(both(i), orsrc, (int)(on ? off + lo : kConvOob), cb * 2, 0);
                    }
                } else {
                    const uint32_t off = otab[(wn * NT + nt) * 32 + l32].x;
                    const uint32_t vo = off == kConvOob ? off : off + (4u * h + odd) * cs - odd * 2u;
#pragma unroll
                    for (int i = 0; i < 16; i += 2) {
                        const int r = 8 * (i / 4) + i % 4;      // + 4 * h + odd
                        const uint32_t v = full || cb + r + 4 * h + (int)odd < P.Cout ? vo : kConvOob;
                        __builtin_amdgcn_raw_buffer_store_b32(both(i), orsrc, (int)v, (int)((uint32_t)(cb + r) * cs), 0);
                    }
                }
            } else {
                const uint32_t lo = SWAP ? (uint32_t)l32 * cs : (uint32_t)(4 * h) * cs;
                const uint32_t offl = otab[(wn * NT + nt) * 32 + l32].x;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int r = 8 * (i / 4) + i % 4;          // + 4 * h
                    const uint32_t off = SWAP ? otab[(wn * NT + nt) * 32 + r + 4 * h].x : offl;
                    const bool on = full || cb + (SWAP ? l32 : r + 4 * h) < P.Cout;
                    const int vo = (int)(on && off != kConvOob ? off + lo : kConvOob), so = (int)((uint32_t)(SWAP ? cb : cb + r) * cs);
                    const elem_t v = stored(acc[mt][nt][i]);
                    if constexpr (ES == 4) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), orsrc, vo, so, 0);
                    else __builtin_amdgcn_raw_buffer_store_b16((short)v, orsrc, vo, so, 0);
                }
            }
        }
    }

    if constexpr (SPL) {
        auto &exact = accs[NS - 1];
        const int vote = __ballot(again != 0) != 0;
        auto barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };      // (__syncthreads waits for the stores)
        int *votes = reinterpret_cast<int *>(conv_lds);
        barrier();                 // all have read their last patch
        if (lane == 0) votes[wave] = vote;
        barrier();
        if ((votes[0] | votes[1] | votes[2] | votes[3]) == 0) return;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            apk[mt] = static_cast<const char *>(P.wp) + ((size_t)S.w0 + (size_t)std::min(co_w / 32 + mt, P.NMB - 1) * nk * (64 * NP)) * 16;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 16; ++e) exact[mt][nt][e] = 0.f;
        }
        for (int ck = 0; ck < nck; ++ck) {
            __syncthreads();
            // two units of four floats in the places of the first two pieces
            for (int t = tid; t < ntask; t += kThreads) {
                int u, pp;
                split(t, u, pp);
                const uint2 at = ptab[pp];
                const int c0 = ck * CK + u * UE;
                uint32_t v[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    v[e] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, (int)(at.x != kConvOob && c0 + e < P.Cin ? at.x + (uint32_t)(c0 + e) * ((uint32_t)P.in_sc * ES) : kConvOob), 0, 0);
                uint4 *d = patch + (size_t)u * NP * S.NPOS + (at.y & 0xffffu);
                d[0] = uint4{v[0], v[1], v[2], v[3]};
                d[S.NPOS] = uint4{v[4], v[5], v[6], v[7]};
            }
            __syncthreads();
            const bool more = ck + 1 < nck;
            const int *list = reinterpret_cast<const int *>(RES || more ? stab : stab + conv_step_list(taps, KS));
            for (int i = 0; i < (more ? n_full : n_last); ++i) {
                u32x4c b0[NT], b1[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    b0[nt] = *reinterpret_cast<const u32x4c *>(patch_b + (pos[nt] + list[i]));
                    b1[nt] = *reinterpret_cast<const u32x4c *>(patch_b + (pos[nt] + list[i] + piece));
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    u32x4c w[NP];
#pragma unroll
                    for (int q = 0; q < NP; ++q) w[q] = *reinterpret_cast<const u32x4c *>(apk[mt] + lane16 + 1024 * q);
                    apk[mt] += 1024 * NP;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const float a = e & 1 ? joined_high(w[0][e / 2], w[1][e / 2], w[NP - 1][e / 2]) : joined_low(w[0][e / 2], w[1][e / 2], w[NP - 1][e / 2]);
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt) {
                            const float b = __uint_as_float(e < 4 ? b0[nt][e & 3] : b1[nt][e & 3]);
                            exact[mt][nt] = SWAP ? __builtin_amdgcn_mfma_f32_32x32x2f32(b, a, exact[mt][nt], 0, 0, 0)
                                                 : __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, exact[mt][nt], 0, 0, 0);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int r = 8 * (e / 4) + 4 * h + e % 4, co = co_w + (SWAP ? l32 : r);
                const uint32_t off = otab[(wn * NT + nt) * 32 + (SWAP ? r : l32)].x;
                const bool on = (again >> (nt * 16 + e) & 1) != 0 && off != kConvOob && co < P.Cout;
                const float v = bias && on ? add_bias(exact[0][nt][e], bias_of(co)) : exact[0][nt][e];
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), orsrc, (int)(on ? off + (uint32_t)co * cs : kConvOob), 0, 0);
            }
    }
}

template <int DT, int VEC, bool SWAP, int MT, int NT, bool PACKED, bool BIG, bool RES, int NC, int GW>
static hipError_t launch_conv_classes(const ConvHead &P, const ConvSub *sub, hipStream_t st)
{
    const void *k = reinterpret_cast<const void *>(conv_kernel<DT, VEC, SWAP, MT, NT, PACKED, BIG, RES, NC, GW>);
    if (P.lds_bytes > 64 * 1024) {
        static bool attr_set[64] = {};   // per device; a repeated call only sets it again
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
        if (dev < 0 || dev >= 64 || !attr_set[dev]) {
            hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            if (e != hipSuccess) return e;
            if (dev >= 0 && dev < 64) attr_set[dev] = true;
        }
    }
    ConvArgs<NC> A;
    static_cast<ConvHead &>(A) = P;
    std::copy(sub, sub + P.nsub, A.sub);
    hipLaunchKernelGGL((conv_kernel<DT, VEC, SWAP, MT, NT, PACKED, BIG, RES, NC, GW>), dim3((unsigned)((P.nwg + 7) / 8 * 8)), dim3(kThreads),
                       (unsigned)P.lds_bytes, st, A);
    return hipGetLastError();
}

template <int DT, int VEC, bool SWAP, int MT, int NT, bool PACKED, bool BIG, bool RES = false, int GW = 1>
static hipError_t launch_conv_one(const ConvHead &P, const ConvSub *sub, hipStream_t st)
{
    if (P.nsub == 1) return launch_conv_classes<DT, VEC, SWAP, MT, NT, PACKED, BIG, RES, 1, GW>(P, sub, st);
    if constexpr (conv_many(MT, NT, PACKED, BIG, RES)) {
        if (P.nsub > kConvSubs) return launch_conv_classes<DT, VEC, SWAP, MT, NT, PACKED, BIG, RES, kConvSubsMany, GW>(P, sub, st);
    }
    if (P.nsub > kConvSubs) return hipErrorInvalidValue;
    return launch_conv_classes<DT, VEC, SWAP, MT, NT, PACKED, BIG, RES, kConvSubs, GW>(P, sub, st);
}

template <int DT, int VEC, bool SWAP> static hipError_t launch_conv_shape(const ConvHead &P, const ConvSub *sub, hipStream_t st)
{
    if (P.big) {
        if constexpr (VEC == 0) return launch_conv_one<DT, VEC, SWAP, 2, 2, false, true>(P, sub, st);
        else return hipErrorInvalidValue;
    }
    const int shape = P.MT * 10 + P.NT;
    if (P.res) {
        if constexpr (!conv_split(DT, true)) {
            if (shape == 24) return launch_conv_one<DT, VEC, SWAP, 2, 4, true, false, true>(P, sub, st);
            if (shape == 22) return launch_conv_one<DT, VEC, SWAP, 2, 2, true, false, true>(P, sub, st);
        }
        if (shape == 12) return launch_conv_one<DT, VEC, SWAP, 1, 2, true, false, true>(P, sub, st);
        return launch_conv_one<DT, VEC, SWAP, 1, 1, true, false, true>(P, sub, st);
    }
    if (P.wp) {
        if constexpr (!conv_split(DT, true)) {
            if (shape == 24) return launch_conv_one<DT, VEC, SWAP, 2, 4, true, false>(P, sub, st);
            if (shape == 22) return launch_conv_one<DT, VEC, SWAP, 2, 2, true, false>(P, sub, st);
        }
        if (shape == 12) return launch_conv_one<DT, VEC, SWAP, 1, 2, true, false>(P, sub, st);
        return launch_conv_one<DT, VEC, SWAP, 1, 1, true, false>(P, sub, st);
    }
    if (shape == 22) return launch_conv_one<DT, VEC, SWAP, 2, 2, false, false>(P, sub, st);
    if (shape == 12) return launch_conv_one<DT, VEC, SWAP, 1, 2, false, false>(P, sub, st);
    if (P.WM == 4) return launch_conv_one<DT, VEC, SWAP, 1, 1, false, false, false, 4>(P, sub, st);
    if (P.WM == 2) return launch_conv_one<DT, VEC, SWAP, 1, 1, false, false, false, 2>(P, sub, st);
    return launch_conv_one<DT, VEC, SWAP, 1, 1, false, false>(P, sub, st);
}

template <int DT> static hipError_t launch_conv_dt(const ConvHead &P, const ConvSub *sub, hipStream_t st)
{
    if (P.vec == 1) {
        if constexpr (DT == XCONV_F32) return hipErrorInvalidValue;
        else return launch_conv_shape<DT, 1, false>(P, sub, st);
    }
    if (P.vec == 2) return launch_conv_shape<DT, 2, true>(P, sub, st);
    return P.swap ? launch_conv_shape<DT, 0, true>(P, sub, st) : launch_conv_shape<DT, 0, false>(P, sub, st);
}

}  // namespace xc
