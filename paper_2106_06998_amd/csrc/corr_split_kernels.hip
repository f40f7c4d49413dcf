// Offset-wise correlation G[m,j,ky,kx] = sum_{b,oy,ox} dY[b,m,oy,ox] * A[b, oy*sh+ky-ph, ox*sw+kx-pw, j]
// (Algorithm 1, backward step 3 with the shift of step 4; Eq. (2)/(5) when A = X) for fp32 storage on the 16-bit matrix cores:
// every float is the sum of three bf16 numbers, and six products of 32x32x16 matrix instructions (192 cycles) do the work of 512
// cycles of fp32 ones (split8, common.h; the products h*h are summed apart from the smaller ones).  A workgroup with sums that the pieces do
// not hold walks through its steps a second time, on fp32 matrix instructions.  Same division of labour as the other producer/consumer kernels:
//
//   waves 0-3 (consumers)  read fragments from LDS and issue matrix instructions.  Each owns 32 output channels x kSplitTiles
//                          tiles of 32 columns: one kernel offset x 32 columns of A, or (WJ = 1, few probing vectors) two kernel
//                          offsets x 16 columns side by side, where the lanes of the second half read another pixel.
//   waves 4-7 (producers)  bring dY (NCHW) and A (channels-last) from global memory into registers, D steps ahead, split them and
//                          write the pieces to LDS.
//
// The 16-byte LDS unit holds one piece of the 8 images of one (pixel, channel), so that a kernel offset or a stride only changes
// which unit a lane reads.  A k-step is two pixels of dY (lanes 0-31 and 32-63) x 8 images.  The waves that WM x WJ leaves over
// (WK) take every WK-th k-step and are added up in LDS at the end.  A step is one output row of one strip of 8 images; rows of A
// live in a ring of kH + sh, dY row pieces are double-buffered; one barrier per step.
//
// Bound by the matrix instructions: one wave a SIMD issues them (160 registers of accumulators leave room for one consumer and one
// producer each), 41 cycles apart for 32 each takes, since neighbours add to the same two sums, and 5 tiles hold 9 offsets.  In C4 (8 x 64 x
// 256x256, 16 columns; 67 us in the trace) a workgroup's 16 steps take 50 us of 3.1 us each, 2.7 without the producers; its first step arrives after
// 7 us.  Against the kernel on fp32 instructions (corr_ws32_kernels.hip) the backward call of C4 takes 105 -> 74 us, of C2 (128 x 64 x 32x32,
// four steps a workgroup) 36.6 -> 31, exact gradients of both 401 -> 355 and 106 -> 79.
#include <type_traits>

#include "common.h"
#include "launch.h"
#include "ws_pos.h"

namespace xc {

namespace {

typedef float f32x16s __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4s __attribute__((ext_vector_type(4)));
typedef int i32x4s __attribute__((ext_vector_type(4)));

constexpr int kSplitTiles = 5;       // accumulator tiles of a consumer wave
constexpr int kSplitOffsets = 10;    // kernel offsets a workgroup accumulates
__host__ __device__ inline int split_sum_units(const WsArgs &P) { return (4 - P.WM * P.WJ) * kSplitTiles * 4 * 64; }   // LDS of the sums along the reduction; the votes are behind them

// Cycles of a step of w columns: its k-steps (those of the wave with the most) or the staging, which takes as long for a narrow
// strip.  Steps are shared out by them, so that workgroups with steps of a narrow last strip take more of them (28 columns in
// strips of 12, 12 and 4, equal numbers of steps: workgroups took 52 to 100 us).
__host__ __device__ inline int split_cost(const WsArgs &P, int w)
{
    const int WK = 4 / (P.WM * P.WJ), mul = ((w >> 1) + WK - 1) / WK * 1150, stage = 1000 * P.NTASK + 500;
    return (mul > stage ? mul : stage) + 150;
}
// first step of workgroup x; P.SQ and P.SR: the cost of all groups of images over the workgroups
__host__ __device__ inline int split_group(const WsArgs &P) { return P.Ho * ((P.NSTRIP - 1) * (split_cost(P, P.CW) >> 6) + (split_cost(P, P.Wo - (P.NSTRIP - 1) * P.CW) >> 6)); }
__device__ inline int split_step(const WsArgs &P, int x)
{
    const int full = split_cost(P, P.CW) >> 6, last = split_cost(P, P.Wo - (P.NSTRIP - 1) * P.CW) >> 6;
    const int u = x * P.SQ + (x < P.SR ? x : P.SR);
    const int group = split_group(P);
    const int bg = u / group, in_group = u - bg * group;
    int strip = in_group / (P.Ho * full);
    strip = strip < P.NSTRIP - 1 ? strip : P.NSTRIP - 1;
    const int w = strip < P.NSTRIP - 1 ? full : last;
    const int y = (in_group - strip * P.Ho * full + w - 1) / w;
    return __builtin_amdgcn_readfirstlane((bg * P.NSTRIP + strip) * P.Ho + y);
}

}  // namespace

// LDS units, in the order written: A [ring row][column of the strip][piece][J_WG], dY [2][slot][piece][M_WG].  Lanes of a fragment read
// take 16 consecutive units of 256 aligned bytes each.  A producer's lanes hold neighbouring pixels, whose units lie multiples of 256
// bytes apart: the channel of a unit is therefore xored with 4 * (slot / 4) (dY) or the column with the pixel's number modulo 4 (A), so that the writes spread
// over the banks.
// WJ: columns of A in halves of a tile (16 * WJ = J_WG).  NTASK: staging tasks per producer thread and step; D: steps whose loads are in flight; VOL: dY is read in place as the depth slots
// of volumes (WsParams::vol_*)
template <int WJ, int NTASK, int D, bool VOL>
__global__ __launch_bounds__(kWsThreads, 2) void corr_split_kernel(const std::conditional_t<VOL, WsParams, WsArgs> P)
{
    draw_z_slice(P.zout, P.nz, P.zdist, P.zseed);
    extern __shared__ uint4 split_lds[];
    uint4 *lds_b = split_lds;
    uint4 *lds_a = split_lds + P.NRING * P.b_row_units;
    constexpr int kJ = 16 * WJ;       // columns of A (P.J_WG)

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tm, tj;
    fast_divmod((int)blockIdx.y, P.NTM, frcp(P.NTM), tj, tm);
    const int m0 = tm * P.M_WG;
    const int jb = tj * P.J_WG;
    int set = 0, og = blockIdx.z;
    if constexpr (VOL) set_and_group(P.NOG, set, og);
    const int o_first = og * kSplitOffsets;
    const int noff = (P.K2 - o_first) < kSplitOffsets ? (P.K2 - o_first) : kSplitOffsets;

    // K-split of this workgroup: neighbouring splits on one die, except for volumes read in place (see corr_ws32_kernel)
    const int bx = VOL ? (int)blockIdx.x : xcd_block(blockIdx.x, gridDim.x);
    const int t_begin = split_step(P, bx), NI = split_step(P, bx + 1) - t_begin;  // steps of this workgroup
    const int a_slot = kSplit * P.M_WG, b_col = kSplit * kJ;    // units of a slot of dY and of a staged column of A
    const int wk_shift = 2 - (P.WM >> 1) - (WJ >> 1), WK = 1 << wk_shift;     // WM and WJ are 1 or 2
    // Votes of the consumers, once all have read their last fragments: sums that are no finite numbers, with a factor or a sum beyond what the
    // pieces hold (split8), are computed once more on the fp32 matrix instructions, from floats in the places of the first two pieces.
    int *votes = reinterpret_cast<int *>(split_lds + split_sum_units(P));
    auto again = [&]() __attribute__((always_inline)) {
        ws_barrier();
        const int any = votes[0] | votes[1] | votes[2] | votes[3];
        ws_barrier();
        return __builtin_amdgcn_readfirstlane(any) != 0;
    };

    if (wave < 4) {
        // =========================== consumers ===========================
        __builtin_amdgcn_s_setprio(3);
        const int l32 = lane & 31, h = lane >> 5;
        const int wm = wave & (P.WM - 1), wj = (wave >> (P.WM >> 1)) & (WJ - 1), wk = wave >> (2 - wk_shift);
        const int per = WJ == 2 ? (noff + 1) / 2 : noff;      // offsets of this wave: from wj * per on

        f32x16s big[kSplitTiles], rest[kSplitTiles];            // sums of the products h*h and of the smaller ones
#pragma unroll
        for (int t = 0; t < kSplitTiles; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) big[t][e] = rest[t][e] = 0.f;

        // offset and column of this lane in tile t; an offset past the last is computed as the first one and not written
        const int j = WJ == 2 ? l32 : l32 & 15;
        auto offset_of = [&](int t) {
            const int i = WJ == 2 ? t : 2 * t + (l32 >> 4);
            return i < per && wj * per + i < noff ? o_first + wj * per + i : -1;
        };
        // through the steps of this workgroup: products of the pieces (0) or of floats, into `rest` (1; rare, and not scheduled by hand)
        auto walk = [&](auto pass) __attribute__((always_inline)) {
            WsPos pc = ws_pos_of(P, t_begin);
            const int ring_bytes = P.NRING * P.b_row_units * 16, row_bytes = P.b_row_units * 16;
            const int a_lane = ring_bytes + ((2 * wk + h) * a_slot + wm * 32 + l32) * 16;         // k-step wk
            const int step_a = 2 * WK * a_slot * 16, step_b = 2 * WK * P.sw * b_col * 16;
            const int flip_b = (2 * WK * P.sw & 3) * 16;                            // how the column's xor changes from a k-step to the next (2 * WK * sw is even)
            const int a_piece = P.M_WG * 16;
            auto read = [](int addr) __attribute__((always_inline)) { return *reinterpret_cast<const __attribute__((address_space(3))) u32x4s *>((uint32_t)addr); };
            int pa, pb[kSplitTiles], q = wk;
            u32x4s a[kSplit], bp[kSplit], b[kSplit];      // fragments of dY, of a tile of A and of the next one
            auto load_a = [&](u32x4s (&dst)[kSplit]) __attribute__((always_inline)) {
                const int addr = pa ^ ((q >> 1 & 3) << 6);
#pragma unroll
                for (int p = 0; p < kSplit; ++p) dst[p] = read(addr + p * a_piece);
            };
            auto load_b = [&](u32x4s (&dst)[kSplit], int t) __attribute__((always_inline)) {
                dst[0] = read(pb[t]);        // in the order of their use
                dst[2] = read(pb[t] + 2 * kJ * 16);
                dst[1] = read(pb[t] + kJ * 16);
            };
            // address of tile t's fragments in the k-step after the one it was read for
            int move = 0, turn = 0;
            auto next_b = [&](int t) __attribute__((always_inline)) {
                const uint32_t x = ((uint32_t)pb[t] ^ (uint32_t)turn) + (uint32_t)move, y = x - (uint32_t)ring_bytes;
                pb[t] = (int)(x < y ? x : y);
            };
            // Three products of a tile and the other three of the tile before it in turn: one wave a SIMD issues a matrix instruction
            // every 55 cycles where each one adds to the sum of the last, every 35-40 where they alternate.
            auto mma = [&](int t, int p, const u32x4s (&x)[kSplit], const u32x4s (&y)[kSplit]) {
                f32x16s &c = kSplitA[p] + kSplitB[p] > 0 ? rest[t] : big[t];
                c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x[kSplitA[p]]), __builtin_bit_cast(bf16x8, y[kSplitB[p]]), c, 0, 0, 0);
            };
            auto copy = [](u32x4s (&dst)[kSplit], const u32x4s (&src)[kSplit]) {
#pragma unroll
                for (int p = 0; p < kSplit; ++p) dst[p] = src[p];
            };

            // k-steps of this wave in a step (0 where a narrow strip has fewer than waves) and in all of them
            auto ksteps = [&](const WsPos &p) { return __builtin_amdgcn_readfirstlane((ws_cw_sub(P, p) / 2 - wk + WK - 1) >> wk_shift); };
            int total = 0;
            {
                WsPos p = pc;
                for (int steps = NI; steps > 0;) {
                    const int n = P.Ho - p.y < steps ? P.Ho - p.y : steps;
                    total += n * ksteps(p);
                    steps -= n;
                    p.y = 0;
                    p.strip = p.strip + 1 == P.NSTRIP ? 0 : p.strip + 1;
                }
            }
            // A run: the steps down one strip.  Its steps have n k-steps each; `rows` are left of it, this one included.
            int i = 0, n, left, rows, row_move, row_turn;
            auto begin_run = [&]() {
                q = wk;
                pa = (i & 1) * P.a_units * 16 + a_lane;
#pragma unroll
                for (int t = 0; t < kSplitTiles; ++t) {
                    int o = offset_of(t), ky, kx;
                    asm volatile("" : "+v"(o));      // (computed here, not kept in registers through the loop)
                    fast_divmod(o < 0 ? o_first : o, P.kW, frcp(P.kW), ky, kx);
                    int slot = pc.rowmod + ky;
                    slot = slot >= P.NRING ? slot - P.NRING : slot;
                    const int c = (2 * wk + h) * P.sw + kx;
                    pb[t] = (slot * P.b_row_units + c * b_col + (j ^ (c & 3))) * 16;
                }
                n = left = ksteps(pc);
                rows = __builtin_amdgcn_readfirstlane(P.Ho - pc.y);
                row_move = P.sh * row_bytes - (n - 1) * step_b;
                row_turn = (n - 1) & 1 ? flip_b : 0;
                move = turn = 0;
            };
            // from the last step of a run to the first one with k-steps of this wave
            auto next_run = [&]() {
                do {       // (a run without k-steps of this wave has its barriers all the same)
                    ++i;
                    pc.y = 0;
                    pc.rowmod = 0;
                    pc.strip = pc.strip + 1 == P.NSTRIP ? 0 : pc.strip + 1;
                    ws_barrier();      // the producers refill the whole ring first
                    ws_barrier();
                    if (ksteps(pc) > 0) break;
                    for (int y = 1; y < P.Ho && i + 1 < NI; ++y, ++i) ws_barrier();
                } while (i + 1 < NI);
                begin_run();
            };
            // What the next k-step of this wave is: how the addresses move ...
            auto look_ahead = [&]() __attribute__((always_inline)) {
                const bool same = left > 1, run = rows > 1;
                move = same ? step_b : run ? row_move : 0;
                turn = same ? flip_b : run ? row_turn : 0;
            };
            // ... and the way there.  At the end of a step, the fragments read so far are in registers behind the barrier, so that the
            // step's buffer and the ring rows it alone used go back to the producers
            auto advance = [&]() __attribute__((always_inline)) {
                if (--left > 0) {
                    q += WK;
                    pa += step_a;
                } else if (--rows > 0) {
                    ++i;
                    ws_barrier();
                    q = wk;
                    pa = (i & 1) * P.a_units * 16 + a_lane;
                    left = n;
                } else {
                    next_run();
                }
            };
            // Tile t is finished beside the first half of tile t + 1.  Each matrix instruction hides four or so others of its wave: `loads`
            // (fragment reads) and `moves` (addresses) are spread behind them (sched_group_barrier: 8 matrix instructions, 2 vector, 0x100 LDS reads).
            auto round = [&](int t, const u32x4s (&an)[kSplit], const u32x4s (&bn)[kSplit], auto &&loads, auto &&moves) __attribute__((always_inline)) {
                const int t1 = (t + 1) % kSplitTiles;
                const u32x4s(&a1)[kSplit] = t + 1 < kSplitTiles ? a : an;
                __builtin_amdgcn_sched_barrier(0);
                loads();
                moves();
                mma(t, 5, a, bp);
                mma(t1, 0, a1, b);
                mma(t, 3, a, bp);
                mma(t1, 1, a1, b);
                mma(t, 4, a, bp);
                mma(t1, 2, a1, b);
                __builtin_amdgcn_sched_group_barrier(8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_group_barrier(8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_group_barrier(8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                __builtin_amdgcn_sched_group_barrier(8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(2, 3, 0);
                __builtin_amdgcn_sched_group_barrier(8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(2, 3, 0);
                __builtin_amdgcn_sched_group_barrier(8, 1, 0);
                __builtin_amdgcn_sched_barrier(0);
                copy(bp, b);
                copy(b, bn);
            };

            begin_run();
            ws_barrier();  // the first dY tile and the rows of the first step are in LDS
            if (total > 0) {
                if (left == 0) {
                    for (int y = pc.y + 1; y < P.Ho; ++y, ++i) ws_barrier();
                    next_run();
                }
                if constexpr (decltype(pass)::value == 1) {
                    for (int n = total; n > 0; --n) {
                        const int addr = pa ^ ((q >> 1 & 3) << 6);
                        a[0] = read(addr);
                        a[1] = read(addr + a_piece);
                        ws_static_for<0, kSplitTiles>([&](auto tc) __attribute__((always_inline)) {
                            constexpr int t = decltype(tc)::value;
                            b[0] = read(pb[t]);
                            b[1] = read(pb[t] + kJ * 16);
#pragma unroll
                            for (int e = 0; e < 8; ++e)
                                rest[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[e / 4][e & 3]), __uint_as_float(b[e / 4][e & 3]), rest[t], 0, 0, 0);
                        });
                        if (n == 1) break;
                        look_ahead();
                        ws_static_for<0, kSplitTiles>([&](auto tc) __attribute__((always_inline)) { next_b(decltype(tc)::value); });
                        advance();
                    }
                } else {
                    load_a(a);
                    load_b(bp, 0);
                    load_b(b, 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int p = 0; p < 3; ++p) mma(0, p, a, bp);
                    // the fragments of tile t + 2 are on their way beside tiles t and t + 1 (behind the last tile those of the next k-step)
                    u32x4s an[kSplit], bn[kSplit];
                    for (int n = total; n > 1; --n) {
                        ws_static_for<0, kSplitTiles>([&](auto tc) __attribute__((always_inline)) {
                            constexpr int t = decltype(tc)::value;
                            if constexpr (t + 3 == kSplitTiles) look_ahead();
                            if constexpr (t + 2 == kSplitTiles) advance();
                            round(t, an, bn, [&]() __attribute__((always_inline)) {
                                load_b(bn, (t + 2) % kSplitTiles);
                                if constexpr (t + 2 == kSplitTiles) load_a(an);
                            }, [&]() __attribute__((always_inline)) { next_b((t + 3) % kSplitTiles); });
                        });
                        copy(a, an);
                    }
                    ws_static_for<0, kSplitTiles - 1>([&](auto tc) __attribute__((always_inline)) {
                        constexpr int t = decltype(tc)::value;
                        round(t, a, bn, [&]() __attribute__((always_inline)) { if constexpr (t + 2 < kSplitTiles) load_b(bn, t + 2); },
                              [&]() __attribute__((always_inline)) { if constexpr (t + 3 < kSplitTiles) next_b(t + 3); });
                    });
                    mma(kSplitTiles - 1, 5, a, bp);
                    mma(kSplitTiles - 1, 3, a, bp);
                    mma(kSplitTiles - 1, 4, a, bp);
                }
            }
            // steps behind the last one with k-steps of this wave
            for (WsPos p = ws_pos_of(P, t_begin + i); i + 1 < NI; ++i) {
                p = ws_advance(P, p);
                if (p.y == 0) ws_barrier();
                ws_barrier();
            }
        };
        // (nothing but the sums is kept from one walk to the other)
        if (NI > 0) {
            walk(std::integral_constant<int, 0>{});
            float odd_sum = 0.f;       // NaN as soon as a sum is not finite
#pragma unroll
            for (int t = 0; t < kSplitTiles; ++t)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    big[t][e] = (big[t][e] + rest[t][e]) * kSplitUnscale;
                    odd_sum = fmaf(big[t][e], 0.f, odd_sum);
                }
            const int vote = __ballot(odd_sum != 0.f) != 0;
            ws_barrier();
            if (lane == 0) votes[wave] = vote;
            if (again()) {
#pragma unroll
                for (int t = 0; t < kSplitTiles; ++t)
#pragma unroll
                    for (int e = 0; e < 16; ++e) rest[t][e] = 0.f;
                walk(std::integral_constant<int, 1>{});
#pragma unroll
                for (int t = 0; t < kSplitTiles; ++t)
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (!(fabsf(big[t][e]) < __builtin_inff())) big[t][e] = rest[t][e];
            }
        }

        // the waves along the reduction meet in LDS: [wave][tile][quad of rows][lane]
        if (WK > 1) {
            f32x4 *sum = reinterpret_cast<f32x4 *>(split_lds);
            ws_barrier();
            if (wk > 0) {
#pragma unroll
                for (int t = 0; t < kSplitTiles; ++t)
#pragma unroll
                    for (int g = 0; g < 4; ++g)
                        sum[((wave - 4 / WK) * kSplitTiles * 4 + t * 4 + g) * 64 + lane] = f32x4{big[t][4 * g], big[t][4 * g + 1], big[t][4 * g + 2], big[t][4 * g + 3]};
            }
            ws_barrier();
            if (wk > 0) return;
            for (int w = 1; w < WK; ++w) {
                const int other = wave + (w - 1) * (4 / WK);
#pragma unroll
                for (int t = 0; t < kSplitTiles; ++t)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 v = sum[(other * kSplitTiles * 4 + t * 4 + g) * 64 + lane];
#pragma unroll
                        for (int e = 0; e < 4; ++e) big[t][4 * g + e] += v[e];
                    }
            }
        }

        // accumulator tile: lane (l32, h) holds column l32 and rows 8g + 4h .. + 3
#pragma unroll
        for (int t = 0; t < kSplitTiles; ++t) {
            const int o = offset_of(t);
            if (o < 0) continue;
            float *part = P.part + (size_t)(VOL ? set * P.S + bx : bx) * P.K2 * P.JP * P.MP;
#pragma unroll
            for (int g = 0; g < 4; ++g)
                *reinterpret_cast<f32x4 *>(part + tile_index(o, jb + j, m0 + wm * 32 + 8 * g + 4 * h, P.JP, P.MP)) =
                    f32x4{big[t][4 * g], big[t][4 * g + 1], big[t][4 * g + 2], big[t][4 * g + 3]};
        }
    } else {
        // =========================== producers ===========================
        __builtin_amdgcn_s_setprio(0);
        const int p = tid - kProducers;
        const float *dY = static_cast<const float *>(P.dY);
        const float *Ag = static_cast<const float *>(P.A);
        if constexpr (VOL) Ag = reinterpret_cast<const float *>(static_cast<const char *>(P.A) + set_offset(set, P.set_sd, P.set_run, P.set_slice));
        const int HoWo = P.Ho * P.Wo;
        // bytes between the planes of consecutive channels and between consecutive images of the batch
        const uint32_t dy_plane_bytes = (uint32_t)HoWo * 4u * (VOL ? (uint32_t)P.vol_Do : 1u);
        const uint32_t dy_img_bytes = VOL ? (uint32_t)HoWo * 4u : (uint32_t)P.C_out * (uint32_t)HoWo * 4u;
        const float rcp_period = frcp(VOL ? P.vol_period : 1);
        const uint32_t a_img_bytes = (uint32_t)P.H * (uint32_t)P.W * (uint32_t)P.CS * 4u;
        constexpr int JC = kJ >> 2, jc_shift = WJ == 2 ? 3 : 2;   // 4-column vectors per staged pixel
        const int rows_new = P.sh < P.kH ? P.sh : P.kH;                  // rows a step adds to the ring
        const int rows_old = P.kH - rows_new;                            // rows it inherits from its predecessor
        const float rcp_bwc = frcp(P.BWc);

        // Task slots of this thread.  Slots below NA_pad (whole waves) stage dY: chunk of 4 columns fastest (neighbouring lanes read
        // neighbouring 16-byte pieces of one (image, channel) row).  The remaining slots stage the rows of A the step adds: column vector fastest.
        bool is_a[NTASK];
        uint32_t t_goff[NTASK];    // byte offset inside an image without the step's part, or kOOR
        int t_lds[NTASK], t_aux[NTASK];
        const int nch = P.CWs >> 2;
        const float rcp_nch = frcp(nch);
#pragma unroll
        for (int k = 0; k < NTASK; ++k) {
            const int s = p + kProducers * k;
            is_a[k] = __builtin_amdgcn_readfirstlane((int)(s < P.NA_pad)) != 0;
            if (is_a[k]) {
                int ch, m;
                fast_divmod(s, nch, rcp_nch, m, ch);
                t_goff[k] = (s < P.NA && m0 + m < P.C_out) ? (uint32_t)(m0 + m) * dy_plane_bytes + 16u * ch : kOOR;
                t_lds[k] = 4 * ch * a_slot + (m ^ ((ch & 3) << 2));
                t_aux[k] = 4 * ch;          // first column of the chunk
            } else {
                const int w = s - P.NA_pad;
                const int jc = w & (JC - 1);
                int c, rr;
                fast_divmod(w >> jc_shift, P.BWc, rcp_bwc, rr, c);
                const bool has = w < P.TB;
                t_goff[k] = has ? ((uint32_t)(rr * P.W + c) * (uint32_t)P.CS + (uint32_t)(jb + 4 * jc)) * 4u : kOOR;
                t_lds[k] = c * b_col + 4 * jc;
                t_aux[k] = c | (rr << 16);
            }
        }

        // Buffer resources built by hand: a group with fewer than 8 images, or a step that does not exist, gets a smaller (or empty)
        // resource: reads past it return zero.
        auto rsrc_of = [&](const float *base, int bg, uint32_t img_bytes, bool live) __attribute__((always_inline)) {
            bg = __builtin_amdgcn_readfirstlane(bg);
            int left = P.B - bg * 8;
            left = left < 8 ? left : 8;
            left = (live && left > 0) ? left : 0;
            const uint64_t addr = reinterpret_cast<uint64_t>(base + (size_t)bg * 8 * (img_bytes / 4));
            i32x4s r;
            r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)addr);
            r.y = __builtin_amdgcn_readfirstlane((int)(uint32_t)((addr >> 32) & 0xffffu));
            r.z = __builtin_amdgcn_readfirstlane((int)((uint32_t)left * img_bytes));
            r.w = 0x00020000;
            settle_resource(r);
            return r;
        };
        // Loads of the software pipeline: opaque instructions, waited for by hand (stage_wait); nothing reads a stage between its
        // loads and its wait.
        auto buf16_async = [](u32x4s &dst, i32x4s r, uint32_t voff) {
            asm volatile("buffer_load_dwordx4 %0, %1, %2, 0 offen" : "=v"(dst) : "v"(voff), "s"(r) : "memory");
        };
        // The 4 x 8 values of a task: value e of the 8 images is unit e * step (dY: the next slot) or e ^ flip (A: the next column), its
        // pieces `piece` units apart; as floats, images 0-3 are in the place of the first piece and 4-7 in that of the second.
        bool floats = false;
        auto put = [&](uint4 *dst, int step, int flip, int piece, const u32x4s (&r)[8]) __attribute__((always_inline)) {
            // (one branch for the task: with one for each value the exact gradient of C4 takes 376 us for 361)
            if (floats) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    uint4 *unit = dst + (step ? e * step : e ^ flip);
                    unit[0] = uint4{r[0][e], r[1][e], r[2][e], r[3][e]};
                    unit[piece] = uint4{r[4][e], r[5][e], r[6][e], r[7][e]};
                }
                return;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                uint4 *unit = dst + (step ? e * step : e ^ flip);
                float v[8];
                uint4 w[kSplit];
#pragma unroll
                for (int img = 0; img < 8; ++img) {
                    const unsigned int u = r[img][e];
                    v[img] = __uint_as_float(u);
                }
                split8(v, w);
#pragma unroll
                for (int x = 0; x < kSplit; ++x) unit[x * piece] = w[x];
            }
        };

        // ---- loads of step ps: its dY row piece and the rows it adds to the ring
        auto issue = [&](const WsPos &ps, bool live, u32x4s (&r)[NTASK][8]) __attribute__((always_inline)) {
            const int cw = ws_cw_sub(P, ps);
            const uint32_t fs = (uint32_t)(ps.y * P.Wo + ps.strip * P.CW) * 4u;
            // dY: byte offset of each of the group's 8 images, or kOOR for one that does not exist
            i32x4s rsA;
            uint32_t doff[8];
            if constexpr (!VOL) {
                rsA = rsrc_of(dY, ps.bg, dy_img_bytes, live);
            } else {
                // the whole tensor behind one resource; image -> (volume, depth slot), empty slots read as zero
                const uint64_t addr = reinterpret_cast<uint64_t>(dY);
                rsA.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)addr);
                rsA.y = __builtin_amdgcn_readfirstlane((int)(uint32_t)((addr >> 32) & 0xffffu));
                rsA.z = __builtin_amdgcn_readfirstlane((int)(live ? P.vol_bytes : 0u));
                rsA.w = 0x00020000;
                settle_resource(rsA);
                const uint32_t vol_stride = (uint32_t)P.C_out * dy_plane_bytes;
#pragma unroll
                for (int img = 0; img < 8; ++img) {
                    const int i = __builtin_amdgcn_readfirstlane(ps.bg) * 8 + img;
                    int bv, z;
                    fast_divmod(i, P.vol_period, rcp_period, bv, z);
                    doff[img] = (uint32_t)__builtin_amdgcn_readfirstlane(
                        (int)((i < P.B && z < P.vol_Do) ? (uint32_t)bv * vol_stride + (uint32_t)z * dy_img_bytes : kOOR));
                }
            }
            const i32x4s rsB = rsrc_of(Ag, ps.bg, a_img_bytes, live);
            const int iy0 = ps.y * P.sh + rows_old - P.ph;   // input row of the first added row
            const int ix0 = ps.strip * P.CW * P.sw - P.pw;
            const uint32_t origin = (uint32_t)(iy0 * P.W + ix0) * ((uint32_t)P.CS * 4u);  // wraps when negative; exact for every in-range pixel
#pragma unroll
            for (int k = 0; k < NTASK; ++k) {
                if (is_a[k]) {
                    const uint32_t voff = (t_goff[k] != kOOR && t_aux[k] < cw) ? t_goff[k] + fs : kOOR;
#pragma unroll
                    for (int img = 0; img < 8; ++img) {
                        if constexpr (!VOL) buf16_async(r[k][img], rsA, voff + (uint32_t)img * dy_img_bytes);
                        else buf16_async(r[k][img], rsA, (voff != kOOR && doff[img] != kOOR) ? voff + doff[img] : kOOR);
                    }
                } else {
                    const int c = t_aux[k] & 0xffff, rr = t_aux[k] >> 16;
                    const bool in = t_goff[k] != kOOR && (unsigned)(iy0 + rr) < (unsigned)P.H && (unsigned)(ix0 + c) < (unsigned)P.W;
                    const uint32_t voff = in ? origin + t_goff[k] : kOOR;
#pragma unroll
                    for (int img = 0; img < 8; ++img) buf16_async(r[k][img], rsB, voff + (uint32_t)img * a_img_bytes);
                }
            }
        };
        // the loads of a stage are followed by those of D - 1 younger stages
        auto stage_wait = [&](u32x4s (&r)[NTASK][8]) __attribute__((always_inline)) {
            constexpr int kYounger = (D - 1) * NTASK * 8;
#pragma unroll
            for (int k = 0; k < NTASK; ++k)
                asm volatile("s_waitcnt vmcnt(%8)"
                             : "+v"(r[k][0]), "+v"(r[k][1]), "+v"(r[k][2]), "+v"(r[k][3]), "+v"(r[k][4]), "+v"(r[k][5]), "+v"(r[k][6]), "+v"(r[k][7])
                             : "n"(kYounger)
                             : "memory");
        };
        // ---- registers -> LDS
        auto write = [&](const WsPos &ps, int buf, const u32x4s (&r)[NTASK][8]) __attribute__((always_inline)) {
            int slot0 = ps.rowmod + rows_old;   // ring slot of the first added row
            slot0 = slot0 >= P.NRING ? slot0 - P.NRING : slot0;
#pragma unroll
            for (int k = 0; k < NTASK; ++k) {
                int slot = slot0 + (t_aux[k] >> 16);
                slot = slot >= P.NRING ? slot - P.NRING : slot;
                uint4 *dst = is_a[k] ? lds_a + buf * P.a_units + t_lds[k] : lds_b + slot * P.b_row_units + t_lds[k];
                // (rows of channels beyond the last are written too: zeros)
                if (is_a[k] ? p + kProducers * k < P.NA : t_goff[k] != kOOR)
                    put(dst, is_a[k] ? a_slot : 0, t_aux[k] & 3, is_a[k] ? P.M_WG : kJ, r[k]);
            }
        };
        // ---- the rows a step inherits, loaded and written at once (start of a run)
        auto prime = [&](const WsPos &ps) __attribute__((always_inline)) {
            const i32x4s rsB = rsrc_of(Ag, ps.bg, a_img_bytes, true);
            const int total = rows_old * P.BWc * JC;
            const int iy0 = ps.y * P.sh - P.ph, ix0 = ps.strip * P.CW * P.sw - P.pw;
            for (int base = 0; base < total; base += kProducers) {
                u32x4s r[8];
                const int idx = base + p;
                const int jc = idx & (JC - 1);
                int c, rr;
                fast_divmod(idx >> jc_shift, P.BWc, rcp_bwc, rr, c);
                const int iy = iy0 + rr, ix = ix0 + c;
                const bool in = idx < total && (unsigned)iy < (unsigned)P.H && (unsigned)ix < (unsigned)P.W;
                const uint32_t voff = in ? ((uint32_t)(iy * P.W + ix) * (uint32_t)P.CS + (uint32_t)(jb + 4 * jc)) * 4u : kOOR;
                int slot = ps.rowmod + rr;
                slot = slot >= P.NRING ? slot - P.NRING : slot;
#pragma unroll
                for (int img = 0; img < 8; ++img) buf16_async(r[img], rsB, voff + (uint32_t)img * a_img_bytes);
                asm volatile("s_waitcnt vmcnt(0)"
                             : "+v"(r[0]), "+v"(r[1]), "+v"(r[2]), "+v"(r[3]), "+v"(r[4]), "+v"(r[5]), "+v"(r[6]), "+v"(r[7])
                             :
                             : "memory");
                if (idx < total) put(lds_b + slot * P.b_row_units + c * b_col + 4 * jc, 0, c & 3, kJ, r);
            }
        };

        while (NI > 0) {
            WsPos pw = ws_pos_of(P, t_begin);  // step whose data is written next
            WsPos pi = pw;                     // step whose loads are issued next
            u32x4s st[D][NTASK][8];
            // (the wait of the inherited rows covers the older loads of the first step as well)
            issue(pi, true, st[0]);
            pi = ws_advance(P, pi);
            prime(pw);
#pragma unroll
            for (int d = 1; d < D; ++d) {
                issue(pi, d < NI, st[d]);
                pi = ws_advance(P, pi);
            }
            for (int i0 = 0; i0 < NI; i0 += D) {
                ws_static_for<0, D>([&](auto dc) __attribute__((always_inline)) {
                    constexpr int d = decltype(dc)::value;
                    const int i = i0 + d;
                    if (i < NI) {
                        if (i > 0 && pw.y == 0) {
                            ws_barrier();  // the consumers have left the previous run: its ring rows are free
                            prime(pw);
                        }
                        stage_wait(st[d]);
                        write(pw, i & 1, st[d]);
                        issue(pi, i + D < NI, st[d]);
                        pw = ws_advance(P, pw);
                        pi = ws_advance(P, pi);
                        ws_barrier();
                    }
                });
            }
            // the last (empty) prefetches: their registers are theirs until they are back
#pragma unroll
            for (int d = 0; d < D; ++d)
#pragma unroll
                for (int k = 0; k < NTASK; ++k)
                    asm volatile("s_waitcnt vmcnt(0)"
                                 : "+v"(st[d][k][0]), "+v"(st[d][k][1]), "+v"(st[d][k][2]), "+v"(st[d][k][3]), "+v"(st[d][k][4]), "+v"(st[d][k][5]),
                                   "+v"(st[d][k][6]), "+v"(st[d][k][7])
                                 :
                                 : "memory");
            if (floats) break;
            ws_barrier();
            floats = again();
            if (!floats) break;
        }
        if (WK > 1) {      // the consumers' sums
            ws_barrier();
            ws_barrier();
        }
    }
}

// ---------------------------------------------------------------------------
// host: launch plan
// ---------------------------------------------------------------------------
static const size_t kSplitLdsLimit = 160 * 1024;

size_t corr_split_lds_bytes(const WsParams &P)
{
    const size_t stage = ((size_t)2 * P.a_units + (size_t)P.NRING * P.b_row_units) * 16;
    const size_t sums = ((size_t)split_sum_units(P) + 1) * 16;
    return stage > sums ? stage : sums;
}

bool plan_corr_split(WsParams &P, int B, int C_out, int H, int W, int kH, int kW, int sh, int sw, int ph, int pw, int CS, int nsets, int splits)
{
    P.B = B; P.C_out = C_out; P.H = H; P.W = W;
    P.kH = kH; P.kW = kW; P.sh = sh; P.sw = sw; P.ph = ph; P.pw = pw;
    P.Ho = (H + 2 * ph - kH) / sh + 1;
    P.Wo = (W + 2 * pw - kW) / sw + 1;
    P.CS = CS;
    P.K2 = kH * kW;
    P.NBG = ceil_div(B, 8);
    P.NOG = ceil_div(P.K2, kSplitOffsets);
    // up to 4 images fill half of a unit, and few offsets few of the tiles: there the fp32 instructions are as fast
    if (B <= 4 || 5 * P.K2 < 3 * kSplitOffsets * P.NOG) return false;
    if (P.Wo % 4 != 0) return false;       // rows of dY are read and multiplied in whole vectors of 4 columns
    if (kH > 8 || sh > 8) return false;
    // a group of 8 images is addressed with 32-bit byte offsets
    if ((long long)8 * C_out * P.Ho * P.Wo * 4 > (1LL << 30) || (long long)8 * H * W * CS * 4 > (1LL << 30)) return false;
    P.WJ = CS % 32 == 0 ? 2 : 1;
    P.WM = C_out > 32 ? 2 : 1;
    P.M_WG = 32 * P.WM; P.J_WG = 16 * P.WJ;
    P.NTM = ceil_div(C_out, P.M_WG);
    P.NTJ = CS / P.J_WG;
    P.MP = P.NTM * P.M_WG;
    P.JP = CS;
    P.MT = 2;
    P.NSUB = 1;
    P.NRING = kH + sh;
    P.BSTR = P.J_WG;
    const int rows_new = sh < kH ? sh : kH;
    auto geometry = [&](int cw) {
        P.CW = cw; P.CWs = cw;
        P.NSTRIP = ceil_div(P.Wo, cw);
        P.BWc = (cw - 1) * sw + kW;
        P.a_units = cw * kSplit * P.M_WG;
        P.b_row_units = P.BWc * kSplit * P.J_WG;
        P.NA = P.M_WG * (cw / 4);
        P.NA_pad = round_up(P.NA, 64);
        P.TB = rows_new * P.BWc * (P.J_WG / 4);
        P.TS = P.TB;
        P.NTASK = ceil_div(P.NA_pad + P.TB, kProducers);
    };
    // strip width: of those that fit, the one of the least cost, then the narrowest
    int best = 0, best_cost = 0;
    for (int cw = (P.Wo < 64 ? P.Wo : 64) & ~3; cw >= 4; cw -= 4) {
        geometry(cw);
        if (corr_split_lds_bytes(P) > kSplitLdsLimit || P.NTASK > 2) continue;
        const int cost = (P.NSTRIP - 1) * split_cost(P, cw) + split_cost(P, P.Wo - (P.NSTRIP - 1) * cw);
        if (best == 0 || cost <= best_cost) { best = cw; best_cost = cost; }
    }
    if (best == 0) return false;
    geometry(best);
    P.NS = P.NBG * P.NSTRIP * P.Ho;
    if ((long long)P.NBG * split_group(P) > (1LL << 30)) return false;
    // K-split: one workgroup per compute unit
    int target = splits > 0 ? splits : choose_splits(256 / (P.NTM * P.NTJ * P.NOG * nsets), P.NS, nsets);
    if (target > P.NS) target = P.NS;
    if (target < 1) target = 1;
    P.S = target;
    if (splits > 0) return true;
    // The kernel on fp32 instructions has less code and a shorter first step: it is done first where there are few steps.  In
    // us, with what both take besides: the steps of a workgroup here at 1.85 GHz, and there the tiles' products (64 a cycle and SIMD)
    // at nine tenths of 1.95.  56 drawn layers: 0.42-1.04 of its time where this kernel is taken, 0.86-1.26 where it is not.
    const int nwj = CS / 16, wj = nwj % 4 == 0 && C_out <= 16 ? 4 : nwj % 2 == 0 && C_out <= 32 ? 2 : 1;
    const double here = (double)P.NBG * split_group(P) * 64 / P.S / 1850;
    const double there = (double)round_up(B, 4) * P.Ho * P.Wo * round_up(C_out, 64 / wj) * CS * ceil_div(P.K2, 9) * 9 * nsets * 2 / (64.0 * 4 * 256) / 1770;
    return here + 4.5 < there;
}

template <int WJ, int NTASK, int D, bool VOL> static hipError_t launch_split_cfg(const WsParams &P, hipStream_t st)
{
    const size_t lds = corr_split_lds_bytes(P);
    static bool done = false;  // per instantiation: the attribute sticks to the function
    if (!done && lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(corr_split_kernel<WJ, NTASK, D, VOL>), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)kSplitLdsLimit);
        if (e != hipSuccess) return e;
        done = true;
    }
    WsParams Q = P;
    Q.SQ = P.NBG * split_group(P) / P.S;      // (split_step)
    Q.SR = P.NBG * split_group(P) % P.S;
    hipLaunchKernelGGL((corr_split_kernel<WJ, NTASK, D, VOL>), dim3(P.S, P.NTM * P.NTJ, P.NOG * (P.nsets > 1 ? P.nsets : 1)), dim3(kWsThreads), lds, st, Q);
    return hipGetLastError();
}

template <int WJ> static hipError_t launch_split_wj(const WsParams &P, hipStream_t st)
{
    if (P.vol_period != 0) return P.NTASK == 1 ? launch_split_cfg<WJ, 1, 3, true>(P, st) : launch_split_cfg<WJ, 2, 2, true>(P, st);
    return P.NTASK == 1 ? launch_split_cfg<WJ, 1, 3, false>(P, st) : launch_split_cfg<WJ, 2, 2, false>(P, st);
}

hipError_t launch_corr_split(const WsParams &P, hipStream_t st) { return P.WJ == 2 ? launch_split_wj<2>(P, st) : launch_split_wj<1>(P, st); }

}  // namespace xc
