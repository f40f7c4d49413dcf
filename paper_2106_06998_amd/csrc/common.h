// Internal definitions shared by the HIP translation units of libxconv.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "../../include/xconv.h"

namespace xc {

constexpr int kThreads = 256;  // every kernel runs 4 wavefronts of 64 lanes per workgroup
constexpr int kMaxGridZ = 65535;  // largest third extent of a grid: launches over more images go in pieces

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

enum KernelId {
    K_GEN_Z = 0,
    K_PROBE = 1,
    K_PROBE_GENERIC = 2,
    K_CORR = 3,
    K_REDUCE = 4,
    K_TO_NHWC = 5,
    K_UNPACK = 6,
    K_EXPAND = 7,
    K_REPACK = 8,
    K_PACK_Z = 9,
    K_ZERO_GAPS = 10,
    K_GEN_ZIMG = 11,
    K_SCALE = 12,
    K_PIXEL_FWD = 13,
    K_RELU = 14,
    K_CONV = 15,
    K_PASS2 = 16,
    K_DIAG = 17,
    K_BIAS = 18,
    K_COUNT = 19
};

// Where the probe output of a voxel goes in Xt.  sd == 0: plain order, pixel `first` of the
// input is pixel `first` of Xt.  Volumetric layers (sd = depth stride >= 1): Xt is sd runs of
// `run` depth slices; slice z of image `img` is slot (z + pd) / sd of the image's `period`
// slots in run (z + pd) % sd, so that kernel-depth offset kz pairs output slice oz with slot
// oz + kz / sd of run kz % sd.
struct SliceMap {
    int HWs, D, pd, sd, period;
    long long run;
    __host__ __device__ long long slice_of(long long img, int z) const
    {
        const int t = z + pd;
        return (long long)(t % sd) * run + img * period + t / sd;
    }
    // HW = D * HWs pixels per image
    __host__ __device__ long long out_pixel(long long first, int HW) const
    {
        if (sd == 0) return first;
        const long long img = first / HW;
        const int rem = (int)(first - img * HW);
        const int z = rem / HWs;
        return slice_of(img, z) * HWs + (rem - z * HWs);
    }
};

__host__ __device__ inline int round_up(int a, int b) { return (a + b - 1) / b * b; }
__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Layout of one fp32 tile of correlation sums (a K-split's partial tile, or the reduced tile): [K2][MP/4][JP][4].
// Four consecutive output channels of one (offset, column) are a 16-byte element, and the JP columns of such a
// channel quad are contiguous: the lanes of a matrix-instruction result (one column each, four rows per register
// group) store runs of 16-byte elements, and the second pass reads a quad's columns as one run.
__host__ __device__ inline size_t tile_index(int o, int j, int m, int JP, int MP)
{
    return ((((size_t)o * (size_t)(MP >> 2) + (size_t)(m >> 2)) * (size_t)JP + (size_t)j) << 2) + (size_t)(m & 3);
}

// ---- storage-type conversions (device) ------------------------------------
__device__ inline uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // NaN stays NaN
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ inline uint16_t f32_to_f16_rne(float f)
{
    _Float16 h = (_Float16)f;  // v_cvt_f16_f32: round to nearest even
    return __builtin_bit_cast(uint16_t, h);
}
__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__device__ inline float f16_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }

template <int DT> __device__ inline uint16_t f32_to_st16(float f)
{
    if constexpr (DT == XCONV_BF16) return f32_to_bf16_rne(f);
    else return f32_to_f16_rne(f);
}
template <int DT> __device__ inline float st16_to_f32(uint16_t h)
{
    if constexpr (DT == XCONV_BF16) return bf16_to_f32(h);
    else return f16_to_f32(h);
}

// 16x16x32 MFMA on eight 16-bit values per lane (passed as the raw 16 bytes).
template <int DT> __device__ inline f32x4 mfma16(const uint4 &a, const uint4 &b, f32x4 c)
{
    if constexpr (DT == XCONV_BF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}

// A float x as three bf16 numbers (8 + 8 + 8 bits of the 24), each rounded to nearest: h + m + l = x * kSplitScale exactly, for every
// float below kSplitTop, subnormal ones too (the last bit of the smallest is 2^-149; scaled, it is a normal bf16 number).  A product of two
// such sums, less its terms below 2^-25 (m*l, l*m, l*l), is six products on the 16-bit matrix cores in place of one on the fp32
// ones, which take 16 times as long (kSplitA, kSplitB); sums of them are scaled back by kSplitUnscale.
// From kSplitTop on (2.0e31, infinities) and for NaN the pieces are infinities and NaN, and a sum of products beyond 1.2e24 overflows too: then
// the sum is no finite number, whatever the other factors are, and the kernel computes it again on the fp32 matrix instructions.
constexpr int kSplit = 3;
constexpr int kSplitProducts = 6;
constexpr int kSplitA[kSplitProducts] = {2, 0, 1, 1, 0, 0}, kSplitB[kSplitProducts] = {0, 2, 1, 0, 1, 0};   // small terms first
constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f, kSplitTop = 0x1p104f;
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ inline uint32_t bf16_pair(float a, float b) { return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2)); }
// eight floats in pieces
__device__ __forceinline__ void split8(const float (&x)[8], uint4 (&out)[kSplit])
{
    uint32_t p[kSplit][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i] * kSplitScale, b = x[2 * i + 1] * kSplitScale;
#pragma unroll
        for (int q = 0; q < kSplit; ++q) {
            const uint32_t w = bf16_pair(a, b);
            p[q][i] = w;
            if (q + 1 < kSplit) {
                a -= __uint_as_float(w << 16);
                b -= __uint_as_float(w & 0xffff0000u);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < kSplit; ++q) out[q] = uint4{p[q][0], p[q][1], p[q][2], p[q][3]};
}
// Packed weights keep every float: one that the pieces do not hold is a NaN, so that no sum with it is finite, and its own bits in the
// other two places.
constexpr uint32_t kSplitRaw = 0x7fc0u;
__device__ inline void split8_packed(const float (&x)[8], uint4 (&out)[kSplit])
{
    split8(x, out);
    uint32_t p[kSplit][4];
#pragma unroll
    for (int q = 0; q < kSplit; ++q) p[q][0] = out[q].x, p[q][1] = out[q].y, p[q][2] = out[q].z, p[q][3] = out[q].w;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        if (fabsf(x[e]) < 0.5f * kSplitTop) continue;
        const uint32_t bits = __float_as_uint(x[e]), v[kSplit] = {kSplitRaw, bits >> 16, bits & 0xffffu};
#pragma unroll
        for (int q = 0; q < kSplit; ++q)
            p[q][e / 2] = e & 1 ? (p[q][e / 2] & 0xffffu) | (v[q] << 16) : (p[q][e / 2] & 0xffff0000u) | v[q];
    }
#pragma unroll
    for (int q = 0; q < kSplit; ++q) out[q] = uint4{p[q][0], p[q][1], p[q][2], p[q][3]};
}
// the float of the pieces in the upper halves of h, m and l
__device__ inline float joined(uint32_t h, uint32_t m, uint32_t l)
{
    if (h == kSplitRaw << 16) return __uint_as_float(m | (l >> 16));
    return (__uint_as_float(h) + __uint_as_float(m) + __uint_as_float(l)) * (1.f / kSplitScale);
}
__device__ inline float joined_low(uint32_t h, uint32_t m, uint32_t l) { return joined(h << 16, m << 16, l << 16); }
__device__ inline float joined_high(uint32_t h, uint32_t m, uint32_t l) { return joined(h & 0xffff0000u, m & 0xffff0000u, l & 0xffff0000u); }

// In-register transpose of an 8 (rows q) x 2*NW (16-bit columns) block held as
// rows[q][w] (two columns per 32-bit word) into per-column vectors: column t
// gets the eight row values packed in q order.
template <int NW> __device__ inline void transpose_rows8(const uint32_t (&rows)[8][NW], uint4 (&cols)[2 * NW])
{
    // One byte-permute per output word: v_perm_b32 picks its four bytes from the pair {second, first} operand
    // (selector values 0-3: bytes of the second operand, 4-7: bytes of the first).
    constexpr uint32_t kLow = 0x05040100u;    // low halves:  a.b0 a.b1 b.b0 b.b1
    constexpr uint32_t kHigh = 0x07060302u;   // high halves: a.b2 a.b3 b.b2 b.b3
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        // even column: low halves of each row pair; odd column: high halves
        cols[2 * w].x = __builtin_amdgcn_perm(rows[1][w], rows[0][w], kLow);
        cols[2 * w].y = __builtin_amdgcn_perm(rows[3][w], rows[2][w], kLow);
        cols[2 * w].z = __builtin_amdgcn_perm(rows[5][w], rows[4][w], kLow);
        cols[2 * w].w = __builtin_amdgcn_perm(rows[7][w], rows[6][w], kLow);
        cols[2 * w + 1].x = __builtin_amdgcn_perm(rows[1][w], rows[0][w], kHigh);
        cols[2 * w + 1].y = __builtin_amdgcn_perm(rows[3][w], rows[2][w], kHigh);
        cols[2 * w + 1].z = __builtin_amdgcn_perm(rows[5][w], rows[4][w], kHigh);
        cols[2 * w + 1].w = __builtin_amdgcn_perm(rows[7][w], rows[6][w], kHigh);
    }
}

// Quotient and remainder of small non-negative integers (n, d < 2^22) through one float
// multiplication and a correction step: a handful of instructions where the integer division
// of the instruction set takes some thirty.  rd = frcp(d).
__device__ inline float frcp(int d) { return __builtin_amdgcn_rcpf((float)d); }
__device__ inline void fast_divmod(int n, int d, float rd, int &q, int &r)
{
    q = (int)((float)n * rd);
    r = n - q * d;
    if (r < 0) {
        r += d;
        --q;
    } else if (r >= d) {
        r -= d;
        ++q;
    }
}

// ---------------------------------------------------------------------------
// Z[s]: SplitMix64 in counter form.  Word ctr of the stream of `seed` is
// fin(key + gamma*(ctr+1)) with key = fin(seed + gamma).
// ---------------------------------------------------------------------------
__host__ __device__ inline uint64_t mix_fin(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
__host__ __device__ inline uint64_t stream_word(uint64_t key, uint64_t ctr)
{
    return mix_fin(key + 0x9E3779B97F4A7C15ull * (ctr + 1ull));
}
// `dist` carries the distribution in its low byte and, above it, keep_q15: 0 for dense probes,
// else entry idx is kept with probability keep_q15 / 32768 and zero otherwise (block-sparse
// probing vectors, Eq. (7)); the keep decision compares the top 15 bits of word idx of a
// second stream (seed xor kMaskStream), so kept entries equal those of the dense matrix.
constexpr uint64_t kMaskStream = 0x5851F42D4C957F2Dull;
struct ProbeGen {
    int dist, keep_q15;
    uint64_t key, mkey;
};
__host__ __device__ inline ProbeGen probe_gen(int dist, uint64_t seed)
{
    ProbeGen g;
    g.dist = dist & 0xff;
    g.keep_q15 = dist >> 8;
    g.key = mix_fin(seed + 0x9E3779B97F4A7C15ull);
    g.mkey = mix_fin((seed ^ kMaskStream) + 0x9E3779B97F4A7C15ull);
    return g;
}
// keep decision `block` of block-sparse probing vectors (Eq. (7)); always true for dense probes
__host__ __device__ inline bool probe_keep(const ProbeGen &g, uint64_t block)
{
    return g.keep_q15 == 0 || (int)(stream_word(g.mkey, block) >> 49) < g.keep_q15;
}
__host__ __device__ inline float probe_value(const ProbeGen &g, uint64_t idx);
// entry idx of Z; with block-sparse probes it is zero unless its own keep decision says keep
__host__ __device__ inline float probe_entry(const ProbeGen &g, uint64_t idx)
{
    return probe_keep(g, idx) ? probe_value(g, idx) : 0.0f;
}
__host__ __device__ inline float probe_value(const ProbeGen &g, uint64_t idx)
{
    // +-1: entry idx is bit idx % 64 of word idx / 64 (the bits of a SplitMix64 output are independent fair bits), so one
    // generator word serves 64 entries and a workgroup can draw a whole matrix from a few hundred words
    if (g.dist == XCONV_RADEMACHER) return ((stream_word(g.key, idx >> 6) >> (idx & 63)) & 1ull) ? -1.0f : 1.0f;
    // Box-Muller in double on two 53-bit uniforms, u1 in (0,1], u2 in [0,1)
    const double u1 = ((double)(stream_word(g.key, 2ull * idx) >> 11) + 1.0) * 0x1.0p-53;
    const double u2 = (double)(stream_word(g.key, 2ull * idx + 1ull) >> 11) * 0x1.0p-53;
    return (float)(sqrt(-2.0 * log(u1)) * cos(6.283185307179586476925 * u2));
}

// ---- launch plan of the correlation kernel (host fills, kernel reads) ------
struct CorrArgs {
    const void *dY;    // [B, C_out, Ho, Wo] storage dtype
    const void *A;     // channels-last activation-like tensor [B, H, W, CS] storage dtype (Xt, or X for the exact path)
    float *part;       // [S] partial tiles of fp32 sums, each in the layout of tile_index()
    int B, C_out, H, W, Ho, Wo;
    int kH, kW, sh, sw, ph, pw;
    int CS;            // channel stride of A (multiple of 16)
    int NBG;           // batch groups (BI images each)
    int RB, CW, CWp;   // output rows and columns per step; CWp = CW rounded up to 4
    int NSTRIP, NBAND; // steps per batch group = NSTRIP * NBAND
    int NR, NOLD, NNEW;  // rows of A per step: NR = (RB-1)*sh + kH; NOLD kept from the previous step, NNEW loaded
    int BWc;           // columns of A staged per row = (CWp-1)*sw + kW
    int WM, WJ, WK;    // wave arrangement inside a workgroup (product 4)
    int M_WG, J_WG;    // workgroup tile: output channels and probe columns
    int ASTR, BSTR;    // LDS strides (units) per pixel slot / per staged column
    int NCHR;          // vector chunks of dY staged per row and output channel
    int NTM, NTJ;      // tiles along C_out and along the probe columns
    int S, NS;         // K-splits and total steps
    int SQ, SR;        // NS / S and NS % S (set at launch): workgroup x takes SQ steps, one more if x < SR
    int K2, NOG;       // kernel offsets and offset groups of <= 9
    int MP, JP;        // padded extents of the partial buffer
    int dy_plane;      // elements between consecutive (image, channel) planes of dY as the kernel reads it (whole 16-byte vectors)
    int a_units, b_units;  // LDS units of the two staging tiles
    int AL;            // every staged row segment of dY starts on a 16-byte vector
    // Z[s] for the expansion that follows (Alg. 1 backward step 2): when zout is set, the launch's workgroups
    // each draw a slice of its nz entries from (zdist, zseed) before they start on the correlation
    float *zout;
    int nz, zdist;
    uint64_t zseed;
};
// Volumetric layers: kernel-depth offset `set` is a third extent of the grid and reads A that many bytes further on; its
// partial tiles follow those of the offset before.  One launch with nsets times fewer K-splits each in place of nsets
// launches: the start of a workgroup and the partial tiles are paid once for all of them.  The kernels of 2-D layers take the
// argument without these.
struct DepthSets {
    int nsets, set_sd;
    long long set_run, set_slice;   // bytes of a run of depth slices and of one slice (set_offset)
};
struct CorrParams : CorrArgs, DepthSets {};


// ---- launch plan of the producer/consumer correlation kernel (16-bit storage) ----
struct WsArgs {
    const void *dY;    // [B, C_out, Ho, Wo] storage dtype
    const void *A;     // channels-last [B, H, W, CS] storage dtype
    float *part;       // [S] partial tiles of fp32 sums, each in the layout of tile_index()
    int B, C_out, H, W, Ho, Wo;
    int kH, kW, sh, sw, ph, pw;
    int CS, NBG;            // channel stride of A; groups of 8 images
    int CW, NSTRIP;         // output columns per strip, strips per output row
    int CWs, NSUB;          // output columns per sub-step (multiple of 4), sub-steps per row-step
    int BWc, NRING;         // staged columns per ring row; ring rows (kH + sh)
    int WM, WJ, M_WG, J_WG, NTM, NTJ;
    int S, NS;              // K-splits, row-steps in total (NBG * NSTRIP * Ho)
    int SQ, SR;             // NS / S and NS % S (set at launch): workgroup x takes SQ row-steps, one more if x < SR
    int K2, NOG, MP, JP;
    int a_units;            // LDS units of one dY buffer (CWs * M_WG)
    int b_row_units, BSTR;  // LDS units per ring row, per staged column (J_WG + 1)
    int NA, NA_pad;         // dY tasks per sub-step and the same rounded up to whole waves
    int TS, TB;             // A tasks per sub-step slice, per row-step (sh * BWc * J_WG/8)
    int MT, NTASK;          // 16-row tiles per consumer wave; tasks per producer thread
    // Volumetric layers read dY [Bv, C_out, Do, Ho*Wo] in place: image i of the kernel's batch is depth
    // slot i % vol_period of volume i / vol_period, a zero image when the slot is >= vol_Do.  0: plain dY.
    int vol_period, vol_Do;
    uint32_t vol_bytes;     // bytes of the whole dY tensor (below 2^30)
    // Z[s] for the expansion that follows, drawn by this launch (see CorrParams)
    float *zout;
    int nz, zdist;
    uint64_t zseed;
};
struct WsParams : WsArgs, DepthSets {};
// (with the 24 bytes of DepthSets every estimate of a 2-D layer took 0.2-0.4 us more: C2 36.6 -> 36.9 us for the backward pass)
static_assert(sizeof(CorrArgs) <= 232 && sizeof(WsArgs) <= 232, "arguments of the 2-D correlation kernels");

// (kernel-depth offset, offset group) of a workgroup: the third extent of the grid counts both
__device__ inline void set_and_group(int nog, int &set, int &group)
{
    set = 0;
    group = blockIdx.z;
    while (group >= nog) {
        group -= nog;
        ++set;
    }
}

// Bytes from A to the slices of kernel-depth offset `set`
__device__ inline long long set_offset(int set, int sd, long long run, long long slice)
{
    long long off = 0;
    while (set >= sd) { set -= sd; off += slice; }
    return off + set * run;
}

// Number of K-splits: `target` workgroups or up to a quarter fewer, the count that leaves the fewest idle steps (ties go to the
// smaller count: as many steps per workgroup, fewer partial tiles).  With several kernel-depth offsets per launch only whole
// multiples of 8, which xcd_block needs.
inline int choose_splits(int target, int NS, int nsets)
{
    target = target < 1 ? 1 : target;
    target = target > NS ? NS : target;
    const int step = nsets > 1 && target >= 16 ? 8 : 1;
    int bestS = target / step * step;
    double best_eff = 0.0;
    for (int S = bestS; S >= 1 && S >= target * 3 / 4; S -= step) {
        const double eff = (double)NS / ((double)S * ceil_div(NS, S)) * ((double)S / target);
        if (eff > best_eff - 1e-9) { best_eff = eff > best_eff ? eff : best_eff; bestS = S; }
    }
    return bestS;
}

// Entries wg*threads + tid, + (workgroups * threads), ... of Z[s], drawn by the calling thread (Alg. 1 backward
// step 2: the probing matrix is regenerated from the seed, never stored between the passes).
__device__ inline void draw_z_slice(float *zout, int nz, int dist, uint64_t seed)
{
    if (!zout) return;
    const int nwg = gridDim.x * gridDim.y * gridDim.z;
    const int wg = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const ProbeGen gen = probe_gen(dist, seed);
    for (int i = wg * (int)blockDim.x + (int)threadIdx.x; i < nz; i += nwg * (int)blockDim.x) zout[i] = probe_entry(gen, (uint64_t)i);
}

// Workgroups are handed to the chip's 8 dies in turn (workgroup b runs on die b % 8, each with an L2 of
// its own).  With a grid whose first extent is a multiple of 8 this gives the workgroups of one die neighbouring
// pieces of work (tiles of the probe, K-splits of the correlation: consecutive output rows of one group of images),
// so that a cache line which straddles two pieces (planes and rows are not line-aligned) is fetched from memory
// once, by one L2, instead of once by each of two.
__device__ inline int xcd_block(int b, int grid)
{
    return (grid & 7) == 0 ? (b & 7) * (grid >> 3) + (b >> 3) : b;
}

// ---- forward convolution / exact input gradient as implicit GEMMs (conv_core.h, conv_kernels.hip) ----
constexpr int kConvUnits = 8;   // 16-byte units of channels per staged chunk ...
constexpr int kConvUnitsSplit = 4;   // ... of products whose floats are split (three times 16 bytes each)
constexpr int kConvGatherM = 64;   // output channels that a group of kConvUnits / 2 k-steps of gathered weights covers (no workspace)
constexpr int kConvResident = 128;   // most contraction channels whose whole patch is kept in LDS
constexpr int kConvOverread = 3 * kSplit * 1024; // bytes behind the packed weights that the last requests may touch (three k-steps ahead)
constexpr int kConvSubs = 4;    // classes of output positions per launch ...
constexpr int kConvSubsMany = 16;   // ... of the kernels that take many (conv_many)

// 16-byte entries of a list of k-steps (four steps each, one more that only prefetches touch)
__host__ __device__ inline int conv_step_list(int taps, int steps_per_tap) { return (taps * steps_per_tap + 3) / 4 + 1; }

// Quotients by a number the host knows: one multiplication and a shift (n < 2^31).  For d >= 2 and l = ceil(log2 d),
// m = floor(2^(31+l) / d) + 1 < 2^32 gives floor(n / d) = floor(n m / 2^(31+l)); d = 1 passes n through.
struct FastDiv {
    uint32_t m, pass;
    int sh, d;
    __host__ __device__ int div(int n) const
    {
#ifdef __HIP_DEVICE_COMPILE__
        return (int)((__umulhi((uint32_t)n, m) + ((uint32_t)n & pass)) >> sh);
#else
        return n / d;
#endif
    }
    __host__ __device__ void divmod(int n, int &q, int &r) const
    {
        q = div(n);
        r = n - q * d;
    }
};
inline FastDiv fast_div(int d)
{
    FastDiv f{0, ~0u, 0, d < 1 ? 1 : d};
    if (f.d > 1) {
        int l = 1;
        while ((1LL << l) < f.d) ++l;
        f.m = (uint32_t)((1ull << (31 + l)) / (unsigned)f.d + 1);
        f.pass = 0;
        f.sh = l - 1;
    }
    return f;
}

// One class of output positions: an ordinary convolution with its own taps.  The forward convolution is one class; the
// input gradient of a strided layer is up to sh*sw of them (output positions by their remainder modulo the stride; those that no
// kernel offset reaches are zeros and no class).
struct ConvSub {
    int kH, kW, ph, pw;        // taps and padding in front (negative: the first source row lies inside)
    int Ho, Wo;                // output positions of the class
    int oy0, ox0;              // its first output row and column (the steps are ConvParams::osy, osx)
    int ky0, kx0, kys, kxs;    // kernel offset of tap (i, j): (ky0 + i*kys, kx0 + j*kxs), in the order they are summed
    int SW, TPS, TU;           // columns per strip, tiles per strip, positions per tile
    int sth, stw;              // staged rows (columns) per output row (column): min(stride, taps)
    int PWv, PH, PWs, NPOS, NPPmax;   // staging tasks per patch row, columns per remainder class, LDS positions per row and in all, tasks per unit
    FastDiv dSW, dHo, dHV, dPWv, dTPS, dkW;   // quotients by SW, Ho, staged rows of a whole image, PWv, TPS, kW
    int wgs;                   // workgroups of the class
    int images;                // most images a tile touches (host)
    long long w0;              // first 16-byte unit of its packed weights
};
struct ConvHead {
    const void *in;    // activation-like tensor the contraction runs over (X, or dY for the input gradient)
    const void *w;     // weights [C_out, C_in, kH, kW] in the storage type
    const void *wp;    // the same in fragment order (side_jobs.h), or null: fragments are gathered from w
    const void *bias;  // per output channel in the storage type, or null
    void *out;         // Y, or dX
    int B, Cin, Cout;  // images, contraction channels and output channels of this product
    int Hi, Wi;        // extent of `in`
    int sh, sw;        // stride of the source position (1 for the input gradient)
    int osy, osx;      // output step between the positions of a class
    int kWfull;        // kernel width of w
    long long in_sb, out_sb;                              // element strides: image,
    int in_sc, in_sy, in_sx, out_sc, out_sy, out_sx;      // channel, row, column
    int w_sco, w_sci;                                     // weights: output channel of the product, contraction channel
    int MT, NT, WM;    // 32-row tiles and 32-column tiles per wave, waves along the output channels
    FastDiv dNMT, dks, dksl;   // quotients by NMT and by the k-steps per tap of a full and of the last chunk
    int NMT, NMB;      // tiles of output channels, blocks of 32 packed output channels
    int vec, swap, big;   // how the input is read, which side of the accumulator the channels are on, 64-bit addresses
    int pair;             // 16-bit outputs: neighbouring positions (channels-last: channels) share an aligned 4-byte word
    int rev;              // taps reach back: tap (i, j) reads patch position (kH-1-i, kW-1-j) (input gradient)
    int res;              // all channels of a patch resident
    int nsub, nwg, lds_bytes;
};
// The argument of a launch of up to N classes: one, kConvSubs or kConvSubsMany (3.4 KB: 0.3-0.6 us more per launch than the 1 KB of
// kConvSubs, 27 -> 14 us for the nine classes of 64 -> 32 channels 3x3 at stride 3, 57x57, batch 16, bf16, in one launch for three)
template <int N> struct ConvArgs : ConvHead {
    ConvSub sub[N];
};
typedef ConvArgs<kConvSubsMany> ConvParams;
// tiles and weights of which there are kernels for many classes: the classes of a large stride have few taps each
constexpr bool conv_many(int MT, int NT, bool packed, bool big, bool res) { return MT == NT && !big && (res || !packed); }

// packed floats are multiplied as sums of three bf16 numbers
constexpr bool conv_split(int dtype, bool packed) { return dtype == XCONV_F32 && packed; }
// waves per SIMD that the registers of a kernel leave room for
constexpr int conv_occupancy(int MT, int NT, bool split, bool packed)
{
    return split ? (MT * NT >= 2 ? 3 : 4) : MT * NT >= 8 || !packed ? 2 : MT * NT >= 4 ? 3 : 4;
}

// Small jobs that a launch carries along in workgroups of its own, in place of a launch each (4-6 us on the stream for work
// of 1 us): the weights of a convolution in fragment order, and the sum of the pieces of a bias gradient.  The probe (forward)
// and the second pass of the weight gradient (backward) carry them; the convolution that reads the weights follows.
struct PackClass {
    int kH, kW, ky0, kx0, kys, kxs;   // as in ConvSub
    int n;                            // fragments (64 x 16 bytes)
    long long w0;
};
template <int N> struct PackJobs {
    int total;                        // fragments and channels: one wave each
    int groups;                       // workgroups of the carrying launch that do them, in front of its own
    int nsub, NMB, Cin, Cout, w_sco, w_sci, kWfull;
    int res, es;                      // resident patches, bytes per element
    int C, S, dtype;                  // bias gradient: channels, pieces, storage type
    const void *w;
    void *packed;
    const float *part;
    void *db;
    PackClass sub[N];
};
// Those that other launches carry.  The kernels take them as one more argument, so that a launch without any runs a kernel without
// the code and the argument (C4 estimate 134.5 -> 133.9 us, 133.6 before there were any jobs).
typedef PackJobs<kConvSubs> SideJobs;

}  // namespace xc
