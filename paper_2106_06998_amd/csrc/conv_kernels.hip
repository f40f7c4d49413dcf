// Host side of the forward convolution and the exact input gradient: classes of output positions, tiles, launches
// (the kernels are in conv_core.h).
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <string>
#include <unordered_map>
#include <vector>

#include "common.h"
#include "launch.h"
#include "side_jobs.h"

namespace xc {

hipError_t launch_conv_f32(const ConvHead &P, const ConvSub *sub, hipStream_t st);
hipError_t launch_conv_bf16(const ConvHead &P, const ConvSub *sub, hipStream_t st);
hipError_t launch_conv_f16(const ConvHead &P, const ConvSub *sub, hipStream_t st);

namespace {

constexpr int kLdsMax = 160 * 1024;
constexpr long long kMaxPos = 1LL << 30;       // positions over the batch in one launch (32-bit tile arithmetic)
constexpr long long kMaxReach = 0x7f000000;    // bytes a tile reads or writes from its first image on (32-bit offsets in a 2 GiB buffer descriptor)
constexpr long long kMaxReachBig = 0xfffffffe; // elements of the same with 64-bit addresses (32-bit tables, all ones marks the outside)

// see expected_cycles
struct ConvModel {
    double e24, e22, e12, e11;   // share of the 16-bit matrix rate of the wave tiles (MT, NT)
    double ef32;                 // ... of the fp32 rate
    double task;                 // cycles per staging task
    double in_bpc, out_bpc;      // bytes per cycle and compute unit
    double chunk, overlap;       // k-steps per overlapping step, how completely steps overlap
    double start, per_chunk;     // cycles per round, and per chunk of one
    double alone, pair;          // surcharges for one and two workgroups per unit
    double gather;               // cycles per gathered group of k-steps
};
constexpr ConvModel kConvModel = {0.58, 0.465, 0.55, 0.575, 1.0, 367, 30.7, 15.1, 16, 0.634, 13900, 0, 1.5, 0.145, 600};
constexpr ConvModel kConvModelSplit = {0, 0, 0.656, 0.635, 0, 594, 15.7, 33.6, 1e9, 0.352, 6490, 1870, 0.911, 0, 0};

int env_value(const char *name)
{
    const char *e = getenv(name);
    return e ? atoi(e) : 0;
}
// channels of a staged unit and units of a chunk; packed: with weights in fragment order, so that floats are split
int units_elems(int dtype, bool packed) { return dtype == XCONV_F32 && !conv_split(dtype, packed) ? 4 : 8; }
int chunk_units(int dtype, bool packed) { return conv_split(dtype, packed) ? kConvUnitsSplit : kConvUnits; }
int pieces(int dtype, bool packed) { return conv_split(dtype, packed) ? kSplit : 1; }
int elem_size(int dtype) { return dtype == XCONV_F32 ? 4 : 2; }

void image_strides(int layout, int C, int H, int W, long long &sb, int &sc, int &sy, int &sx)
{
    if (layout == XCONV_NHWC) { sb = (long long)H * W * C; sc = 1; sy = W * C; sx = C; }
    else { sb = (long long)C * H * W; sc = H * W; sy = W; sx = 1; }
}

// classes of output positions of the product
std::vector<ConvSub> make_subs(const xconv_desc *d, int transposed, int Ho, int Wo)
{
    std::vector<ConvSub> v;
    if (!transposed) {
        ConvSub s{};
        s.kH = d->kH; s.kW = d->kW; s.ph = d->pad_h; s.pw = d->pad_w;
        s.Ho = Ho; s.Wo = Wo;
        s.kys = s.kxs = 1;
        v.push_back(s);
        return v;
    }
    // input row iy = a + sh*t takes dY row (iy + ph - ky)/sh where that divides: taps ky = ky0 + sh*i, row t + (a+ph-ky0)/sh - i,
    // i.e. a unit-stride convolution whose taps reach back (ConvParams::rev)
    auto axis = [](int a, int k, int s, int p, int &n, int &first, int &pad) {
        first = (a + p) % s;
        n = first < k ? (k - 1 - first) / s + 1 : 0;
        pad = (n - 1) - (a + p - first) / s;
    };
    for (int a = 0; a < std::min(d->stride_h, d->H); ++a) {
        ConvSub s{};
        axis(a, d->kH, d->stride_h, d->pad_h, s.kH, s.ky0, s.ph);
        if (s.kH == 0) continue;                      // zeros (ConvPlan::fill)
        for (int b = 0; b < std::min(d->stride_w, d->W); ++b) {
            axis(b, d->kW, d->stride_w, d->pad_w, s.kW, s.kx0, s.pw);
            if (s.kW == 0) continue;
            s.kys = d->stride_h; s.kxs = d->stride_w;
            s.oy0 = a; s.ox0 = b;
            s.Ho = (d->H - a + d->stride_h - 1) / d->stride_h;
            s.Wo = (d->W - b + d->stride_w - 1) / d->stride_w;
            v.push_back(s);
        }
    }
    return v;
}

int ksteps(int dtype, bool packed, int C) { return ceil_div(C, 2 * units_elems(dtype, packed)); }
long long packed_units(const ConvSub &s, int dtype, int Cin, int Cout)
{
    return (long long)ceil_div(Cout, 32) * ksteps(dtype, true, Cin) * s.kH * s.kW * 64 * pieces(dtype, true);
}

// LDS of a workgroup: patch, tables, lists of the k-steps, gathered weights (conv_kernel's layout)
long long conv_lds(const ConvParams &P, const ConvSub &c, int dtype, int TN, int nks)
{
    const int units = chunk_units(dtype, P.wp != nullptr), KS = units / 2, np = pieces(dtype, P.wp != nullptr);
    const int taps = c.kH * c.kW;
    const long long tables = (c.NPPmax + TN + 1) / 2 * 16;
    if (P.res) return 2LL * nks * np * c.NPOS * 16 + tables + conv_step_list(taps, nks) * 16;
    if (P.wp) return 2LL * units * np * c.NPOS * 16 + tables + 2 * conv_step_list(taps, KS) * 16;
    const int last = nks - (nks - 1) / KS * KS;
    return (nks > KS ? 2LL * kConvUnits : 2LL * nks) * c.NPOS * 16 + tables +
           ((nks > KS ? round_up(taps * KS, 8) : 0) + round_up(taps * last, 8)) * 8 + 2 * KS * kConvGatherM / 32 * 1024;
}

// What a launch has to do, summed over its workgroups
struct Work {
    double mma = 0;        // 32x32 fragment pairs per wave
    double tasks = 0;      // staging tasks per thread
    double groups = 0;     // gathered groups of k-steps
    double in = 0, out = 0;   // bytes of the cache lines touched (a strip narrower than the image uses lines partly)
    long long wgs = 0;
    int lds = 0;
};

// Lays one class out for tiles of TU of the TN positions on nst strips and adds up its work; false when the patch does not fit
// or a tile's offsets from its first image would not.
bool lay_out(ConvSub &s, const ConvParams &P, int dtype, int nst, int TU, int TN, Work &w)
{
    const int es = elem_size(dtype), nks = ksteps(dtype, P.wp != nullptr, P.Cin), VW = P.vec == 1 ? 2 : 1;
    const int taps = s.kH * s.kW, SW = ceil_div(s.Wo, std::min(nst, s.Wo));
    s.SW = SW;
    s.TU = TU;
    s.sth = std::min(P.sh, s.kH);
    s.stw = std::min(P.sw, s.kW);
    const long long NR = (long long)P.B * s.Ho;
    const bool rows = TU % SW == 0;              // tiles begin at the start of a row
    const int nr = (int)std::min<long long>(rows ? TU / SW : (SW + TU - 2) / SW + 1, NR);
    const int nb = rows && s.Ho % nr == 0 ? 0 : std::min(nr >= 2 ? (nr - 2) / s.Ho + 1 : 0, P.B - 1);
    // (a strip takes a row of every image in turn: a narrow one of images with few rows crosses many of them)
    s.images = nb + 1;
    const long long reach = s.images * std::max(P.in_sb, P.out_sb);
    if (P.big ? reach > kMaxReachBig : reach * es > kMaxReach) return false;
    const int NPR = (nr - 1) * s.sth + nb * (s.kH - s.sth) + s.kH;
    const int PWl = (SW - 1) * s.stw + s.kW + (VW - 1);
    s.PWv = std::max(1, ceil_div(PWl, VW));
    s.PH = ceil_div(s.PWv * VW, s.stw);
    s.PWs = s.stw * s.PH;
    s.NPOS = round_up(NPR * s.PWs, 16);
    s.NPPmax = NPR * s.PWv;
    s.TPS = (int)((NR * SW + TU - 1) / TU);
    const long long lds = conv_lds(P, s, dtype, TN, nks);
    if (lds > kLdsMax || s.NPOS > 65535) return false;
    const double n = (double)ceil_div(s.Wo, SW) * s.TPS * P.NMT;
    const int TM = std::min(32 * P.MT * P.WM, P.Cout);
    const bool cl = P.swap;
    const double in_row = cl ? (double)PWl * P.Cin * es : nst == 1 ? (double)P.Wi * es : PWl * es + 64.0;
    const double out_row = cl ? (double)TU * TM * es : nst == 1 ? TU * es + 32.0 : (double)nr * (SW * es + 48.0);
    w.mma += n * taps * nks * P.MT * P.NT;
    w.groups += n * taps * nks * (P.MT * P.WM) / (kConvUnits / 2 * kConvGatherM / 32);
    w.tasks += n * s.NPPmax * 2.0 * nks / kThreads;
    w.in += n * NPR * in_row * (cl ? 1 : P.Cin);
    w.out += n * out_row * (cl ? 1 : TM);
    w.wgs += (long long)n;
    w.lds = std::max(w.lds, (int)lds);
    return true;
}

// Expected cycles of a launch.  The matrix instructions of the busiest compute unit and its staging and stores (issue or memory,
// whichever is slower) overlap where the unit has several workgroups in turn or a workgroup has several chunks; each round of
// workgroups pays a start-up.  The constants are a fit to the measured times of 3300 tile configurations of 60 products (fp32
// and 16-bit, both layouts, 1x1 to 5x5, strides 1 and 2); picking by them costs 1 % against the best configuration of each.
// Gathered weights add a share for each group (453 products of strides 1 to 4, 1x1 to 7x7, in up to five configurations: 1.8 %;
// 2.0 to 3.3 % with a third of that share up to seven times as much, 5 % without).
// Split floats have constants of their own, a fit to 3087 configurations of 60 layers' two products, resident and in chunks: picking
// by them costs 1.4 % (4.6 % with those of the others and a guess at the rate).
double expected_cycles(const ConvParams &P, int dtype, const Work &w, int ncu)
{
    const bool packed = P.wp != nullptr, split = conv_split(dtype, packed);
    const int shape = P.MT * 10 + P.NT, nks = ksteps(dtype, packed, P.Cin);
    const ConvModel &m = split ? kConvModelSplit : kConvModel;
    const double eff = shape == 24 ? m.e24 : shape == 22 ? m.e22 : shape == 12 ? m.e12 : m.e11;
    const double clk = split ? 32.0 * kSplitProducts / eff : dtype == XCONV_F32 ? 256.0 / m.ef32 : 32.0 / eff;
    const int occ = std::max(1, std::min(kLdsMax / w.lds, packed ? conv_occupancy(P.MT, P.NT, split, true) : P.MT * P.NT >= 4 ? 2 : 3));
    const double q = (double)((w.wgs + ncu - 1) / ncu), rounds = (double)((w.wgs + (long long)ncu * occ - 1) / ((long long)ncu * occ));
    const double tm = w.mma / w.wgs * clk * q;
    const double ts = std::max(w.tasks / w.wgs * m.task * q, w.in / ncu / m.in_bpc) + w.out / ncu / m.out_bpc;
    const double steps = rounds * (P.res ? 1.0 : std::max(1.0, nks / m.chunk));
    double t = m.start * rounds + std::max(tm, ts) + std::min(tm, ts) / std::pow(steps, m.overlap);
    if (split && !P.res) t += m.per_chunk * rounds * ((nks + kConvUnitsSplit / 2 - 1) / (kConvUnitsSplit / 2));
    if (!P.wp) t += m.gather * w.groups / w.wgs * q;
    if (occ == 1) t += m.alone * ts;
    if (occ == 2) t += m.pair * tm;
    return t;
}

// the tiles of the least expected time, which is returned; -1 where none fits
double plan(ConvParams &P, int dtype, int ncu)
{
    const int force = env_value("XCONV_CONV_SHAPE"), force_wm = env_value("XCONV_CONV_WM");
    const int force_strips = env_value("XCONV_CONV_STRIPS"), force_rows = env_value("XCONV_CONV_ROWS");
    const bool packed = P.wp != nullptr, split = conv_split(dtype, packed);
    const int units = chunk_units(dtype, packed), nks = ksteps(dtype, packed, P.Cin);
    int wide = 1;
    for (int i = 0; i < P.nsub; ++i) wide = std::max(wide, P.sub[i].Wo);
    double best = -1;
    ConvParams bp = P;
    // tiles of TN positions or of whole rows only (fewer positions, but no partly used row and halo); only where no patch fits
    // (large strides or kernels on narrow images), less
    for (int part = 1; part <= 512 && (best < 0 || (split && part <= 2)); part *= 2)
        for (const int shape : {24, 22, 12, 11})
            for (int WM = 1; WM <= 4; WM *= 2) {
                ConvParams C = P;
                C.MT = shape / 10; C.NT = shape % 10; C.WM = WM;
                const int TM = 32 * C.MT * WM, TN = 32 * C.NT * (4 / WM);
                if (split && shape > 12) continue;
                if (force && !P.big && (packed || force != 24) && !(split && force > 12) && P.nsub <= kConvSubs && shape != force) continue;
                if (force_wm && WM != force_wm) continue;
                if (!P.wp && (C.NT > 2 || (WM > 1 && shape != 11))) continue;   // (the gathers there are)
                if (P.big && shape != 22) continue;
                if (P.nsub > kConvSubs && !conv_many(C.MT, C.NT, P.wp != nullptr, P.big, P.res)) continue;
                if (WM > 1 && TM / 2 >= P.Cout) continue;                           // half of the waves would have no channels
                if (TN / part < 1) continue;
                C.NMT = ceil_div(P.Cout, TM);
                // whole rows, then every width of strips from 2 TN columns down (a tile stages two rows of a wider one, most of them
                // for nothing), so that the search does not grow with the image: a 1x1 layer on 10000 x 10000 took 490 ms, now 0.3
                for (int nst = 0, SW = wide + 1; SW > 1;) {
                    nst = nst == 0 ? 1 : std::max(ceil_div(wide, SW - 1), ceil_div(wide, 2 * TN));
                    SW = ceil_div(wide, nst);
                    if (part == 1 && nst > 1 && SW < 8) break;
                    for (int rows = 0; rows < 2; ++rows) {
                        int TU = TN / part;
                        if (force_strips && part == 1 && (nst != force_strips || rows != force_rows)) continue;
                        if (rows) {
                            if (TU % SW == 0 || SW > TU) continue;
                            TU = TU / SW * SW;
                        }
                        Work w;
                        bool fits = true;
                        long long most = 0;      // workgroups of the largest class
                        for (int i = 0; i < P.nsub && fits; ++i) {
                            C.sub[i] = P.sub[i];
                            const long long before = w.wgs;
                            fits = lay_out(C.sub[i], C, dtype, nst, TU, TN, w);
                            most = std::max(most, w.wgs - before);
                            fits = fits && most * P.nsub < 0x3fffffff;
                            C.sub[i].wgs = (int)(w.wgs - before);
                        }
                        if (!fits) continue;
                        const double t = expected_cycles(C, dtype, w, ncu);
                        if (best >= 0 && t >= best) continue;
                        best = t;
                        bp = C;
                        bp.nwg = (int)(most * P.nsub);
                        bp.lds_bytes = w.lds;
                    }
                }
            }
    if (best < 0) return best;
    P = bp;
    P.dNMT = fast_div(P.NMT);
    P.dks = fast_div(P.res ? nks : units / 2);
    P.dksl = fast_div(P.res ? nks : nks - (nks - 1) / (units / 2) * (units / 2));
    for (int i = 0; i < P.nsub; ++i) {
        ConvSub &s = P.sub[i];
        s.dSW = fast_div(s.SW); s.dHo = fast_div(s.Ho); s.dHV = fast_div((s.Ho - 1) * s.sth + s.kH);
        s.dPWv = fast_div(s.PWv); s.dTPS = fast_div(s.TPS); s.dkW = fast_div(s.kW);
    }
    return best;
}

}  // namespace

// every kernel offset belongs to one class at most
size_t conv_ws_bytes(const xconv_desc *d, int transposed)
{
    const int Cin = transposed ? d->C_out : d->C_in, Cout = transposed ? d->C_in : d->C_out;
    return (size_t)ceil_div(Cout, 32) * ksteps(d->dtype, true, Cin) * d->kH * d->kW * 64 * 16 * pieces(d->dtype, true) + kConvOverread;
}

// One launch of a product: a class group of a run of images.  The pointers of P are filled in per call.
struct ConvLaunch {
    ConvParams P;
    size_t in_off, out_off;   // bytes of the run's first image
    bool pack;                // the weights of these classes are packed in front of it
};
struct ConvPlan {
    int dtype;
    size_t fill;                      // bytes of the output, cleared in front of the launches where no kernel offset reaches some of it; else 0
    std::vector<ConvLaunch> launches;
};

namespace {

std::mutex g_conv_mu;
// plans by their key (the raw integers), handed out by reference; emptied when a program has gone through very many shapes
std::unordered_map<std::string, std::shared_ptr<const ConvPlan>> g_conv_plans;
constexpr size_t kConvPlans = 4096;

int device_cus()
{
    static int cus[64] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
    if (!cus[dev] && (hipDeviceGetAttribute(&cus[dev], hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus[dev] <= 0)) cus[dev] = 256;
    return cus[dev];
}

// align, oalign: alignment of the input and the output pointer in bytes, up to 16
bool make_plan(ConvPlan &out, const xconv_desc *d, int transposed, bool packed, int align, int oalign, int ncu)
{
    // a 1x1 convolution at unit stride knows no rows: one row of H*W positions per image
    xconv_desc flat = *d;
    if (d->kH == 1 && d->kW == 1 && d->stride_h == 1 && d->stride_w == 1 && d->pad_h == 0 && d->pad_w == 0) {
        flat.W = d->H * d->W;
        flat.H = 1;
        d = &flat;
    }
    const int Ho = (d->H + 2 * d->pad_h - d->kH) / d->stride_h + 1, Wo = (d->W + 2 * d->pad_w - d->kW) / d->stride_w + 1;
    const int es = elem_size(d->dtype), ue = units_elems(d->dtype, packed), units = chunk_units(d->dtype, packed);
    ConvParams P{};
    P.Cin = transposed ? d->C_out : d->C_in;
    P.Cout = transposed ? d->C_in : d->C_out;
    P.Hi = transposed ? Ho : d->H;
    P.Wi = transposed ? Wo : d->W;
    const int Hout = transposed ? d->H : Ho, Wout = transposed ? d->W : Wo;
    P.sh = transposed ? 1 : d->stride_h;
    P.sw = transposed ? 1 : d->stride_w;
    P.osy = transposed ? d->stride_h : 1;
    P.osx = transposed ? d->stride_w : 1;
    P.kWfull = d->kW;
    P.rev = transposed;
    image_strides(d->layout, P.Cin, P.Hi, P.Wi, P.in_sb, P.in_sc, P.in_sy, P.in_sx);
    image_strides(d->layout, P.Cout, Hout, Wout, P.out_sb, P.out_sc, P.out_sy, P.out_sx);
    P.w_sco = transposed ? d->kH * d->kW : d->C_in * d->kH * d->kW;
    P.w_sci = transposed ? d->C_in * d->kH * d->kW : d->kH * d->kW;
    P.NMB = ceil_div(P.Cout, 32);
    const bool nhwc = d->layout == XCONV_NHWC;
    P.swap = nhwc;
    std::vector<ConvSub> subs = make_subs(d, transposed, Ho, Wo);
    long long covered = 0, w0 = 0;
    for (const ConvSub &s : subs) covered += (long long)s.Ho * s.Wo;
    out.fill = covered < (long long)Hout * Wout ? (size_t)d->B * P.out_sb * es : 0;
    for (ConvSub &s : subs) {
        s.w0 = w0;
        w0 += packed_units(s, d->dtype, P.Cin, P.Cout);
    }
    // images per launch: 32-bit row and tile arithmetic
    const int bstep = (int)std::max<long long>(1, std::min<long long>(d->B, kMaxPos / ((long long)Hout * Wout)));
    // 64-bit addresses for images past the descriptor, and for few channels on very large planes: lanes past the last channel are
    // masked by an offset past the descriptor, but the scalar offset of their channel, up to a whole unit or block, counts as
    // well, and the hardware's bounds check subtracts it from the size.  (Stopping it at the last channel in the kernel cost the 1x1
    // layers 2-4 %.)
    const int in_ch = round_up(P.Cin, P.Cin > units * ue ? units * ue : 2 * ue);
    const bool huge = std::max(P.in_sb, P.out_sb) * es > kMaxReach || (long long)in_ch * P.in_sc * es > kMaxReach ||
                      (long long)round_up(P.Cout, 32) * P.out_sc * es > kMaxReach;
    // (an image that fits 32-bit offsets never needs 64-bit addresses, and patches of so few channels are resident: a tile of one
    // position fits)
    const size_t per = !huge && (!packed || P.Cin <= kConvResident) ? kConvSubsMany : kConvSubs;
    for (size_t s0 = 0; s0 < subs.size(); s0 += per) {
        P.nsub = (int)std::min<size_t>(per, subs.size() - s0);
        for (int i = 0; i < P.nsub; ++i) P.sub[i] = subs[s0 + i];
        for (int bb = 0; bb < d->B; bb += bstep) {
            P.B = std::min(bstep, d->B - bb);
            // 32-bit offsets where an image fits them and a tile layout does that keeps to few enough images (lay_out); 64-bit
            // addresses otherwise.  Further runs take the kernel of the first, which the weights are packed for: what fits that
            // many images fits fewer
            const ConvLaunch *first = bb ? &out.launches.back() : nullptr;
            ConvLaunch L{};
            bool found = false;
            for (int big = first ? first->P.big : huge; big <= (first ? first->P.big : 1) && !found; ++big) {
                P.big = big;
                P.vec = 0;
                if (!P.big && nhwc && P.Cin % (16 / es) == 0 && align % 16 == 0) P.vec = 2;
                bool pairs = !P.big && !nhwc && es == 2 && P.Wi % 2 == 0 && align % 4 == 0;
                for (int i = 0; i < P.nsub; ++i) pairs = pairs && P.sub[i].kW >= P.sw;
                if (pairs) P.vec = 1;
                double best = -1;
                for (int res = first ? first->P.res : packed && !big && P.Cin <= kConvResident; res >= (first ? first->P.res : 0); --res) {
                    ConvParams C = P;
                    C.wp = packed && !P.big ? &out : nullptr;   // only whether it is set counts here
                    C.res = res;
                    const double t = plan(C, d->dtype, ncu);
                    if (t < 0 || (found && t >= best)) continue;
                    best = t;
                    L.P = C;
                    found = true;
                    if (!conv_split(d->dtype, C.wp != nullptr)) break;   // (a resident patch that fits is the better one)
                }
            }
            if (!found) return false;
            // words of two outputs: channels-last, neighbouring channels; planes, neighbouring columns of an even strip of a unit-step class
            L.P.pair = es == 2 && !L.P.big && oalign % 4 == 0 && (nhwc ? P.Cout % 2 == 0 : P.osx == 1 && Wout % 2 == 0);
            for (int i = 0; i < P.nsub && !nhwc; ++i) L.P.pair = L.P.pair && L.P.sub[i].SW % 2 == 0 && L.P.sub[i].TU % 2 == 0;
            L.in_off = (size_t)bb * P.in_sb * es;
            L.out_off = (size_t)bb * P.out_sb * es;
            L.pack = L.P.wp && bb == 0;
            out.launches.push_back(L);
        }
    }
    return true;
}

std::shared_ptr<const ConvPlan> conv_plan(const xconv_desc *d, int transposed, bool packed, int align, int oalign)
try {
    const int ncu = device_cus();
    // (the overrides of tests and sweeps are part of the key)
    const int key[24] = {d->B, d->C_in, d->C_out, d->H, d->W, d->kH, d->kW, d->stride_h, d->stride_w, d->pad_h, d->pad_w, d->dtype, d->layout,
                         transposed, packed, align, ncu, env_value("XCONV_CONV_SHAPE"), env_value("XCONV_CONV_WM"), oalign,
                         env_value("XCONV_CONV_STRIPS"), env_value("XCONV_CONV_ROWS"), 0, 0};
    const std::string k(reinterpret_cast<const char *>(key), sizeof(key));
    {
        std::lock_guard<std::mutex> lk(g_conv_mu);
        const auto it = g_conv_plans.find(k);
        if (it != g_conv_plans.end()) return it->second;
    }
    auto p = std::make_shared<ConvPlan>();
    p->dtype = d->dtype;
    if (!make_plan(*p, d, transposed, packed, align, oalign, ncu)) return nullptr;
    std::lock_guard<std::mutex> lk(g_conv_mu);
    if (g_conv_plans.size() >= kConvPlans) g_conv_plans.clear();
    g_conv_plans.emplace(k, p);
    return p;
} catch (...) {
    return nullptr;      // out of host memory: the entry points are C
}

}  // namespace

bool conv_plan_info(const xconv_desc *d, int transposed, bool packed, int32_t *out)
{
    const auto p = conv_plan(d, transposed, packed, 16, 4);
    if (!p) return false;
    int npack = 0;
    const ConvLaunch *worst = nullptr;
    const ConvSub *cls = nullptr;
    for (const ConvLaunch &L : p->launches) {
        npack += L.pack;
        for (int i = 0; i < L.P.nsub; ++i)
            if (!cls || L.P.sub[i].images > cls->images) { worst = &L; cls = &L.P.sub[i]; }
    }
    if (!cls) {      // nothing but zeros
        std::fill(out, out + 16, 0);
        return true;
    }
    const ConvParams &P = worst->P;
    const int32_t v[16] = {(int32_t)p->launches.size(), npack, P.MT * 10 + P.NT, P.WM, P.res, P.big, P.vec, P.pair,
                           P.nsub, P.B, cls->Ho, cls->Wo, cls->SW, cls->TU, cls->images, P.lds_bytes};
    std::copy(v, v + 16, out);
    return true;
}

// the jobs alone in a launch
template <int N> __global__ __launch_bounds__(kThreads) void side_jobs_kernel(const PackJobs<N> J) { side_jobs<0, kThreads>(J, blockIdx.x, gridDim.x); }

template <int N> static hipError_t launch_jobs(const PackJobs<N> &J, hipStream_t st)
{
    if (J.total <= 0) return hipSuccess;
    hipLaunchKernelGGL(side_jobs_kernel<N>, dim3((unsigned)side_groups<kThreads>(&J)), dim3(kThreads), 0, st, J);
    return hipGetLastError();
}

hipError_t launch_side_jobs(const SideJobs &J, hipStream_t st) { return launch_jobs(J, st); }

ConvPlanRef find_conv_plan(const xconv_desc *d, int transposed, const void *in, const void *out, bool packed)
{
    const uintptr_t ia = reinterpret_cast<uintptr_t>(in);
    return conv_plan(d, transposed, packed, ia % 16 == 0 ? 16 : ia % 4 == 0 ? 4 : 2, reinterpret_cast<uintptr_t>(out) % 4 == 0 ? 4 : 2);
}

// the packing of one launch's weights as a job
template <int N> static void add_pack_job(PackJobs<N> &J, const ConvLaunch &L, int dtype, const void *w, void *ws)
{
    const ConvParams &P = L.P;
    J.nsub = P.nsub;
    J.NMB = P.NMB; J.Cin = P.Cin; J.Cout = P.Cout; J.w_sco = P.w_sco; J.w_sci = P.w_sci; J.kWfull = P.kWfull; J.res = P.res;
    J.es = elem_size(dtype);
    J.w = w;
    J.packed = ws;
    const int nks = ksteps(dtype, true, P.Cin);
    for (int i = 0; i < P.nsub; ++i) {
        const ConvSub &s = P.sub[i];
        J.sub[i] = PackClass{s.kH, s.kW, s.ky0, s.kx0, s.kys, s.kxs, P.NMB * nks * s.kH * s.kW, s.w0};
        J.total += J.sub[i].n;
    }
}

bool conv_pack_job(const ConvPlan &plan, const void *w, void *ws, SideJobs &J)
{
    const ConvLaunch *one = nullptr;
    for (const ConvLaunch &L : plan.launches) {
        if (!L.pack) continue;
        if (one || L.P.nsub > kConvSubs) return false;      // more classes than a job holds
        one = &L;
    }
    if (!one) return false;
    add_pack_job(J, *one, plan.dtype, w, ws);
    return true;
}

// zeros; words of 16 bytes between the first and the last that are whole
__global__ __launch_bounds__(kThreads) void zero_fill_kernel(char *out, size_t n)
{
    const size_t head = std::min<size_t>(-reinterpret_cast<uintptr_t>(out) & 15u, n), words = (n - head) / 16;
    const size_t i0 = (size_t)blockIdx.x * kThreads + threadIdx.x, step = (size_t)gridDim.x * kThreads;
    uint4 *w = reinterpret_cast<uint4 *>(out + head);
    for (size_t i = i0; i < words; i += step) w[i] = uint4{0, 0, 0, 0};
    if (i0 < head) out[i0] = 0;
    for (size_t i = head + words * 16 + i0; i < n; i += step) out[i] = 0;
}

hipError_t launch_conv(const ConvPlan &plan, const void *in, const void *w, const void *bias, void *out, void *ws, bool packed, hipStream_t st)
{
    if (plan.fill) {
        hipLaunchKernelGGL(zero_fill_kernel, dim3((unsigned)std::min<size_t>((plan.fill + kThreads * 64 - 1) / (kThreads * 64), 2048)), dim3(kThreads), 0, st,
                           static_cast<char *>(out), plan.fill);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    for (const ConvLaunch &L : plan.launches) {
        hipError_t e = hipSuccess;
        if (L.pack && !packed) {
            if (L.P.nsub > kConvSubs) {
                PackJobs<kConvSubsMany> J{};
                add_pack_job(J, L, plan.dtype, w, ws);
                e = launch_jobs(J, st);
            } else {
                SideJobs J{};
                add_pack_job(J, L, plan.dtype, w, ws);
                e = launch_jobs(J, st);
            }
            if (e != hipSuccess) return e;
        }
        ConvHead P = L.P;
        P.in = static_cast<const char *>(in) + L.in_off;
        P.out = static_cast<char *>(out) + L.out_off;
        P.w = w;
        P.bias = bias;
        P.wp = P.wp ? ws : nullptr;
        e = plan.dtype == XCONV_F32 ? launch_conv_f32(P, L.P.sub, st) : plan.dtype == XCONV_BF16 ? launch_conv_bf16(P, L.P.sub, st) : launch_conv_f16(P, L.P.sub, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace xc
