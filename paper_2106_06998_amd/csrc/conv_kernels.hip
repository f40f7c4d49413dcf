// Host side of the forward convolution and the exact input gradient: classes of output positions, tiles, launches
// (the kernels are in conv_core.h).
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <mutex>
#include <vector>

#include "common.h"
#include "launch.h"

namespace xc {

hipError_t launch_conv_f32(const ConvParams &P, hipStream_t st);
hipError_t launch_conv_bf16(const ConvParams &P, hipStream_t st);
hipError_t launch_conv_f16(const ConvParams &P, hipStream_t st);
hipError_t launch_conv_pack_f32(const ConvParams &P, void *out, hipStream_t st);
hipError_t launch_conv_pack_bf16(const ConvParams &P, void *out, hipStream_t st);
hipError_t launch_conv_pack_f16(const ConvParams &P, void *out, hipStream_t st);

namespace {

constexpr int kLdsMax = 160 * 1024;
constexpr long long kMaxPos = 1LL << 30;       // positions over the batch in one launch (32-bit tile arithmetic)

int units_elems(int dtype) { return dtype == XCONV_F32 ? 4 : 8; }
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
    for (int a = 0; a < std::min(d->stride_h, d->H); ++a)
        for (int b = 0; b < std::min(d->stride_w, d->W); ++b) {
            ConvSub s{};
            axis(a, d->kH, d->stride_h, d->pad_h, s.kH, s.ky0, s.ph);
            axis(b, d->kW, d->stride_w, d->pad_w, s.kW, s.kx0, s.pw);
            if (s.kH == 0 || s.kW == 0) s.kH = s.kW = s.ph = s.pw = 0;
            s.kys = d->stride_h; s.kxs = d->stride_w;
            s.oy0 = a; s.ox0 = b;
            s.Ho = (d->H - a + d->stride_h - 1) / d->stride_h;
            s.Wo = (d->W - b + d->stride_w - 1) / d->stride_w;
            v.push_back(s);
        }
    return v;
}

int ksteps(int dtype, int C) { return ceil_div(C, 2 * units_elems(dtype)); }
long long packed_units(const ConvSub &s, int dtype, int Cin, int Cout)
{
    return (long long)ceil_div(Cout, 32) * ksteps(dtype, Cin) * s.kH * s.kW * 64;
}

// LDS of a workgroup: patch, tables, step lists (conv_kernel's layout; gathered weights come on top)
long long conv_lds(const ConvParams &P, const ConvSub &c, int TN, int nks)
{
    const int taps = c.kH * c.kW;
    return (P.res ? 2LL * nks : 2LL * kConvUnits) * c.NPOS * 16 + (c.NPPmax + TN + 1) / 2 * 16 +
           (P.res ? conv_step_list(taps, nks) : 2 * conv_step_list(taps, kConvUnits / 2)) * 16;
}

// Strips and LDS extents of a class for tiles of TN positions: the strip width with the least work in all (products for
// positions of ragged tiles and strips, staging of the halo).  Returns the cost per launch in cycles of one compute unit.
double plan_sub(ConvSub &s, const ConvParams &P, int TN, double mma_clk, int nks, int lds_max)
{
    const int VW = P.vec == 1 ? 2 : 1;
    const int taps = s.kH * s.kW;
    double best = -1;
    // fewer positions per tile only where the patch of a full tile does not fit (large strides or kernels on narrow images)
    for (int TU = TN; TU >= 1 && best < 0; TU /= 2) {
        ConvSub bs = s;
        for (int nst = 1; nst <= s.Wo; ++nst) {
            const int SW = ceil_div(s.Wo, nst);
            if (nst > 1 && SW < 8 && TU == TN) break;
            if (nst > 1 && ceil_div(s.Wo, SW) != nst) continue;
            ConvSub c = s;
            c.SW = SW;
            c.TU = TU;
            c.sth = std::max(1, std::min(P.sh, s.kH));
            c.stw = std::max(1, std::min(P.sw, s.kW));
            const long long NR = (long long)P.B * s.Ho;
            const int nr = (int)std::min<long long>((SW + TU - 2) / SW + 1, NR);
            const int nb = std::min(nr >= 2 ? (nr - 2) / s.Ho + 1 : 0, P.B - 1);
            const int NPR = std::max(1, (nr - 1) * c.sth + nb * std::max(0, s.kH - c.sth) + s.kH);
            const int PWl = (SW - 1) * c.stw + s.kW + (VW - 1);
            c.PWv = std::max(1, ceil_div(PWl, VW));
            c.PH = ceil_div(c.PWv * VW, c.stw);
            c.PWs = c.stw * c.PH;
            c.NPOS = round_up(NPR * c.PWs, 16);
            c.NPPmax = NPR * c.PWv;
            c.TPS = (int)((NR * SW + TU - 1) / TU);
            if (conv_lds(P, c, TN, nks) > lds_max || c.NPOS > 65535) continue;
            const double ntask = (double)c.NPPmax * 2 * nks / kThreads;
            const double cost = (double)nst * c.TPS * (taps * nks * mma_clk + ntask * 120.0 + 2500.0);
            if (best < 0 || cost < best) { best = cost; bs = c; }
        }
        s = bs;
    }
    return best;
}

struct Shape { int MT, NT; double eff; };
// wave tiles of the kernel, with the share of the matrix rate each was measured at on large layers (16-bit storage)
const Shape kShapes[] = {{2, 4, 0.60}, {2, 2, 0.45}, {1, 2, 0.33}, {1, 1, 0.22}};

bool plan(ConvParams &P, int dtype, int ncu)
{
    int force = 0, force_wm = 0;
    if (const char *e = getenv("XCONV_CONV_SHAPE")) force = atoi(e);
    if (const char *e = getenv("XCONV_CONV_WM")) force_wm = atoi(e);
    const int nks = ksteps(dtype, P.Cin);
    double best = -1;
    ConvParams bp = P;
    for (const Shape &sh : kShapes)
        for (int WM = 1; WM <= 4; WM *= 2) {
            if (force && !P.big && (P.wp || force != 24) && sh.MT * 10 + sh.NT != force) continue;
            if (force_wm && WM != force_wm) continue;
            if (!P.wp && (sh.NT > 2 || 32 * sh.MT * WM > kConvGatherM)) continue;
            if (P.big && sh.MT * sh.NT != 4) continue;
            if (WM > 1 && 32 * sh.MT * (WM / 2) >= P.Cout) continue;         // half of the waves would have no channels
            ConvParams C = P;
            C.MT = sh.MT; C.NT = sh.NT; C.WM = WM;
            const int extra = P.wp ? 0 : 2 * (kConvUnits / 2) * sh.MT * WM * 1024;   // LDS of the gathered weights
            const int TM = 32 * sh.MT * WM, TN = 32 * sh.NT * (4 / WM);
            C.NMT = ceil_div(P.Cout, TM);
            // cycles of a wave's products of one k-step
            const double per = sh.MT * sh.NT * (dtype == XCONV_F32 ? 256.0 / 0.85 : 32.0 / sh.eff);
            double cost = 0;
            long long nwg = 0;
            int lds = 0;
            bool ok = true;
            for (int i = 0; i < P.nsub && ok; ++i) {
                const double c = plan_sub(C.sub[i], C, TN, per, nks, kLdsMax - extra);
                if (c < 0) { ok = false; break; }
                cost += c * C.NMT;
                C.sub[i].wg0 = (int)nwg;
                nwg += (long long)ceil_div(C.sub[i].Wo, C.sub[i].SW) * C.sub[i].TPS * C.NMT;
                lds = std::max(lds, (int)conv_lds(P, C.sub[i], TN, nks) + extra);
            }
            if (!ok || nwg > 0x3fffffff) continue;
            C.nwg = (int)nwg;
            C.lds_bytes = lds;
            // average workgroup times the workgroups of the busiest compute unit
            const double rounds = (double)((nwg + ncu - 1) / ncu);
            double t = cost / nwg * rounds;
            if (rounds < 2 || lds > kLdsMax / 2) t *= 1.3;               // one wave per SIMD: its latencies are not covered
            if (best < 0 || t < best) { best = t; bp = C; }
        }
    if (best < 0) return false;
    P = bp;
    return true;
}

}  // namespace

size_t conv_ws_bytes(const xconv_desc *d, int transposed)
{
    const int Ho = (d->H + 2 * d->pad_h - d->kH) / d->stride_h + 1, Wo = (d->W + 2 * d->pad_w - d->kW) / d->stride_w + 1;
    long long n = 0;
    for (const ConvSub &s : make_subs(d, transposed, Ho, Wo))
        n += packed_units(s, d->dtype, transposed ? d->C_out : d->C_in, transposed ? d->C_in : d->C_out);
    return (size_t)n * 16 + kConvOverread;
}

namespace {

// One launch of a product: a class group of a run of images.  The pointers of P are filled in per call.
struct ConvLaunch {
    ConvParams P;
    size_t in_off, out_off;   // bytes of the run's first image
    bool pack;                // the weights of these classes are packed in front of it
};
struct ConvPlan {
    int key[20];
    std::vector<ConvLaunch> launches;
};
std::mutex g_conv_mu;
std::vector<std::shared_ptr<const ConvPlan>> g_conv_plans;   // the last 64 products, handed out by reference
constexpr size_t kConvPlans = 64;

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
    const int Ho = (d->H + 2 * d->pad_h - d->kH) / d->stride_h + 1, Wo = (d->W + 2 * d->pad_w - d->kW) / d->stride_w + 1;
    const int es = elem_size(d->dtype), ue = units_elems(d->dtype);
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
    long long w0 = 0;
    for (ConvSub &s : subs) {
        s.w0 = w0;
        w0 += packed_units(s, d->dtype, P.Cin, P.Cout);
    }
    // images per launch: 32-bit row and tile arithmetic
    const int bstep = (int)std::max<long long>(1, std::min<long long>(d->B, kMaxPos / ((long long)Hout * Wout)));
    for (size_t s0 = 0; s0 < subs.size(); s0 += kConvSubs) {
        P.nsub = (int)std::min<size_t>(kConvSubs, subs.size() - s0);
        for (int i = 0; i < P.nsub; ++i) P.sub[i] = subs[s0 + i];
        for (int bb = 0; bb < d->B; bb += bstep) {
            P.B = std::min(bstep, d->B - bb);
            // a tile reads the images of at most 512 positions: offsets from its first image fit a 2 GiB buffer descriptor
            // unless a few images exceed that
            const long long span = (512 / std::max(1, (Hout / P.osy) * (Wout / P.osx)) + 2) * std::max(P.in_sb, P.out_sb) * es;
            P.big = span >= 0x7f000000LL;
            P.vec = 0;
            if (!P.big && nhwc && P.Cin % ue == 0 && align % 16 == 0) P.vec = 2;
            bool pairs = !P.big && !nhwc && es == 2 && P.Wi % 2 == 0 && align % 4 == 0;
            for (int i = 0; i < P.nsub; ++i) pairs = pairs && P.sub[i].kW >= P.sw;
            if (pairs) P.vec = 1;
            ConvLaunch L{};
            L.P = P;
            L.P.wp = packed && !P.big ? &out : nullptr;   // only whether it is set counts here
            L.P.res = L.P.wp && P.Cin <= kConvResident;
            if (!plan(L.P, d->dtype, ncu)) {
                L.P.res = 0;
                if (!plan(L.P, d->dtype, ncu)) return false;
            }
            // words of two outputs: channels-last, neighbouring channels; planes, neighbouring columns of an even strip of a unit-step class
            L.P.pair = es == 2 && !P.big && oalign % 4 == 0 && (nhwc ? P.Cout % 2 == 0 : P.osx == 1 && Wout % 2 == 0);
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
{
    const char *fs = getenv("XCONV_CONV_SHAPE"), *fw = getenv("XCONV_CONV_WM");   // overrides of tests and sweeps
    const int ncu = device_cus();
    const int key[20] = {d->B, d->C_in, d->C_out, d->H, d->W, d->kH, d->kW, d->stride_h, d->stride_w, d->pad_h, d->pad_w, d->dtype, d->layout,
                         transposed, packed, align, ncu, fs ? atoi(fs) : 0, fw ? atoi(fw) : 0, oalign};
    {
        std::lock_guard<std::mutex> lk(g_conv_mu);
        for (const auto &p : g_conv_plans)
            if (memcmp(p->key, key, sizeof(key)) == 0) return p;
    }
    auto p = std::make_shared<ConvPlan>();
    memcpy(p->key, key, sizeof(key));
    if (!make_plan(*p, d, transposed, packed, align, oalign, ncu)) return nullptr;
    std::lock_guard<std::mutex> lk(g_conv_mu);
    if (g_conv_plans.size() >= kConvPlans) g_conv_plans.erase(g_conv_plans.begin());
    g_conv_plans.push_back(p);
    return p;
}

}  // namespace

hipError_t launch_conv(const xconv_desc *d, int transposed, const void *in, const void *w, const void *bias, void *out, void *ws,
                       hipStream_t st)
{
    const uintptr_t ia = reinterpret_cast<uintptr_t>(in);
    const auto plan = conv_plan(d, transposed, ws != nullptr, ia % 16 == 0 ? 16 : ia % 4 == 0 ? 4 : 2, reinterpret_cast<uintptr_t>(out) % 4 == 0 ? 4 : 2);
    if (!plan) return hipErrorInvalidConfiguration;
    for (const ConvLaunch &L : plan->launches) {
        ConvParams P = L.P;
        P.in = static_cast<const char *>(in) + L.in_off;
        P.out = static_cast<char *>(out) + L.out_off;
        P.w = w;
        P.bias = bias;
        P.wp = P.wp ? ws : nullptr;
        hipError_t e = hipSuccess;
        if (L.pack) {
            e = d->dtype == XCONV_F32 ? launch_conv_pack_f32(P, ws, st) : d->dtype == XCONV_BF16 ? launch_conv_pack_bf16(P, ws, st) : launch_conv_pack_f16(P, ws, st);
            if (e != hipSuccess) return e;
        }
        e = d->dtype == XCONV_F32 ? launch_conv_f32(P, st) : d->dtype == XCONV_BF16 ? launch_conv_bf16(P, st) : launch_conv_f16(P, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace xc
