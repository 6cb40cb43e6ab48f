// C ABI entry points of libowt: descriptor checks, launch planning, tuning, launches.
#include <algorithm>
#include <array>
#include <atomic>
#include <map>
#include <mutex>
#include <vector>

#include "owt_host.hpp"
#include "sconv.hpp"
#include "sconv_bf16.hpp"
#include "sfilter.hpp"
#include "sfilter_bf16.hpp"

namespace owt {

static thread_local char g_err[512] = "";

owt_status fail(owt_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return st;
}
void clear_error() { g_err[0] = 0; }

const TileInfo kTiles[NUM_TILES + 5] = {
    {TILE_128x128, 2, 2, 32, 1.00f, 128},
    {TILE_128x64, 2, 1, 16, 0.90f, 128},
    {TILE_64x128, 1, 2, 16, 0.90f, 64},
    {TILE_64x64, 1, 1, 16, 0.75f, 64},
    {TILE_256x64, 4, 1, 32, 1.00f, 256},
    {TILE_128x64H, 4, 1, 32, 1.00f, 128},
    {TILE_128x128H, 4, 2, 32, 1.00f, 128},
    {TILE_512x64, 4, 1, 32, 1.00f, 512},
    {TILE_256x64P, 4, 1, 32, 1.00f, 256},
};

static inline long cdiv(long a, long b) { return (a + b - 1) / b; }
static inline size_t pad256(size_t n) { return (n + 255) & ~(size_t)255; }

bool fill_geom(Geom &g, int N, int C, int H, int W, int K, int R, int S, int sh, int sw, int ph, int pw)
{
    g.N = N; g.C = C; g.H = H; g.W = W; g.K = K; g.R = R; g.S = S;
    g.sh = sh; g.sw = sw; g.ph = ph; g.pw = pw; g.bf16 = 0; g.masked = 0;
    g.P = (H + 2 * ph - R) / sh + 1;
    g.Q = (W + 2 * pw - S) / sw + 1;
    if (H + 2 * ph - R < 0 || W + 2 * pw - S < 0) return false;
    g.dC.set(C); g.dS.set(S); g.dK.set(K); g.dQ.set(g.Q); g.dPQ.set(g.P * g.Q);
    g.dW.set(W); g.dHW.set(H * W); g.dsh.set(sh); g.dsw.set(sw);
    return true;
}

// ------------------------------------------------------------ launch planning
// A pass can run as the gather kernel (igemm.hpp; any shape) or, for stride-1
// forward / backward-data, as the panel-resident kernel (dconv.hpp).  Every
// (kernel, tile, split) that fits is a candidate; a cost model picks one unless
// owt_conv_autotune has timed them for this descriptor.
enum { KIND_GATHER = 0, KIND_DIRECT = 1, KIND_DFILTER = 2, KIND_SFILTER = 3, KIND_SCONV = 4, KIND_DIRECT16 = 5, KIND_DFILTER16 = 6, KIND_SCONV16 = 7, KIND_SFILTER16 = 8, KIND_FCGEMM = 9, KIND_DFILTER2 = 10, KIND_SCONV2 = 11, KIND_SFILTER2 = 12, KIND_DFILTER16B = 13, KIND_SFILTER16B = 14, KIND_XCONV = 15, KIND_XFILTER = 16, KIND_XGATHER = 17, KIND_XFC = 18, KIND_IFILTER16 = 19, KIND_DIRECT16X = 20, KIND_IGATHER16 = 21, KIND_XCONVS = 22, KIND_DIRECT16S = 23, KIND_IFILTER16B = 24, KIND_XFCS = 25 };

// Kernels that multiply fp32 operands on the bf16 matrix unit (split3.hpp), the shard's for either storage type, and those for
// bf16 storage of any channel count: a call whose scratch is too small for one of them is served by the kernels before them.
static inline bool is_split_kind(int kind)
{
    return kind == KIND_XCONV || kind == KIND_XFILTER || kind == KIND_XGATHER || kind == KIND_XFC || kind == KIND_IFILTER16 || kind == KIND_DIRECT16X ||
           kind == KIND_IGATHER16 || kind == KIND_XCONVS || kind == KIND_DIRECT16S || kind == KIND_IFILTER16B || kind == KIND_XFCS;
}

struct PassDims { long M, Ncols, Kd; bool va, vb; };

static PassDims conv_dims(const Geom &g, int pass)
{
    PassDims r;
    const bool c4 = g.C % 4 == 0, k4 = g.K % 4 == 0;
    if (pass == OWT_PASS_FWD) {
        r.M = (long)g.N * g.P * g.Q; r.Ncols = g.K; r.Kd = (long)g.R * g.S * g.C; r.va = r.vb = c4;
    } else if (pass == OWT_PASS_BWD_DATA) {
        r.M = (long)g.N * g.H * g.W; r.Ncols = g.C; r.Kd = (long)g.R * g.S * g.K; r.va = k4; r.vb = c4;
    } else {
        r.M = g.K; r.Ncols = (long)g.R * g.S * g.C; r.Kd = (long)g.N * g.P * g.Q; r.va = k4; r.vb = c4;
    }
    return r;
}

static void dconv_frame(const Geom &g, int pass, GemmParams &p)
{
    if (pass == OWT_PASS_FWD) {
        p.Hi = g.H; p.Wi = g.W; p.Ho = g.P; p.Wo = g.Q; p.pah = g.ph; p.paw = g.pw; p.Cred = g.C;
    } else {
        p.Hi = g.P; p.Wi = g.Q; p.Ho = g.H; p.Wo = g.W; p.pah = g.R - 1 - g.ph; p.paw = g.S - 1 - g.pw; p.Cred = g.K;
    }
    p.dWo.set(p.Wo); p.dHoWo.set(p.Ho * p.Wo);
}

// A strided forward pass seen as a stride-1 one over blocks of sh x sw input pixels: RB x SB taps of sh*sw*C channels.
static int blocks_r(const Geom &g) { return (g.R + g.sh - 1) / g.sh; }
static int blocks_s(const Geom &g) { return (g.S + g.sw - 1) / g.sw; }
static void blocks_frame(const Geom &g, GemmParams &p)
{
    p.Hi = g.P + blocks_r(g) - 1; p.Wi = g.Q + blocks_s(g) - 1; p.Ho = g.P; p.Wo = g.Q; p.pah = p.paw = 0; p.Cred = g.sh * g.sw * g.C;
    p.dWo.set(p.Wo); p.dHoWo.set(p.Ho * p.Wo);
}

// LDS panel rows a tile of BM consecutive output pixels of a stride-1 pass (or of a strided forward pass over blocks)
// needs, or -1 when its input pixels are not one contiguous run.
// per_image: tiles start anew with every image.
static long panel_rows(const Geom &g, int pass, const PassDims &dm, long BM, bool blocks = false, bool per_image = false)
{
    if (pass == OWT_PASS_BWD_FILTER || (!blocks && (g.sh != 1 || g.sw != 1))) return -1;
    GemmParams f; memset(&f, 0, sizeof(f));
    if (blocks) blocks_frame(g, f); else dconv_frame(g, pass, f);
    const long taps_h = blocks ? blocks_r(g) : g.R, taps_w = blocks ? blocks_s(g) : g.S;
    if (f.Ho > f.Hi || f.Wo > f.Wi) return -1;
    const long image = (long)f.Ho * f.Wo;
    auto pin = [&](long m) {
        const long n = m / image, rem = m - n * image, ho = rem / f.Wo;
        return n * f.Hi * f.Wi + (ho - f.pah) * f.Wi + (rem - ho * f.Wo - f.paw);
    };
    long need = 0;
    // (tile starts repeat modulo the image after `image` tiles)
    const long end = per_image ? image : dm.M;
    for (long m0 = 0, i = 0; m0 < end && i <= image; m0 += BM, i++) {
        const long last = (m0 + BM < end ? m0 + BM : end) - 1;
        const long rows = pin(last) - pin(m0) + (taps_h - 1) * f.Wi + taps_w;
        if (rows > need) need = rows;
    }
    return need;
}

// The same for the direct kernel, or -1 when the pass does not qualify.
static long direct_panel_rows(const Geom &g, int pass, const PassDims &dm, long BM = 128)
{
    if (pass == OWT_PASS_BWD_FILTER || g.R * g.S == 1) return -1;
    if ((pass == OWT_PASS_FWD ? g.C : g.K) % 4 || (pass == OWT_PASS_BWD_DATA && dm.Ncols % 4)) return -1;
    return panel_rows(g, pass, dm, BM);
}

// Geometry of the bf16-MFMA small-channel strided forward kernel; false when it does not apply (bf16
// storage, window starts and image rows that are multiples of 4 values, K a multiple of 4, the filter
// bank of 64 filters plus one band of rows within 150 KB of LDS).
static bool sconv16_geom(const Geom &g, SConv16Geom &sg)
{
    if (!g.bf16 || (g.sw * g.C) % 4 || (g.W * g.C) % 4 || g.C > 16 || g.K % 4 || (g.sh == 1 && g.sw == 1)) return false;
    sg.SEG = g.S * g.C;
    sg.LPAD = (4 - (g.pw * g.C) % 4) % 4;
    sg.SLOTS = (sg.SEG + sg.LPAD + 7) & ~7;
    sg.OCT = sg.SLOTS / 8;
    sg.NG = ((g.R * sg.OCT + 3) / 4) * 2;          // groups of 16 slots, an even number of them
    sg.KSLOTS = sg.NG * 16;
    sg.WP = sg.KSLOTS + 8;
    const int a = g.pw * g.C + sg.LPAD + g.W * g.C, b = (g.Q - 1) * g.sw * g.C + sg.SLOTS;
    sg.PITCH = ((a > b ? a : b) + 7) & ~7;
    sg.ROWS = (kSConv16TP - 1) * g.sh + g.R;
    // the padded tail of the reduction (up to 3 octets) reads past filter row R-1: those panel rows exist and stay zero
    sg.ZROWS = sg.ROWS + 1 + (3 + sg.OCT - 1) / sg.OCT;
    sg.MPIX = kSConv16TP * g.Q;
    sg.units_per_image = (g.P + kSConv16TP - 1) / kSConv16TP;
    sg.units = g.N * sg.units_per_image;
    sg.BIAS = 64 * sg.WP + 2 * sg.ZROWS * sg.PITCH;
    const size_t lds = ((size_t)sg.BIAS + 128) * 2;                  // filter bank + two bands + 64 fp32 biases
    // the output staging blocks follow when the 160 KB of a CU still hold them
    sg.STAGE = lds + (size_t)kSConv16StageValues * 2 <= 160 * 1024 ? (int)(lds / 2) : 0;
    return sg.OCT >= 2 && sg.MPIX <= 256 && lds <= 150 * 1024 && sg.ROWS < 256 &&
           (long)sg.ROWS * (g.W * g.C / 4) <= (long)(kSConv16NT / 2) * kSConv16PNP;
}

// Tap grouping and panel size of the direct filter-gradient kernel for one variant; false when it
// does not apply (needs stride 1, P == H, Q == W, C and K multiples of 4, R*S or S equal to the variant's tap count, and a
// 32-pixel chunk whose padded-coordinate span fits the variant's LDS panel).
static bool dfilter_fits(const Geom &g, int variant, int &taps, int &groups)
{
    const DFilterVariant &v = kDFilterVariants[variant];
    if (g.sh != 1 || g.sw != 1 || g.P != g.H || g.Q != g.W || g.C % 4 || g.K % 4) return false;
    if (g.R * g.S == v.tmax) { taps = g.R * g.S; groups = 1; }
    else if (g.S == v.tmax) { taps = g.S; groups = g.R; }
    else return false;
    const long Wp = g.W + 2 * g.pw, Hp = g.H + 2 * g.ph, PQ = (long)g.P * g.Q;
    long span = 31 + (31 / g.Q + 1) * (Wp - g.Q);
    if (v.aligned) {        // chunks cut per image: worth it only when the short last chunk wastes little
        if (((PQ + 31) / 32) * 32 * 100 > PQ * 104) return false;
    } else {
        span += (31 / PQ + 1) * (Hp - g.P) * Wp;
    }
    const long rows = span + (groups > 1 ? 0 : g.R - 1) * Wp + g.S;
    return rows <= v.prf && (long)g.N * Hp * Wp < 0x7fffffffL;
}

// The same for the kernel with the in-work-group pixel split (fp32 storage; chunks of 32*WP pixels).
static bool dfilter2_fits(const Geom &g, int variant, int &taps, int &groups)
{
    const DFilter2Variant &v = kDFilter2Variants[variant];
    if (g.bf16 || g.masked || g.sh != 1 || g.sw != 1 || g.P != g.H || g.Q != g.W || g.C % 4 || g.K % 4) return false;
    const long Wp = g.W + 2 * g.pw, Hp = g.H + 2 * g.ph, PQ = (long)g.P * g.Q, last = 32 * v.WP - 1;
    if (v.SW > 0) {
        if (g.S != v.SW || g.R * g.S != v.tmax || Wp != v.WPC) return false;
        taps = v.tmax; groups = 1;
    } else {
        if (g.S != v.tmax) return false;
        taps = g.S; groups = g.R;
    }
    // buffer descriptors hold byte counts in 32 bits, and bit 31 of an offset marks "reads as zero"
    if ((long)g.N * g.H * g.W * g.C * 4 >= 0x7fffffffL || (long)g.N * PQ * g.K * 4 >= 0x7fffffffL) return false;
    // the loaders' two LDS tables have 1024 entries, and a chunk may touch two images at most
    if (Hp * Wp > 1024 || PQ > 1024 || 32 * v.WP > PQ) return false;
    const long span = last + (last / g.Q + 1) * (Wp - g.Q) + (last / PQ + 1) * (Hp - g.P) * Wp;
    const long rows = span + (groups > 1 ? 0 : g.R - 1) * Wp + g.S;
    return rows <= v.prows && (long)g.N * Hp * Wp < 0x7fffffffL;
}

// The same for the bf16-MFMA variant (64-pixel chunks, 16-byte pieces: C and K multiples of 8).
static bool dfilter16_fits(const Geom &g, int variant, int &taps, int &groups)
{
    const DFilter16Variant &v = kDFilter16Variants[variant];
    if (!g.bf16 || g.sh != 1 || g.sw != 1 || g.P != g.H || g.Q != g.W || g.C % 8 || g.K % 8) return false;
    if (g.R * g.S == v.tmax) { taps = g.R * g.S; groups = 1; }
    else if (g.S == v.tmax) { taps = g.S; groups = g.R; }
    else return false;
    const long Wp = g.W + 2 * g.pw, Hp = g.H + 2 * g.ph, PQ = (long)g.P * g.Q, last = kDFilter16BP - 1;
    const long span = last + (last / g.Q + 1) * (Wp - g.Q) + (last / PQ + 1) * (Hp - g.P) * Wp;
    const long rows = span + (groups > 1 ? 0 : g.R - 1) * Wp + g.S;
    return rows <= v.prf && (long)g.N * Hp * Wp < 0x7fffffffL;
}

// The bf16 filter-gradient kernel whose operands stream straight into LDS: as above, plus dz taken as it is, loader
// tables of 1024 entries, chunks that touch at most two images, and 32-bit byte offsets into x.
static bool dfilter16b_fits(const Geom &g, int variant, int &taps, int &groups)
{
    const DFilter16bVariant &v = kDFilter16bVariants[variant];
    if (!g.bf16 || g.masked || g.sh != 1 || g.sw != 1 || g.P != g.H || g.Q != g.W || g.C % 8 || g.K % 8) return false;
    const long Wp = g.W + 2 * g.pw, Hp = g.H + 2 * g.ph, PQ = (long)g.P * g.Q, last = kDFilter16BP - 1;
    if (v.SW > 0) {
        if (g.S != v.SW || g.R * g.S != v.tmax || Wp != v.WPC) return false;
        taps = v.tmax; groups = 1;
    } else {
        if (g.S != v.tmax) return false;
        taps = g.S; groups = g.R;
    }
    if (Hp * Wp > 1024 || PQ > 1024 || kDFilter16BP > PQ) return false;
    if ((size_t)g.N * g.H * g.W * g.C * 2 >= 0x7fffffffull || (size_t)g.N * PQ * g.K * 2 >= 0x7fffffffull) return false;
    const long span = last + (last / g.Q + 1) * (Wp - g.Q) + (Hp - g.P) * Wp;      // 64 pixels, their row ends, one image end
    const long rows = span + (groups > 1 ? 0 : g.R - 1) * Wp + g.S;
    return rows <= v.prf;
}

// Geometry of the small-channel strided filter-gradient kernel; false when it does not apply
// (needs window starts and image rows that are multiples of 4 floats, at most 16 blocks of 32
// slots (four accumulators per wavefront in each of four column groups), at most 150 KB of LDS).
static bool sfilter_geom(const Geom &g, SFilterGeom &sg)
{
    if ((g.sw * g.C) % 4 || (g.W * g.C) % 4 || g.K % 4) return false;
    sg.SEG = g.S * g.C;
    sg.LPAD = (4 - (g.pw * g.C) % 4) % 4;
    sg.SLOTS = (sg.SEG + sg.LPAD + 3) & ~3;
    const int a = g.pw * g.C + sg.LPAD + g.W * g.C, b = (g.Q - 1) * g.sw * g.C + sg.SLOTS;
    sg.PITCH = ((a > b ? a : b) + 3) & ~3;
    sg.ROWS = g.sh + g.R;                         // two output rows
    sg.NB = (g.R * sg.SEG + 31) / 32;             // blocks of 32 densely packed (r, s, c) slots
    sg.DZP = (2 * g.Q + 1) & ~1;
    sg.units_per_image = (g.P + 1) / 2;
    sg.units = g.N * sg.units_per_image;
    const size_t lds = ((size_t)sg.ROWS * sg.PITCH + (size_t)sg.DZP * 68) * 4 + (size_t)sg.DZP * 4;
    return sg.NB <= 4 * kSFilterACCS && lds <= 150 * 1024 && g.C <= 16 &&
           sg.ROWS < 256 && g.Q < 65536 &&
           (long)sg.ROWS * (g.W * g.C / 4) <= (long)kSFilterNT * kSFilterPNP && (long)sg.DZP * 16 <= (long)kSFilterNT * kSFilterDNP;
}

// Geometry of the bf16-MFMA small-channel strided filter-gradient kernel; false when it does not apply
// (bf16 storage, K a multiple of 8, window starts and image rows that are multiples of 4 values, at
// most 16 blocks of 32 columns, one band of rows + its dz values within 150 KB of LDS).
static bool sfilter16_geom(const Geom &g, SFilter16Geom &sg)
{
    if (!g.bf16 || (g.sw * g.C) % 4 || (g.W * g.C) % 4 || g.K % 8 || g.C > 16) return false;
    sg.SEG = g.S * g.C;
    sg.LPAD = (4 - (g.pw * g.C) % 4) % 4;
    sg.SLOTS = (sg.SEG + sg.LPAD + 3) & ~3;
    const int a = g.pw * g.C + sg.LPAD + g.W * g.C, b = (g.Q - 1) * g.sw * g.C + sg.SLOTS;
    sg.PITCH = ((a > b ? a : b) + 3) & ~3;
    sg.ROWS = (kSFilter16TP - 1) * g.sh + g.R;
    sg.NB = (g.R * sg.SLOTS + 31) / 32;
    sg.MPIX = kSFilter16TP * g.Q;
    sg.NGP = ((sg.MPIX + 31) / 32) * 2;            // groups of 16 pixels, an even number of them
    sg.DZP = sg.NGP * 16;
    sg.units_per_image = (g.P + kSFilter16TP - 1) / kSFilter16TP;
    sg.units = g.N * sg.units_per_image;
    const size_t lds = ((size_t)sg.ROWS * sg.PITCH + (size_t)sg.DZP * 80) * 2 + (size_t)sg.DZP * 4;
    return sg.NB <= (kSFilter16NT / 64) * kSFilter16CB && lds <= 150 * 1024 && sg.ROWS < 256 &&
           (long)sg.ROWS * (g.W * g.C / 4) <= (long)kSFilter16NT * kSFilter16PNP &&
           sg.DZP <= (kSFilter16NT / 8) * kSFilter16DNP;
}

// The bf16 first-layer filter-gradient kernel whose units stream straight into two LDS stages: dz taken as it is,
// 16-byte aligned row data in the panel, both stages within LDS, the loaders' instruction counts, 32-bit byte
// offsets inside one image.
static bool sfilter16b_fits(const Geom &g, const SFilter16Geom &sg)
{
    const long pp8 = ((sg.PITCH + 7) & ~7) / 8, pan_inst = ((long)sg.ROWS * pp8 + 63) / 64, dz_inst = sg.DZP / 8;
    const size_t lds = (size_t)2 * (pan_inst + dz_inst) * 1024 + (size_t)sg.DZP * 4;
    return !g.masked && (g.pw * g.C + sg.LPAD) % 8 == 0 && (g.W * g.C) % 8 == 0 && pan_inst <= 8 * kSFilter16bPNI &&
           dz_inst <= 8 * kSFilter16bDNI && lds <= 158 * 1024 && (size_t)g.H * g.W * g.C * 2 < 0x40000000ull &&
           (size_t)g.P * g.Q * g.K * 2 < 0x40000000ull;
}

// Geometry of the small-channel strided forward kernel; false when it does not apply.
static bool sconv_geom(const Geom &g, SConvGeom &sg)
{
    if ((g.sw * g.C) % 4 || (g.W * g.C) % 4 || g.C > 16 || (g.sh == 1 && g.sw == 1)) return false;
    sg.SEG = g.S * g.C;
    sg.LPAD = (4 - (g.pw * g.C) % 4) % 4;
    sg.SLOTS = (sg.SEG + sg.LPAD + 3) & ~3;
    const int a = g.pw * g.C + sg.LPAD + g.W * g.C, b = (g.Q - 1) * g.sw * g.C + sg.SLOTS;
    sg.PITCH = ((a > b ? a : b) + 3) & ~3;
    // output rows that kSConvBand consecutive pixels can touch, and the input rows under them
    int orows = (g.Q + kSConvBand - 2) / g.Q + 1;
    if (orows > g.P) orows = g.P;
    sg.ROWS = (orows - 1) * g.sh + g.R;
    sg.KSTEPS = (g.R * sg.SLOTS + kSConvBK - 1) / kSConvBK;
    sg.KSLOTS = sg.KSTEPS * kSConvBK;
    sg.MPIX = kSConvBand;
    sg.units_per_image = (g.P * g.Q + kSConvBand - 1) / kSConvBand;
    sg.units = g.N * sg.units_per_image;
    // the padded tail of the reduction runs past filter row R-1: those panel rows exist and stay zero
    const int zr = (orows - 1) * g.sh + (sg.KSLOTS - 1) / sg.SLOTS + 1;
    sg.ZROWS = zr > sg.ROWS + 1 ? zr : sg.ROWS + 1;
    const size_t lds = ((size_t)2 * 64 * (kSConvBK + 4) + (size_t)sg.ZROWS * sg.PITCH) * 4;
    return sg.MPIX <= 256 && lds <= 150 * 1024 && sg.ROWS < 256 && sg.SLOTS >= 8 && sg.KSLOTS <= 2048 &&
           (long)sg.ROWS * (g.W * g.C / 4) <= (long)kSConvNT * kSConvPNP;
}

// The first-layer forward kernel that keeps 32 filters' whole bank in LDS beside the band: fp32 storage, LDS
// capacity, and 32-bit byte offsets into x and y for its buffer descriptors.
static bool sconv2_fits(const Geom &g, const SConvGeom &sg)
{
    const size_t lds = ((size_t)kSConv2KB * (sg.KSLOTS + 4) + (size_t)sg.ZROWS * sg.PITCH) * 4;
    const size_t xb = (size_t)g.N * g.H * g.W * g.C * 4, yb = (size_t)g.N * g.P * g.Q * g.K * 4;
    return lds <= 157 * 1024 && xb < 0x7fffffffull && yb < 0x7fffffffull && sg.KSTEPS * (kSConvBK / 4) <= 512;
}

// The first-layer filter-gradient kernel whose units stream straight into two LDS stages: fp32 storage, dz taken
// as it is, both stages within LDS, the loaders' instruction counts, 32-bit byte offsets inside one image.
static bool sfilter2_fits(const Geom &g, const SFilterGeom &sg)
{
    const long pan_inst = ((long)sg.ROWS * (sg.PITCH / 4) + 63) / 64, dz_inst = ((long)sg.DZP * 17 + 63) / 64;
    const size_t lds = (size_t)2 * (pan_inst + dz_inst) * 1024 + (size_t)sg.DZP * 4;
    return !g.bf16 && !g.masked && pan_inst <= 8 * kSFilter2PNI && dz_inst <= 8 * kSFilter2DNI && lds <= 158 * 1024 &&
           (size_t)g.H * g.W * g.C * 4 < 0x40000000ull && (size_t)g.P * g.Q * g.K * 4 < 0x40000000ull;
}

struct Launch {
    int kind, tile, splits, steps, steps_per_split, tiles_m, tiles_n, pr, taps, groups, ctiles, blocks, tpi;
    size_t partial_bytes, dbias_bytes;
    size_t pre_bytes;   // workspace in front of the partials (re-laid-out filters of the bf16 backward-data kernel)
    double cost;   // model estimate, ~clocks
    bool fitted;   // ... 1260 times the microseconds that timed launches of the kind take, launch and latency included
    double asked;  // what the cost was raised by for other reasons than time, which tuning leaves out
    size_t ws_bytes() const { return pre_bytes + partial_bytes + dbias_bytes; }
};

// Model: the launch's MACs spread over 256 CUs at the tile's relative efficiency, derated when fewer
// than two wavefronts per SIMD are resident (nothing hides load latency then) and by the unevenness
// of the last round of work-groups; a split adds a write+read of the partials and a launch.
static double model_cost(long wgs, int waves_per_wg, int occ, double macs_per_wg, double eff, long splits,
                         long M, long Ncols)
{
    const double per_cu = (double)wgs / 256.0;
    const double resident = (per_cu < occ ? per_cu : occ) * waves_per_wg / 4.0;
    const double lat = resident >= 2.0 ? 1.0 : (resident >= 1.0 ? 0.62 + 0.38 * (resident - 1.0) : 0.62 * resident);
    const double rounds = (double)wgs / (256.0 * occ);
    const double tail = rounds > 1.0 ? 0.5 + 0.5 * rounds / (double)cdiv(wgs, 256L * occ) : 1.0;
    double cost = (double)wgs * macs_per_wg / 256.0 / (128.0 * eff * lat * tail);
    if (splits > 1) cost += 14000.0 + (double)(splits + 1) * M * Ncols * 4.0 / 1300.0;
    return cost;
}

// Work-groups one after the other: the rounds they take at `occ` to a CU, and the work-groups of a CU added up over the rounds.
static void wg_rounds(long wgs, int occ, double &rounds, double &resident)
{
    const long full = wgs / (256L * occ), rest = wgs % (256L * occ);
    rounds = full + (rest > 0);
    resident = full * occ + cdiv(rest, 256);
}

// Microseconds of a bf16 forward or backward-data launch of stride 1 where the kernels that take it differ in kind: what a tap of a
// chunk takes per round and per resident work-group, what the panel takes, the results' stores (twice as long where their number
// per pixel is odd), the reduce pass.  Fitted to 734 timed launches of 70 layers and of draws of other geometries, 0.08 to 0.15 in the
// logarithm.  Held to the clocks of model_cost, which know no latencies, 31 of 103 passes took more than 5 % longer than the
// fastest kernel, up to 1.36 times (49 images 13x9, 200 -> 72 of 5x5: 38 us where dconv16 takes 28); with this 6, up to 1.10 times.
static double conv16_us(const Launch &l, int pass, const Geom &g, const PassDims &dm)
{
    const double mb = l.splits > 1 ? l.splits * dm.M * dm.Ncols * 4e-6 : 0.0;
    const double outs = l.splits > 1 ? 0.0 : dm.M * dm.Ncols * (dm.Ncols % 2 ? 4e-6 : 2e-6);
    const double steps = (double)g.R * g.S * l.steps_per_split, panel = l.steps_per_split * l.pr / 64.0;
    const long wgs = (long)l.tiles_m * l.tiles_n * l.splits;
    double rounds, resident;
    if (l.kind == KIND_DIRECT16X) {
        const bool odd = (pass == OWT_PASS_FWD ? g.C : g.K) % 2 != 0, masked = pass == OWT_PASS_BWD_DATA && g.masked;
        wg_rounds(wgs, odd || masked ? 2 : 3, rounds, resident);
        const double t = odd ? (masked ? 0.328 : 0.340) : (masked ? 0.363 : 0.318), r = odd == masked ? 0.055 : 0.002;
        return 13.0 + steps * (t * rounds + r * resident) + (masked ? 0.0 : odd ? 0.097 : 0.05) * panel * resident + (l.splits > 1 ? 0.6 : 0.0) + 0.85 * mb + 0.35 * outs;
    }
    if (l.kind == KIND_DIRECT16) {
        wg_rounds(wgs, 2, rounds, resident);
        const double t = l.tile == TILE_128x128 ? 0.60 : l.tile == TILE_128x64 ? 0.62 : 0.46, r = l.tile == TILE_128x128 ? 0.073 : l.tile == TILE_128x64 ? 0.0 : 0.10;
        const double q = l.tile == TILE_128x128 ? 0.18 : l.tile == TILE_128x64 ? 0.31 : 0.14;
        return 8.7 + (pass == OWT_PASS_BWD_DATA ? 3.9 : 0.0) + steps * (t * rounds + r * resident) + q * panel * resident + (l.splits > 1 ? 0.6 : 0.0) + 0.56 * mb + 0.82 * outs;
    }
    return l.cost / 1260.0 + 10.0;                       // the kernels on the fp32 instruction
}

// Microseconds of the bf16 filter gradient over images with streamed operands: matrix instructions at 32 clocks, a step's latency per
// round (a row has the columns left of its first product and the rounding to whole stages for steps without any), storing the tile,
// the reduce pass.  Fitted to 3825 timed launches of 210 layers, 0.10 in the logarithm; its choice takes 3 % longer than the fastest.
static double ifilter16b_us(const Launch &l, const Geom &g, const PassDims &dm)
{
    const IFilter16bVariant &v = kIFilter16bVariants[l.tile];
    double rounds, resident;
    wg_rounds((long)l.tiles_m * l.tiles_n * l.splits, v.occ, rounds, resident);
    const double per = l.steps_per_split, idle = (per / g.Q + 1.0) * (v.S - 1 + 0.5 * (v.L - 1)), blocks = v.KB * v.CB * v.S;
    const double us = (l.splits > 1 ? 8.1 + 0.228e-6 * 4.0 * l.splits * dm.M * dm.Ncols : 5.0) + 0.97 * resident * per * blocks * v.WK * v.WC / 4.0 * 32.0 / 2100.0 +
                      rounds * (0.129 * (per + idle) + 0.59 * blocks);
    const double few = (g.K <= 48 ? 1.1 : 1.0) * us;    // (tiles mostly empty: the other kinds' prices come out high there, seven of 210 layers were up to 16 % slower)
    return 1.03 * (few - 3.0 * std::max(0.0, 1.0 - few / 25.0));      // (short ones came out a quarter high)
}

// Microseconds of the fp32 forward and backward-data kernel of few tiles: a step (a tap of a chunk) of each wavefront of a SIMD, with the
// rows of its panels where their values are loaded one by one, and its latency once a round; a panel's pieces of loads; what a work-group
// begins and ends with, the groups' sums and the stores, for each of a CU's; the reduce pass.  Coefficients per pass and tile, fitted to
// 14505 launches of 3000 drawn passes, 0.05 to 0.07 in the logarithm (the tile of 128 pixels, and backward-data's of 32, weighed 3 and 1 %
// more, which is the better choice over these passes).
struct XConvSUs { double at, work, rows, lat, load, wg, round, split, mb; };
static const XConvSUs kXConvSUs[2][kNumXConvSVariants] = {
    {{1.42, 0.22, 4.9e-4, 0.0, 0.0, 0.0, 3.7, 2.84, 0.614}, {2.6, 0.161, 8.5e-4, 0.181, 0.067, 0.785, 0.605, 2.92, 0.474}, {2.58, 0.157, 9.9e-4, 0.225, 0.037, 0.704, 0.632, 2.99, 0.428}},
    {{1.12, 0.275, 7.4e-4, 0.0, 0.068, 3.79, 0.0, 2.9, 0.482}, {2.6, 0.164, 1.28e-3, 0.334, 0.182, 1.18, 0.0, 2.89, 0.365}, {2.66, 0.172, 1.55e-3, 0.333, 0.187, 0.897, 0.262, 2.86, 0.26}}};

// Microseconds of the fp32 filter gradients over images: a position takes a wavefront its fragments' loads and splits (a fragment of
// masked dz half as long again), one after the other for the wavefronts of a SIMD, and a latency; rows of the walk have their first
// columns, a launch its rounds and the tiles' stores.  Coefficients per variant, fitted to 6695 timed launches of 261 layers, 0.05 to
// 0.08 in the logarithm; the choice by them takes 1 % longer than the fastest launches.  Long walks of xgather's two wavefronts a SIMD come
// out low (the first layer at 128 images: 141 us, 169 to 180 measured, where 2 x 3 blocks take 154).
struct Images32Us { double at, frag, lat, row, round, store, mb, split; };
static const Images32Us kXFilterUs[kNumXFilterVariants] = {
    {0.0, 0.238, 0.0, 0.149, 0.0, 1.18, 0.338, 8.94}, {0.0, 0.191, 0.231, 0.101, 0.0, 1.25, 0.325, 8.15},
    {3.95, 0.178, 0.121, 0.153, 1.93, 0.423, 0.291, 3.44}, {0.0, 0.222, 0.147, 0.170, 0.0, 1.38, 0.385, 5.69}};
static const Images32Us kXGatherUs[kNumXGatherVariants] = {
    {4.92, 0.203, 0.215, 0.0, 0.0, 1.20, 0.379, 3.09}, {3.39, 0.0935, 0.543, 0.0, 0.0, 1.86, 0.433, 2.91},
    {4.08, 0.0647, 0.799, 0.0, 0.695, 0.825, 0.428, 3.25}, {3.54, 0.0673, 0.616, 0.0, 0.729, 0.895, 0.356, 3.41}};
static double images32_us(const Launch &l, const Images32Us &u, int TG, int occ, double frags, int cols, int blocks, const Geom &g, const PassDims &dm)
{
    double rounds, resident;
    if (TG > 1) wg_rounds((long)l.tiles_m * l.tiles_n * l.splits, occ, rounds, resident);
    else rounds = resident = (double)cdiv((long)l.tiles_m * l.tiles_n * l.splits, 1024);
    const double pos = (double)cdiv(l.steps_per_split, TG), rows = cols * (pos / g.Q + 1.0);
    const double walk = TG > 1 && cols == 0 && pos > 48.0 ? 1.0 + (pos - 48.0) / 400.0 : 1.0;
    // (long chains of positions round off more: weighed a little)
    const double chain = 1.0 + std::min(48.0, std::max(0.0, pos - 16.0)) / 400.0;
    return chain * (u.at + walk * u.frag * resident * pos * frags + walk * u.lat * rounds * pos + u.row * resident * rows + u.round * rounds + u.store * resident * blocks +
           (l.splits > 1 ? u.split + u.mb * 4e-6 * l.splits * dm.M * dm.Ncols : 0.0));
}

// The same for bf16 storage: a column of the walk takes a wavefront 31 clocks a matrix instruction and 29 a load (`clocks`), one after the
// other for the wavefronts of a SIMD, and a latency.  Fitted to 3029 timed launches of 130 layers, 0.06 to 0.11 in the logarithm; the choice
// by them takes 1.5 % longer than the fastest launches.
struct Images16Us { double at, work, lat, round, store, mb, split; };
static const Images16Us kIFilter16Us[kNumIFilter16Variants] = {
    {4.20, 0.400, 0.107, 0.0, 0.666, 0.292, 4.13}, {3.36, 0.404, 0.127, 2.17, 0.268, 0.402, 4.58}, {3.60, 0.369, 0.125, 2.38, 0.279, 0.437, 4.09},
    {3.04, 0.396, 0.128, 0.0, 0.719, 0.552, 3.81}, {3.95, 0.316, 0.158, 1.62, 0.320, 0.586, 3.93}, {2.33, 0.517, 0.017, 0.0, 0.806, 0.461, 4.06},
    {3.88, 0.448, 0.055, 0.0, 0.744, 0.625, 2.91}};
static const Images16Us kIGather16Us[kNumIGather16Variants] = {
    {3.25, 0.343, 0.177, 0.433, 0.919, 0.261, 3.64}, {2.24, 0.338, 0.242, 4.54, 0.130, 0.541, 3.34}, {2.72, 0.343, 0.210, 1.16, 0.787, 0.341, 3.69}};
// Long chains of positions round off more; the weight is for the choice of splits alone.
static double images16_chain(const Launch &l) { return 1.0 + std::min(400.0, std::max(0.0, (double)cdiv(l.steps_per_split, 4) - 40.0)) / 500.0; }
static double images16_us(const Launch &l, const Images16Us &u, int occ, double clocks, int cols, int blocks, const Geom &g, const PassDims &dm)
{
    double rounds, resident;
    wg_rounds((long)l.tiles_m * l.tiles_n * l.splits, occ, rounds, resident);
    const double pos = (double)cdiv(l.steps_per_split, 4), columns = pos + (pos / g.Q + 1.0) * (cols - 1);
    return images16_chain(l) * (u.at + u.work * 1e-3 * resident * columns * clocks + u.lat * rounds * columns + u.round * rounds + u.store * resident * blocks +
           (l.splits > 1 ? u.split + u.mb * 4e-6 * l.splits * dm.M * dm.Ncols : 0.0));
}

// What decides whether a call's scratch is refused: the plans and their costs by the models that sizes have been handed out by.  Prices
// and kernels that came later choose among the plans that fit and neither refuse a call nor take one that was refused.
struct Demand { double cost; size_t need; bool passed_over; };      // (passed over where it does not fit: the split-operand kinds)

static const size_t kMaxPartialBytes = (size_t)192 << 20;

// The bf16 filter gradient over images by clocks, a tile to a wavefront: a column `least` clocks at least, 1950 a block for its
// stores, 19000 for launch, first loads and last stores; the reduce pass 4 us and 0.24 us a MB.
struct ImagesDemand { double cost, plain; long per, wgs, splits; size_t need; bool rows; };
static void images16_demand(std::vector<ImagesDemand> &out, const std::vector<long> &ladder, const Geom &g, const PassDims &dm, bool want_db, long tiles, long steps, int occ,
                            double least, double clocks, int cols, int blocks, bool rows)
{
    for (long s : ladder) {
        if (s > 1 && (steps / s < 3 || tiles * s > 8192)) break;
        const long per = cdiv(steps, s), splits = cdiv(steps, per);
        const size_t partial = splits > 1 ? pad256((size_t)splits * dm.M * dm.Ncols * 4) : 0, need = partial + (splits > 1 && want_db ? pad256((size_t)splits * dm.M * 4) : 0);
        if (partial > kMaxPartialBytes) continue;
        const double resident = std::min((double)occ, std::max(1.0, tiles * splits / 1024.0)), column = std::max(least, resident * clocks);
        const double walk = (per + (rows ? (per / g.Q + 1.0) * (cols - 1) : 0.0)) * column + 1950.0 * blocks;
        const double plain = 0.6 * (walk * cdiv(tiles * splits, 1024L * occ) + 19000.0);
        const double cost = plain + (splits > 1 ? 5000.0 + (double)splits * dm.M * dm.Ncols * 4.0 / 3270.0 : 0.0);
        out.push_back({rows ? cost * (1.0 + std::min(400L, std::max(0L, per - 40)) / 500.0) : cost, plain, per, cdiv(tiles * splits, 256), splits, need, rows});
    }
}

// Adds the same to the cost of every launch of a kind, so that the cheapest of them costs `us` microseconds.
static void price_kind(std::vector<Launch> &out, int kind, double clocks_of_cheapest, double us)
{
    for (Launch &l : out)
        if (l.kind == kind) { l.cost += 1260.0 * us - clocks_of_cheapest; l.fitted = true; }
}
static const Launch *cheapest_of(const std::vector<Launch> &out, int kind)
{
    const Launch *best = nullptr;
    for (const Launch &l : out)
        if (l.kind == kind && (!best || l.cost < best->cost)) best = &l;
    return best;
}

// The filter-gradient kernels that take 16 images per matrix instruction form 32-bit byte offsets for whole groups of 16 and
// leave it to the buffer descriptor to read the images past the last as zeros, so no offset may come round past 2^32 into the
// tensor again.  xfilter: every image of the last group, and up to 1 KB past its end for a ragged tile.  xgather: also a place
// outside the image, which gets the offset N * image, at the first seven images of the last group's second half.
static bool image_groups_fit(const Geom &g, bool xgather)
{
    const double groups = 16.0 * (double)cdiv(g.N, 16), images = xgather && g.N + groups - 9.0 > groups ? g.N + groups - 9.0 : groups;
    const double es = g.bf16 ? 2.0 : 4.0, x = (double)g.H * g.W * g.C * es, z = (double)g.P * g.Q * g.K * es;
    return g.N * x < 2147483644.0 && g.N * z < 2147483644.0 && images * x + 1024.0 <= 4294967296.0 && images * z + 1024.0 <= 4294967296.0;
}

// What owt_test_force_variant asked for (tests only; -1 / 0 = the planner decides).
static std::atomic<int> g_force_tile{-1}, g_force_split{-1};
static std::atomic<unsigned> g_force_flags{0};
static inline bool forced(unsigned bit) { return (g_force_flags.load(std::memory_order_relaxed) & bit) != 0; }

static void enumerate(const Geom &g, int pass, const PassDims &dm, bool want_db, std::vector<Launch> &out, std::vector<Demand> *demand = nullptr)
{
    const int force_tile = g_force_tile.load(std::memory_order_relaxed);
    const int force_split = g_force_split.load(std::memory_order_relaxed);
    const bool no_direct = forced(OWT_FORCE_NO_DIRECT);
    const bool vec = dm.va && dm.vb;

    auto add = [&](int kind, int tile, int pr, long steps, long s, double macs_per_step_wg, int occ, double eff) {
        if (force_split > 0) s = force_split < steps ? force_split : steps;
        const long per = cdiv(steps, s), splits = cdiv(steps, per);     // drops empty trailing splits
        const TileInfo &ti = kTiles[tile];
        const long tm = cdiv(dm.M, ti.BM), tn = cdiv(dm.Ncols, 64 * ti.WN);
        Launch l; memset(&l, 0, sizeof(l));
        l.kind = kind; l.tile = tile; l.pr = pr; l.splits = (int)splits; l.steps = (int)steps;
        l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)tn;
        if (splits > 1) {
            l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
            l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
            if (l.partial_bytes > kMaxPartialBytes && force_split <= 0) return;
        }
        l.cost = model_cost(tm * tn * splits, ti.WM * ti.WN, occ, macs_per_step_wg * per, eff, splits, dm.M, dm.Ncols);
        for (const Launch &o : out)
            if (o.kind == l.kind && o.tile == l.tile && o.splits == l.splits) return;
        out.push_back(l);
    };

    static const long kSplits[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256};
    // split counts to try for `tiles` output tiles: the fixed ladder plus the counts that fill one, two
    // or three rounds of the chip's work-group slots exactly (256 CUs x 2 resident work-groups)
    auto split_ladder = [&](long tiles, long slots = 512) {
        std::vector<long> v(kSplits, kSplits + sizeof(kSplits) / sizeof(kSplits[0]));
        for (long rounds = 1; rounds <= 3; rounds++)
            if (slots * rounds / tiles >= 1) v.push_back(slots * rounds / tiles);
        std::sort(v.begin(), v.end());
        v.erase(std::unique(v.begin(), v.end()), v.end());
        return v;
    };
    const long cred = pass == OWT_PASS_FWD ? g.C : g.K;
    for (int t : {TILE_128x128, TILE_128x64, TILE_256x64, TILE_128x64H, TILE_128x128H}) {
        if (no_direct || (force_tile >= 0 && force_tile != t)) continue;
        const long BM = kTiles[t].BM, rows = direct_panel_rows(g, pass, dm, BM);
        int pr;                                        // panel sizes the kernel is instantiated for
        if (t == TILE_256x64) { if (rows < 0 || rows > 384) continue; pr = rows <= 288 ? 288 : 384; }
        else { if (rows < 0 || rows > 256) continue; pr = rows <= 160 ? 160 : ((t == TILE_128x64H && rows <= 244) ? 244 : 256); }
        const long bk = t == TILE_128x64 ? 16 : 32, chunks = cdiv(cred, bk);
        const double macs = (double)BM * 64 * kTiles[t].WN * bk * g.R * g.S;
        for (long s : kSplits) {
            if (s > 1 && (chunks / s < 2 || s > 8)) break;
            add(KIND_DIRECT, t, pr, chunks, s, macs, t == TILE_128x64 ? 5 : (t == TILE_128x64H ? 3 : 2),
                t == TILE_128x64 ? 1.1 : 1.25);
            if (force_split > 0) break;
        }
    }
    // fp32 storage on the bf16 matrix unit with split operands: stride 1, or a strided forward pass over blocks of pixels;
    // at most 32 taps, 32-bit byte offsets.  (A strided pass of a few taps over many channels has mostly empty blocks: at
    // least half of a block's values must meet filter values.)
    const bool blocks = g.sh > 1 || g.sw > 1;
    const long xr = blocks ? blocks_r(g) : g.R, xs = blocks ? blocks_s(g) : g.S, xred = blocks ? (long)g.sh * g.sw * g.C : cred;
    if (!g.bf16 && pass != OWT_PASS_BWD_FILTER && (g.H > 1 || g.W > 1) && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) && xr * xs <= 32 &&
        (!blocks || (pass == OWT_PASS_FWD && 2L * g.R * g.S >= xr * xs * g.sh * g.sw && g.sh * g.sw <= 32 && xred <= 256)) &&
        (size_t)g.N * g.H * g.W * g.C < 0x1fffffffull && (size_t)g.N * g.P * g.Q * g.K < 0x1fffffffull) {
        for (int v = 0; v < kNumXConvVariants; v++) {
            if (force_tile >= 0 && force_tile != kXConvFirstTile + v) continue;
            const XConvVariant &xv = kXConvVariants[v];
            const long BM = 32 * xv.MB * xv.WM, BN = 64 * xv.WN, image = pass == OWT_PASS_FWD ? (long)g.P * g.Q : (long)g.H * g.W;
            // a strided pass has no padding between its blocks: tiles per image when the last, short ones waste under 5 %
            const long tpi = blocks && cdiv(image, BM) * BM * 20 <= image * 21 ? cdiv(image, BM) : 0;
            const long rows = panel_rows(g, pass, dm, BM, blocks, tpi > 0);
            if (rows < 0) continue;
            int pr = 0;
            for (int q = 2; q >= 0; q--)
                if (xv.prs[q] >= rows) pr = xv.prs[q];
            const long tm = tpi ? tpi * g.N : cdiv(dm.M, BM), tn = cdiv(dm.Ncols, BN), chunks = cdiv(xred, 16);
            const size_t packed = (size_t)chunks * xr * xs * tn * 2 * xv.WN * 3072;
            if (!pr || packed >= 0x7fffffffull) continue;
            const double macs = (double)BM * BN * 16 * xr * xs / 1.75;      // against the fp32 instruction's rate
            for (long s0 : kSplits) {
                if (s0 > 1 && force_split <= 0 && (s0 > chunks || s0 > 16)) break;
                const long s = force_split > 0 ? (force_split < chunks ? force_split : chunks) : s0;
                const long per = cdiv(chunks, s), splits = cdiv(chunks, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_XCONV; l.tile = v; l.pr = pr; l.blocks = blocks; l.tpi = (int)tpi; l.splits = (int)splits; l.steps = (int)chunks; l.steps_per_split = (int)per;
                l.tiles_m = (int)tm; l.tiles_n = (int)tn;
                l.pre_bytes = pad256(packed);
                if (splits > 1) l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                l.cost = model_cost(tm * tn * splits, xv.WM * xv.WN, xv.occ, macs * per, xv.eff, splits, dm.M, dm.Ncols) + 5000.0;
                if (splits > 1) l.cost -= 7500.0;             // the reduce pass measures about 5 us on these results
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    // the same for layers of few tiles.  They use no scratch but partial sums; they ask for what the laid-out filters of the kernels
    // above take all the same, so that a call that brings less is served, to the bit, as it was before there were either.
    if (!g.bf16 && !blocks && pass != OWT_PASS_BWD_FILTER && (g.H > 1 || g.W > 1) && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) && xr * xs <= 32 &&
        (size_t)g.N * g.H * g.W * g.C < 0x1fffffffull && (size_t)g.N * g.P * g.Q * g.K < 0x1fffffffull && (size_t)g.K * g.R * g.S * g.C < 0x1fffffffull) {
        double clocks_of = 0.0, us_of = 0.0;            // the cheapest by clocks with a chunk to a panel
        for (int v = 0; v < kNumXConvSVariants; v++) {
            const XConvSVariant &xv = kXConvSVariants[v];
            if ((force_tile >= 0 && force_tile != kXConvSFirstTile + v) || xr * xs < xv.TG) continue;
            const long BM = 32 * xv.WM, rows = panel_rows(g, pass, dm, BM);
            if (rows < 0 || rows > xv.prs[2]) continue;
            const long tm = cdiv(dm.M, BM), tn = cdiv(dm.Ncols, 32), chunks = cdiv(cred, 16);
            for (long s0 : kSplits) {
                const long s = force_split > 0 ? (force_split < chunks ? force_split : chunks) : s0;
                const long per = cdiv(chunks, s), splits = cdiv(chunks, per);
                if (force_split <= 0 && (s0 > chunks || s0 > 8 || tm * tn * splits * xv.WM * xv.TG > 8192)) break;
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_XCONVS; l.tile = v; l.pr = rows <= xv.prs[0] ? xv.prs[0] : rows <= xv.prs[1] ? xv.prs[1] : xv.prs[2];
                l.splits = (int)splits; l.steps = (int)chunks; l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)tn;
                l.pre_bytes = pad256((size_t)chunks * xr * xs * cdiv(dm.Ncols, 64) * 2 * 3072);
                if (splits > 1) l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                // More than 8192 wavefronts (two rounds of the chip), or a SIMD with more than 96 steps to take in all, are left to
                // xconv.hpp: 75 us against 62 at 12912 wavefronts, 34.6 against 29.8 at 112 steps, 42.1 against 37.6 at 168, while 10 % is
                // the most that was won there.
                const long wgs = tm * tn * splits, occ = std::max(1, 16 / (xv.WM * xv.TG)), full = cdiv(wgs, 256);
                const double waves = std::min(occ, full) * xv.WM * xv.TG / 4.0, rounds = (double)cdiv(wgs, 256 * occ);
                const long in_panel = xconvs_chunks(xv.WM, xv.TG, l.pr), panels = cdiv(per, in_panel);
                const long steps = per / in_panel * cdiv(in_panel * xr * xs, xv.TG) + cdiv(per % in_panel * xr * xs, xv.TG);
                // with a chunk to a panel, by clocks: a tap of a chunk 367 (backward-data, with its 4-byte filter loads, 545) times the
                // wavefronts on a SIMD, a panel 1122 and a quarter of one a row and wavefront (twice that with the mask's loads)
                const double loads = pass == OWT_PASS_BWD_DATA && g.masked ? 2.0 : 1.0;
                const double clocks = 0.6 * (rounds * per * (cdiv(xr * xs, xv.TG) * waves * (pass == OWT_PASS_FWD ? 367.0 : 545.0) + 1122.0 + 0.257 * l.pr * loads * waves) + 10900.0) +
                                      (splits > 1 ? 2770.0 + (double)splits * dm.M * dm.Ncols * 4.0 / 933.0 : 0.0);
                const XConvSUs &u = kXConvSUs[pass == OWT_PASS_BWD_DATA][v];
                const double on_simd = (double)full * xv.WM * xv.TG / 4.0, pieces = (double)cdiv(2 * in_panel * l.pr, 64 * xv.WM * xv.TG) * loads;
                l.cost = u.at + on_simd * (u.work * steps + (cred % 4 ? u.rows * per * l.pr : 0.0)) + u.wg * full + rounds * (u.lat * steps + u.load * panels * pieces + u.round) +
                         (splits > 1 ? u.split + u.mb * 4e-6 * splits * dm.M * dm.Ncols : 0.0);
                if (l.partial_bytes <= kMaxPartialBytes && cdiv(xr * xs, xv.TG) * per * waves * rounds <= 96.0) {
                    if (demand) demand->push_back({clocks, l.ws_bytes(), true});
                    if (us_of == 0.0 || clocks < clocks_of) { clocks_of = clocks; us_of = l.cost; }
                }
                if (force_split <= 0 && force_tile < 0 && steps * waves * rounds > 96.0) continue;
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
        // xconv's prices stay, so these stand to its cheapest launch as the microseconds of both do.  xconv's: fitted to 2500 drawn passes that
        // either may be the faster one on, 0.07 in the logarithm: its clocks, rounds, and values that are loaded one by one.  What is nearly as fast
        // here stays here, the error is 0.8 times xconv's.  Of these passes 111 take more than 3 % longer than on the other kernel and all 61.4 ms,
        // the fastest 60.9; with both by clocks 201 and 61.9, with the clocks of one chunk to a panel 264 and 62.1.  Where there is no xconv, as by clocks.
        const Launch *xc = cheapest_of(out, KIND_XCONV);
        double scale = us_of > 0.0 ? clocks_of / us_of : 1260.0;
        if (xc) {
            const bool masks = pass == OWT_PASS_BWD_DATA && g.masked;
            const double rounds = (double)cdiv((long)xc->tiles_m * xc->tiles_n * xc->splits, 256), by_one = cred % 4 ? (masks ? 7.28e-3 : 2.25e-3) : 0.0;
            scale = (masks ? 1.0 : 0.96) * xc->cost / (2.2 + 0.8 * xc->cost / 1260.0 - (xc->splits > 1 ? 1.1 : 0.0) + rounds * (1.1 + by_one * xc->steps_per_split * xc->pr));
        }
        for (Launch &l : out)
            if (l.kind == KIND_XCONVS) l.cost *= scale;
    }
    if (g.bf16 && cred % 8 == 0 && !forced(OWT_FORCE_NO_BF16_MFMA)) {      // the bf16 MFMA: 64-channel chunks, or 32 in the 512x64 tile
        for (int t : {TILE_128x128, TILE_128x64, TILE_256x64, TILE_512x64, TILE_256x64P}) {
            if (no_direct || (force_tile >= 0 && force_tile != t)) continue;
            const long BM = kTiles[t].BM, rows = direct_panel_rows(g, pass, dm, BM);
            int pr;
            const bool pipelined = t == TILE_512x64 || t == TILE_256x64P;
            if (pipelined && (dm.Ncols % 4 || cred % 32 || g.R * g.S > 32)) continue;
            if (t == TILE_512x64) { if (rows < 0 || rows > 624) continue; pr = rows <= 544 ? 544 : 624; }
            else if (t == TILE_256x64 || t == TILE_256x64P) { if (rows < 0 || rows > 384) continue; pr = rows <= 288 ? 288 : 384; }
            else { if (rows < 0 || rows > 256) continue; pr = rows <= 160 ? 160 : 256; }
            const long bk = pipelined ? 32 : 64, chunks = cdiv(cred, bk);
            // ~6x the fp32 MFMA rate; the pipelined tile keeps the matrix unit about 1.5x busier
            const double macs = (double)BM * 64 * kTiles[t].WN * bk * g.R * g.S / (pipelined ? 9.0 : 6.0);
            const size_t n0 = out.size();
            for (long s : kSplits) {
                if (s > 1 && (chunks / s < 1 || s > 8 || s > chunks)) break;
                add(KIND_DIRECT16, t, pr, chunks, s, macs, t == TILE_256x64P ? 3 : 2, 1.25);
                if (force_split > 0) break;
            }
            if (pass == OWT_PASS_BWD_DATA)
                for (size_t i = n0; i < out.size(); i++) out[i].pre_bytes = pad256((size_t)g.K * g.R * g.S * g.C * 2);
        }
    }
    // bf16 storage where the pipelined kernel above is no candidate (channels not in whole chunks of 32, maps wider than its panel,
    // strided layers): the same loop with panel pieces at any address.
    bool whole = false;                                 // the pipelined kernel takes it as it is
    for (const Launch &o : out) whole |= o.kind == KIND_DIRECT16 && (o.tile == TILE_512x64 || o.tile == TILE_256x64P);
    if (g.bf16 && pass != OWT_PASS_BWD_FILTER && (g.H > 1 || g.W > 1) && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) && xr * xs >= 2 && xr * xs <= 32 &&
        (force_tile < 0 ? !whole : force_tile == kDirect16xTile) &&
        (!blocks || (pass == OWT_PASS_FWD && 2L * g.R * g.S >= xr * xs * g.sh * g.sw && g.sh * g.sw <= 32 && xred <= 256)) &&
        (size_t)g.N * g.H * g.W * g.C < 0x3ffffff0ull && (size_t)g.N * g.P * g.Q * g.K < 0x3ffffff0ull) {
        const long rows = panel_rows(g, pass, dm, 256, blocks), chunks = cdiv(xred, 32), tm = cdiv(dm.M, 256), tn = cdiv(dm.Ncols, 64);
        const size_t packed = (size_t)dm.Ncols * xr * xs * chunks * 64;
        if (rows >= 0 && rows <= 512 && packed < 0x7fffffffull) {
            for (long s0 : kSplits) {
                if (s0 > 1 && force_split <= 0 && (s0 > chunks || s0 > 16)) break;
                const long s = force_split > 0 ? (force_split < chunks ? force_split : chunks) : s0;
                const long per = cdiv(chunks, s), splits = cdiv(chunks, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_DIRECT16X; l.tile = 0; l.pr = rows <= 288 ? 288 : rows <= 384 ? 384 : 512; l.blocks = blocks;
                l.splits = (int)splits; l.steps = (int)chunks; l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)tn;
                l.pre_bytes = pad256(packed);
                if (splits > 1) l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                l.cost = model_cost(tm * tn * splits, 4, 2, 256.0 * 64 * 32 * xr * xs * per / 9.0, 1.25, splits, dm.M, dm.Ncols) + 5000.0;
                if (blocks) {                             // fitted to 294 launches of strided layers, 0.09 in the logarithm
                    double rounds, resident;
                    wg_rounds(tm * tn * splits, 2, rounds, resident);
                    const double outs = dm.M * dm.Ncols * (dm.Ncols % 2 ? 4e-6 : 2e-6);
                    l.fitted = true;
                    l.cost = 1260.0 * (15.3 + 0.355 * xr * xs * per * rounds + 0.44 * per * l.pr / 64.0 * resident + (splits > 1 ? 0.6 + 0.85 * splits * dm.M * dm.Ncols * 4e-6 : 0.535 * outs));
                }
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    const bool priced16 = g.bf16 && pass != OWT_PASS_BWD_FILTER && !blocks && !whole && (g.H > 1 || g.W > 1);
    if (priced16)
        for (Launch &l : out) { l.cost = 1260.0 * conv16_us(l, pass, g, dm); l.fitted = true; }
    // bf16 layers of few tiles.  They ask for the scratch of the kernel above, so that a call that brings less is served as it was
    // before there were either.  Layers that the pipelined kernel takes whole keep it (11.1 us against 5.8 for 2 images of 17x16, 64 ->
    // 32): sums in another order round a few bf16 activations the other way, and in a network of a few images one of them moves a
    // pool's maximum.
    double best_us = 0;
    for (const Launch &o : out) best_us = best_us > 0 ? std::min(best_us, o.cost / 1260.0) : o.cost / 1260.0;
    if (g.bf16 && !blocks && (force_tile >= 0 || !whole) && pass != OWT_PASS_BWD_FILTER && (g.H > 1 || g.W > 1) && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) && xr * xs <= 32 &&
        (size_t)g.N * g.H * g.W * g.C < 0x1fffffffull && (size_t)g.N * g.P * g.Q * g.K < 0x1fffffffull &&
        (size_t)g.K * g.R * g.S * g.C < 0x3ffffff0ull) {
        for (int v = 0; v < kNumDConv16SVariants; v++) {
            const DConv16SVariant &xv = kDConv16SVariants[v];
            if ((force_tile >= 0 && force_tile != kDConv16SFirstTile + v) || xr * xs < xv.TG) continue;
            const long BM = 32 * xv.WM, rows = panel_rows(g, pass, dm, BM);
            if (rows < 0 || rows > xv.prs[2]) continue;
            if (pass == OWT_PASS_BWD_DATA && g.masked && cred % 2 && !dconv16s_masked_fits(xv, (int)rows)) continue;
            const long tm = cdiv(dm.M, BM), tn = cdiv(dm.Ncols, 32), chunks = cdiv(cred, 32);
            for (long s0 : kSplits) {
                const long s = force_split > 0 ? (force_split < chunks ? force_split : chunks) : s0;
                const long per = cdiv(chunks, s), splits = cdiv(chunks, per);
                if (force_split <= 0 && (s0 > chunks || s0 > 8 || tm * tn * splits * xv.WM * xv.TG > 8192)) break;
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_DIRECT16S; l.tile = v; l.pr = rows <= xv.prs[0] ? xv.prs[0] : rows <= xv.prs[1] ? xv.prs[1] : xv.prs[2];
                l.splits = (int)splits; l.steps = (int)chunks; l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)tn;
                l.pre_bytes = pad256((size_t)dm.Ncols * xr * xs * chunks * 64);
                if (splits > 1) l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                // 5.15 us; a tap's step 150 clocks times the wavefronts on a SIMD and 36 more a filter load (98 where the 32 lanes' loads of
                // 2 or 4 bytes fall in as many lines), a chunk's panel 866 and its loads; the reduce pass 3.4 us and 0.43 us a MB.
                const int e = cred % 8 == 0 ? 8 : cred % 2 == 0 ? 2 : 1, mk = pass == OWT_PASS_BWD_DATA && g.masked ? 2 : 1;
                const bool fwd = pass == OWT_PASS_FWD;
                const double loads = (!fwd || e == 1 ? 16 : e == 2 ? 8 : 2) * (cred <= 16 ? 0.5 : 1.0), piece = (e == 8 ? 1 : e == 2 ? 4 : 8) * mk * l.pr / 64.0;
                const bool heavy = e == 1 && mk == 2 && l.pr == xv.prs[2] && xv.WM == 1;      // registers for one work-group a CU
                const long wgs = tm * tn * splits, occ = heavy ? 1 : std::max(1, 16 / (xv.WM * xv.TG)), full = cdiv(wgs, 256);
                const double waves = std::min(occ, full) * xv.WM * xv.TG / 4.0, rounds = (double)cdiv(wgs, 256 * occ), taps = cdiv(xr * xs, xv.TG);
                double us = 5.15 + rounds * per * (taps * waves * (150.0 + (fwd && e < 8 ? 98.4 : 36.2) * loads) + 866.0 + 13.0 * piece * waves) / 2100.0;
                // (values and masks one by one: wavefronts wait for a panel's loads in front of their filters, those of the smaller tiles longer.
                // Over 164 passes of wide and of odd layers the choice takes 2512 us, 2592 without this, the fastest kernels 2428)
                if (e == 1 && mk == 2) us = 1.1 * (us + (xv.WM == 4 ? 0.0 : rounds * per * (heavy ? 2.5 : xv.WM == 2 ? 1.0 : 0.5)));
                if (splits > 1) us += 3.35 + 0.426 * splits * dm.M * dm.Ncols * 4e-6;
                if (force_tile < 0 && ((best_us > 0 && us > best_us) || rounds * per * taps * waves > 96.0)) continue;
                l.cost = 1260.0 * us;
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    SConvGeom scg;
    // test hook: tile 20 = only the filter-streaming first-layer forward kernel, 21 = only the filters-in-LDS one
    const bool sconv_ok = pass == OWT_PASS_FWD && !no_direct && (force_tile < kXConvFirstTile || out.empty()) && sconv_geom(g, scg);
    if (sconv_ok && force_tile != 20 && !g.bf16 && sconv2_fits(g, scg)) {
        const long ktiles = cdiv(g.K, kSConv2KB);
        for (long target : {256L, 512L}) {
            long wgs = target / ktiles > 0 ? target / ktiles : 1;
            if (force_split > 0) wgs = force_split;
            if (wgs > scg.units) wgs = scg.units;
            const long per = cdiv(scg.units, wgs), n = cdiv(scg.units, per);
            Launch l; memset(&l, 0, sizeof(l));
            l.kind = KIND_SCONV2; l.splits = 1; l.steps = scg.units; l.steps_per_split = (int)per;
            l.tiles_m = (int)ktiles; l.tiles_n = (int)n;
            l.partial_bytes = pad256((size_t)g.K * scg.KSLOTS * 4);          // the re-laid-out filters
            l.cost = model_cost(ktiles * n, 8, 1, 256.0 * kSConv2KB * scg.KSLOTS * per, 1.2, 1, dm.M, dm.Ncols);
            bool dup = false;
            for (const Launch &o : out) dup |= o.kind == l.kind && o.tiles_n == l.tiles_n;
            if (!dup) out.push_back(l);
            if (force_split > 0) break;
        }
    }
    if (sconv_ok && force_tile != 21) {
        const long ktiles = cdiv(g.K, 64);
        for (long target : {256L, 512L}) {
            long wgs = target / ktiles > 0 ? target / ktiles : 1;
            if (force_split > 0) wgs = force_split;
            if (wgs > scg.units) wgs = scg.units;
            const long per = cdiv(scg.units, wgs), n = cdiv(scg.units, per);
            Launch l; memset(&l, 0, sizeof(l));
            l.kind = KIND_SCONV; l.splits = 1; l.steps = scg.units; l.steps_per_split = (int)per;
            l.tiles_m = (int)ktiles; l.tiles_n = (int)n;
            l.partial_bytes = pad256((size_t)g.K * scg.KSLOTS * 4);          // the re-laid-out filters
            // (bf16 storage: the bf16-MFMA kernel below, when it applies, is the faster one)
            l.cost = model_cost(ktiles * n, 8, 1, 256.0 * 64 * scg.KSLOTS * per, 1.0, 1, dm.M, dm.Ncols) * (g.bf16 ? 2.0 : 1.0);
            bool dup = false;
            for (const Launch &o : out) dup |= o.kind == l.kind && o.tiles_n == l.tiles_n;
            if (!dup) out.push_back(l);
            if (force_split > 0) break;
        }
    }
    SConv16Geom s16g;
    if (pass == OWT_PASS_FWD && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) && sconv16_geom(g, s16g)) {
        const long ktiles = cdiv(g.K, 64);
        for (long target : {256L, 512L}) {
            long wgs = target / ktiles > 0 ? target / ktiles : 1;
            if (force_split > 0) wgs = force_split;
            if (wgs > s16g.units) wgs = s16g.units;
            const long per = cdiv(s16g.units, wgs), n = cdiv(s16g.units, per);
            Launch l; memset(&l, 0, sizeof(l));
            l.kind = KIND_SCONV16; l.splits = 1; l.steps = s16g.units; l.steps_per_split = (int)per;
            l.tiles_m = (int)ktiles; l.tiles_n = (int)n;
            l.partial_bytes = pad256((size_t)g.K * s16g.KSLOTS * 2);        // the re-laid-out filters
            // One work-group a CU (its LDS): the launches and the filter bank, and a unit of four rows what its reduction and its band take
            // (fitted to 83 launches, 0.11 in the logarithm).  Two work-groups a CU go one after the other and load the bank twice: 128
            // images of 224x224 to 96 filters of 11x11 66 us with 256 work-groups, 76 with 512; 39 of 192x192 to 64 21.5 and 29.4.
            l.fitted = true;
            l.cost = 1260.0 * cdiv(ktiles * n, 256) * (8.7 + 0.0065 * s16g.KSLOTS + per * (2.17 + 0.003 * s16g.KSLOTS + 5.0e-5 * s16g.ROWS * g.W * g.C));
            bool dup = false;
            for (const Launch &o : out) dup |= o.kind == l.kind && o.tiles_n == l.tiles_n;
            if (!dup) out.push_back(l);
            if (force_split > 0) break;
        }
    }
    // test hook: tile 22 = only the register-staged first-layer filter-gradient kernel, 23 = only the one that streams
    // its units straight into LDS
    SFilterGeom sfg;
    const bool sfilter_ok = pass == OWT_PASS_BWD_FILTER && !no_direct && force_tile < kXConvFirstTile && (g.sh > 1 || g.sw > 1) && sfilter_geom(g, sfg);
    for (int form = 0; form < 2 && sfilter_ok; form++) {
        if (form == 0 ? force_tile == 23 : (force_tile == 22 || !sfilter2_fits(g, sfg))) continue;
        const long ktiles = cdiv(g.K, 64);
        for (long target : {256L, 512L, 1024L}) {
            long wgs = target / ktiles > 0 ? target / ktiles : 1;
            if (force_split > 0) wgs = force_split;
            if (wgs > sfg.units) wgs = sfg.units;
            const long per = cdiv(sfg.units, wgs), splits = cdiv(sfg.units, per);
            Launch l; memset(&l, 0, sizeof(l));
            l.kind = form ? KIND_SFILTER2 : KIND_SFILTER; l.tile = 0; l.splits = (int)splits; l.steps = sfg.units; l.steps_per_split = (int)per;
            l.tiles_m = (int)ktiles; l.tiles_n = 1;
            if (splits > 1) {
                l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
            }
            l.cost = model_cost(ktiles * splits, 8, form ? 1 : 2, 64.0 * sfg.NB * 32 * sfg.DZP * per, form ? 1.15 : 1.0, splits, dm.M, dm.Ncols);
            bool dup = false;
            for (const Launch &o : out) dup |= o.kind == l.kind && o.splits == l.splits;
            if (!dup) out.push_back(l);
            if (force_split > 0) break;
        }
    }
    // test hook: tile 24 = only the register-staged bf16 first-layer filter-gradient kernel, 25 = only the one that
    // streams its units straight into LDS
    SFilter16Geom sf16g;
    const bool sf16_ok = pass == OWT_PASS_BWD_FILTER && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) && (g.sh > 1 || g.sw > 1) &&
                         sfilter16_geom(g, sf16g);
    for (int form = 0; form < 2 && sf16_ok; form++) {
        if (form == 0 ? force_tile == 25 : (force_tile == 24 || !sfilter16b_fits(g, sf16g))) continue;
        const long ktiles = cdiv(g.K, 64);
        for (long target : {256L, 512L, 1024L}) {
            long wgs = target / ktiles > 0 ? target / ktiles : 1;
            if (force_split > 0) wgs = force_split;
            if (wgs > sf16g.units) wgs = sf16g.units;
            const long per = cdiv(sf16g.units, wgs), splits = cdiv(sf16g.units, per);
            Launch l; memset(&l, 0, sizeof(l));
            l.kind = form ? KIND_SFILTER16B : KIND_SFILTER16; l.tile = 0; l.splits = (int)splits; l.steps = sf16g.units; l.steps_per_split = (int)per;
            l.tiles_m = (int)ktiles; l.tiles_n = 1;
            if (splits > 1) {
                l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
            }
            l.cost = model_cost(ktiles * splits, 8, 1, 64.0 * sf16g.NB * 32 * sf16g.DZP * per / 5.0, form ? 1.3 : 1.0, splits, dm.M, dm.Ncols);
            bool dup = false;
            for (const Launch &o : out) dup |= o.kind == l.kind && o.splits == l.splits;
            if (!dup) out.push_back(l);
            if (force_split > 0) break;
        }
    }
    double images_clocks = 1e30;                        // the cheapest filter gradient over images by the clocks of its matrix and vector instructions
    // fp32 storage on the bf16 matrix unit with split operands: stride 1, one wavefront per (filters, channels, filter row);
    // the bias gradient is summed by the filter row that meets every output row, which there is when P <= H
    if (pass == OWT_PASS_BWD_FILTER && !g.bf16 && g.sh == 1 && g.sw == 1 && g.P <= g.H && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) &&
        image_groups_fit(g, false)) {
        for (int v = 0; v < kNumXFilterVariants; v++) {
            const XFilterVariant &xv = kXFilterVariants[v];
            if ((force_tile >= 0 && force_tile != kXFilterFirstTile + v) || g.S != xv.S) continue;
            const long tm = cdiv(g.K, 32 * xv.KB), ctl = cdiv(g.C, 32), tiles = tm * ctl * g.R, steps = cdiv(g.N, 16) * g.P * g.Q;
            for (long s0 : split_ladder(tiles, xv.TG > 1 ? 512 : 1024)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 4 || tiles * s * xv.TG > 4096)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_XFILTER; l.tile = v; l.splits = (int)splits; l.steps = (int)steps; l.steps_per_split = (int)per;
                l.tiles_m = (int)tm; l.tiles_n = (int)(ctl * g.R); l.ctiles = (int)ctl; l.taps = g.S; l.groups = g.R;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                if (xv.TG == 1 && l.partial_bytes <= kMaxPartialBytes) {
                    const double clocks = 0.6 * (per * (192.0 * xv.KB * xv.S * 1.15) + (per / g.Q + 1.0) * 1600.0 + 6000.0) * cdiv(tiles * splits, 1024) +
                                          (splits > 1 ? 6500.0 + (double)(splits + 1) * dm.M * dm.Ncols * 4.0 / 1300.0 : 0.0);
                    images_clocks = std::min(images_clocks, clocks);
                    if (demand) demand->push_back({clocks, l.ws_bytes(), true});
                }
                l.cost = 1260.0 * images32_us(l, kXFilterUs[v], xv.TG, xfilter_occ(xv.KB, xv.S, xv.TG), (1.0 + xv.KB) + 0.5 * xv.KB * g.masked, xv.S, xv.KB * xv.S, g, dm);
                l.fitted = true;
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    // the same for any geometry, columns packed densely (not the fully-connected shard, whose two backward products share
    // a launch)
    if (pass == OWT_PASS_BWD_FILTER && !g.bf16 && (g.H > 1 || g.W > 1) && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) &&
        image_groups_fit(g, true)) {
        for (int v = 0; v < kNumXGatherVariants; v++) {
            const XGatherVariant &xv = kXGatherVariants[v];
            if (force_tile >= 0 && force_tile != kXGatherFirstTile + v) continue;
            const long tm = cdiv(g.K, 32 * xv.KB), tn = cdiv(dm.Ncols, 32 * xv.CB), tiles = tm * tn, steps = cdiv(g.N, 16) * g.P * g.Q;
            for (long s0 : split_ladder(tiles, xv.TG > 1 ? 512 : 1024)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 4 || tiles * s * xv.TG > 4096)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_XGATHER; l.tile = v; l.splits = (int)splits; l.steps = (int)steps; l.steps_per_split = (int)per;
                l.tiles_m = (int)tm; l.tiles_n = (int)tn; l.blocks = g.sh > 1 || g.sw > 1;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                if (xv.TG == 1 && l.partial_bytes <= kMaxPartialBytes) {
                    const double clocks = 0.6 * (per * (330.0 * (xv.KB + xv.CB) + 100.0) + 6000.0) * cdiv(tiles * splits, 1024) +
                                          (splits > 1 ? 6500.0 + (double)(splits + 1) * dm.M * dm.Ncols * 4.0 / 1300.0 : 0.0);
                    images_clocks = std::min(images_clocks, clocks);
                    if (demand) demand->push_back({clocks, l.ws_bytes(), true});
                }
                l.cost = 1260.0 * images32_us(l, kXGatherUs[v], xv.TG, xv.TG > 1 ? 2 : 1, (xv.KB + xv.CB) + 0.5 * xv.KB * g.masked, 0, xv.KB * xv.CB, g, dm);
                l.fitted = true;
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    if (pass == OWT_PASS_BWD_FILTER && !no_direct) {
        for (int v = 0; v < kNumDFilterVariants; v++) {
            int taps, groups;
            if (force_tile >= 0 && force_tile != v) continue;
            if (!dfilter_fits(g, v, taps, groups)) continue;
            if (v == 2 && g.K % 128 == 0) continue;                  // variant 0 covers it with the same accumulators
            const DFilterVariant &dv = kDFilterVariants[v];
            const long KT = 32 * dv.WK, CT = 32 * dv.WC;
            const long tm = cdiv(g.K, KT), ctl = cdiv(g.C, CT);
            const long steps = dv.aligned ? (long)g.N * cdiv((long)g.P * g.Q, 32) : cdiv(dm.Kd, 32);
            for (long s0 : split_ladder(tm * ctl * groups, 256 * dv.occ)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 2 || tm * ctl * groups * s > 2560)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_DFILTER; l.tile = v; l.splits = (int)splits; l.steps = (int)steps;
                l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)(ctl * groups);
                l.taps = taps; l.groups = groups; l.ctiles = (int)ctl;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                l.cost = model_cost(tm * ctl * groups * splits, dv.WK * dv.WC, dv.occ, (double)KT * CT * 32 * taps * per, 1.2, splits,
                                    dm.M, dm.Ncols);
                bool dup = false;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup && (l.partial_bytes <= kMaxPartialBytes || force_split > 0) &&
                    (force_split > 0 || tm * ctl * groups * splits >= 128 || s0 == 256)) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    if (pass == OWT_PASS_BWD_FILTER && !no_direct) {
        for (int v = 0; v < kNumDFilter2Variants; v++) {
            int taps, groups;
            if (force_tile >= 0 && force_tile != kDFilter2FirstTile + v) continue;
            if (!dfilter2_fits(g, v, taps, groups)) continue;
            const DFilter2Variant &dv = kDFilter2Variants[v];
            const long KT = 32 * dv.WK, CT = 32, BP = 32 * dv.WP;
            const long tm = cdiv(g.K, KT), ctl = cdiv(g.C, CT), steps = cdiv(dm.Kd, BP);
            for (long s0 : split_ladder(tm * ctl * groups, 256)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 2 || tm * ctl * groups * s > 1280)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_DFILTER2; l.tile = v; l.splits = (int)splits; l.steps = (int)steps;
                l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)(ctl * groups);
                l.taps = taps; l.groups = groups; l.ctiles = (int)ctl;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                l.cost = model_cost(tm * ctl * groups * splits, dv.WK * dv.WP, 1, (double)KT * CT * BP * taps * per, 1.3, splits,
                                    dm.M, dm.Ncols);
                bool dup = false;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup && (l.partial_bytes <= kMaxPartialBytes || force_split > 0) &&
                    (force_split > 0 || tm * ctl * groups * splits >= 64 || s0 == 256)) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    if (pass == OWT_PASS_BWD_FILTER && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA)) {
        for (int v = 0; v < kNumDFilter16bVariants; v++) {
            int taps, groups;
            if (force_tile >= 0 && force_tile != kDFilter16bFirstTile + v) continue;
            if (!dfilter16b_fits(g, v, taps, groups)) continue;
            const DFilter16bVariant &dv = kDFilter16bVariants[v];
            const long KT = 32 * dv.KB * dv.WK, CT = 32 * dv.WC;
            const long tm = cdiv(g.K, KT), ctl = cdiv(g.C, CT), steps = cdiv(dm.Kd, kDFilter16BP);
            for (long s0 : split_ladder(tm * ctl * groups, 256)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 2 || tm * ctl * groups * s > 1280)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                if (per > kDFilter16bMaxChunks) { if (force_split > 0) break; continue; }
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_DFILTER16B; l.tile = v; l.splits = (int)splits; l.steps = (int)steps;
                l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)(ctl * groups);
                l.taps = taps; l.groups = groups; l.ctiles = (int)ctl;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                l.cost = model_cost(tm * ctl * groups * splits, dv.WK * dv.WC, 1,
                                    (double)KT * CT * kDFilter16BP * taps * per / 5.0, 1.5, splits, dm.M, dm.Ncols);
                bool dup = false;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup && (l.partial_bytes <= kMaxPartialBytes || force_split > 0) &&
                    (force_split > 0 || tm * ctl * groups * splits >= 64 || s0 == 256)) out.push_back(l);
                if (force_split > 0) break;
            }
        }
        for (int v = 0; v < kNumDFilter16Variants; v++) {
            int taps, groups;
            if (force_tile >= 0 && force_tile != v) continue;
            if (!dfilter16_fits(g, v, taps, groups)) continue;
            const DFilter16Variant &dv = kDFilter16Variants[v];
            const long KT = 32 * dv.KB * dv.WK, CT = 32 * dv.WC;
            const long tm = cdiv(g.K, KT), ctl = cdiv(g.C, CT), steps = cdiv(dm.Kd, kDFilter16BP);
            for (long s0 : split_ladder(tm * ctl * groups, 256)) {            // one or two work-groups per CU
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 2 || tm * ctl * groups * s > 1280)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_DFILTER16; l.tile = v; l.splits = (int)splits; l.steps = (int)steps;
                l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)(ctl * groups);
                l.taps = taps; l.groups = groups; l.ctiles = (int)ctl;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                l.cost = model_cost(tm * ctl * groups * splits, dv.WK * dv.WC, dv.occ,
                                    (double)KT * CT * kDFilter16BP * taps * per / 5.0, 1.2,
                                    splits, dm.M, dm.Ncols);
                bool dup = false;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup && (l.partial_bytes <= kMaxPartialBytes || force_split > 0) &&
                    (force_split > 0 || tm * ctl * groups * splits >= 64 || s0 == 256)) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    // the same with the reduction over images and the operands streamed straight into LDS; one or two images, of which a group of 16 is
    // mostly zeros, are left to the other kernels (2 images 30x22, 288 -> 488: 50 us, 29 on dfilter16b)
    if ((force_tile >= 0 || g.N > 2) && pass == OWT_PASS_BWD_FILTER && g.bf16 && !g.masked && g.sh == 1 && g.sw == 1 && g.P <= g.H && g.C % 8 == 0 && g.K % 8 == 0 && !no_direct &&
        !forced(OWT_FORCE_NO_BF16_MFMA) && image_groups_fit(g, false)) {
        for (int v = 0; v < kNumIFilter16bVariants; v++) {
            const IFilter16bVariant &iv = kIFilter16bVariants[v];
            if ((force_tile >= 0 && force_tile != kIFilter16bFirstTile + v) || g.S != iv.S) continue;
            const long KT = 32 * iv.KB * iv.WK, CT = 32 * iv.CB * iv.WC;
            // dw is stored with 32-bit byte offsets, rows of a ragged tile included, and 2^31 stands for a channel past the last, to
            // which a block's rows are added: no offset may come round past 2^32, nor that one lie inside dw
            if ((double)cdiv(g.K, KT) * KT * dm.Ncols * 4.0 > 2147483648.0) continue;
            const long tm = cdiv(g.K, KT), ctl = cdiv(g.C, CT), tiles = tm * ctl * g.R, steps = cdiv(g.N, 16) * g.P * g.Q;
            for (long s0 : split_ladder(tiles, 256 * iv.occ)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 8 || tiles * s > 2048)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_IFILTER16B; l.tile = v; l.splits = (int)splits; l.steps = (int)steps; l.steps_per_split = (int)per;
                l.tiles_m = (int)tm; l.tiles_n = (int)(ctl * g.R); l.ctiles = (int)ctl; l.taps = g.S; l.groups = g.R;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                l.cost = 1260.0 * ifilter16b_us(l, g, dm);
                l.fitted = true;
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    // bf16 storage where the kernels above are no candidates (channels or filters not in eights, rows too wide for their panels), or
    // would leave most of their 128-wide tiles empty on a large batch: the reduction over images.  Timed, us, kernels above -> this one: 419 images
    // 42x8, 32 -> 32 55 -> 36; 375 images 29x19, 64 -> 32 53 -> 41; 761 images 8x26, 96 -> 8 49 -> 39; but 43 images 17x22, 64 -> 8
    // 18 -> 22; 53 images 25x7, 64 -> 192 27 -> 30; 89 images 20x12, 32 -> 120 5x5 35 -> 42, and whole tiles half as fast.
    bool staged16 = false;
    for (const Launch &o : out) staged16 |= (o.kind == KIND_DFILTER16 || o.kind == KIND_DFILTER16B) && (g.K > 64 || g.C > 96 || g.N < 128);
    std::vector<ImagesDemand> images16;
    if ((force_tile < 0 ? !staged16 : force_tile >= kIFilter16FirstTile && force_tile < kIGather16FirstTile) && pass == OWT_PASS_BWD_FILTER && g.bf16 && g.sh == 1 && g.sw == 1 && g.P <= g.H && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) &&
        image_groups_fit(g, false)) {
        for (int v = 0; v < kNumIFilter16Variants; v++) {
            const IFilter16Variant &iv = kIFilter16Variants[v];
            if ((force_tile >= 0 && force_tile != kIFilter16FirstTile + v) || g.S != iv.S) continue;
            const long tm = cdiv(g.K, 32 * iv.KB), ctl = cdiv(g.C, 32 * iv.CB), tiles = tm * ctl * g.R, steps = cdiv(g.N, 16) * g.P * g.Q;
            const int occ = ifilter16_occ(iv.KB, iv.CB, iv.S), zl = iv.KB == 2 && g.K % 2 ? 16 : 8, xl = iv.CB == 2 && g.C % 2 ? 16 : 8;
            const double column = 31.0 * iv.KB * iv.CB * iv.S + 29.0 * ((g.masked ? 2 : 1) * zl + xl);
            if (demand)
                images16_demand(images16, split_ladder(tiles, 1024L * occ), g, dm, want_db, tiles, steps, occ, 650.0, column, iv.S, iv.KB * iv.CB * iv.S, true);
            for (long s0 : split_ladder(tiles, 256L * occ)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 4 || tiles * s > 2048)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_IFILTER16; l.tile = v; l.splits = (int)splits; l.steps = (int)steps; l.steps_per_split = (int)per;
                l.tiles_m = (int)tm; l.tiles_n = (int)(ctl * g.R); l.ctiles = (int)ctl; l.taps = g.S; l.groups = g.R;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                l.cost = 1260.0 * images16_us(l, kIFilter16Us[v], occ, column, iv.S, iv.KB * iv.CB * iv.S, g, dm);
                l.fitted = true;
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    // the same for any geometry (not the fully-connected shard), where no other kernel on the bf16 matrix unit is a candidate
    bool rows16 = false;
    for (const Launch &o : out)
        rows16 |= o.kind == KIND_DFILTER16 || o.kind == KIND_DFILTER16B || o.kind == KIND_IFILTER16 || o.kind == KIND_SFILTER16 || o.kind == KIND_SFILTER16B;
    if ((force_tile < 0 ? !rows16 : force_tile >= kIGather16FirstTile) && pass == OWT_PASS_BWD_FILTER && g.bf16 && (g.H > 1 || g.W > 1) && !no_direct &&
        !forced(OWT_FORCE_NO_BF16_MFMA) && image_groups_fit(g, true)) {
        for (int v = 0; v < kNumIGather16Variants; v++) {
            const IGather16Variant &iv = kIGather16Variants[v];
            if (force_tile >= 0 && force_tile != kIGather16FirstTile + v) continue;
            const long tm = cdiv(g.K, 32 * iv.KB), tn = cdiv(dm.Ncols, 32 * iv.CB), tiles = tm * tn, steps = cdiv(g.N, 16) * g.P * g.Q;
            const int zl = (iv.KB == 2 && g.K % 2 ? 16 : 8) * (g.masked ? 2 : 1), occ = zl == 32 ? 1 : 2;
            const double position = 31.0 * iv.KB * iv.CB + 29.0 * (zl + 8 * iv.CB);
            if (demand && iv.CB == 3)
                images16_demand(images16, split_ladder(tiles, 1024L * occ), g, dm, want_db, tiles, steps, occ, 700.0, position, 1, iv.KB * iv.CB, false);
            for (long s0 : split_ladder(tiles, 256L * occ)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                else if (s > 1 && (steps / s < 4 || tiles * s > 2048)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_IGATHER16; l.tile = v; l.splits = (int)splits; l.steps = (int)steps; l.steps_per_split = (int)per;
                l.tiles_m = (int)tm; l.tiles_n = (int)tn; l.blocks = g.sh > 1 || g.sw > 1;
                if (splits > 1) {
                    l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                    l.dbias_bytes = want_db ? pad256((size_t)splits * dm.M * 4) : 0;
                }
                l.cost = 1260.0 * images16_us(l, kIGather16Us[v], occ, position, 1, iv.KB * iv.CB, g, dm);
                l.fitted = true;
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    // plain matrix product (the fully-connected shard), fp32 storage: the dense kernel with operands streamed
    // straight into LDS; needs 16-byte aligned operand rows and, in the forward pass, whole 32-deep
    // reduction steps (the backward passes can read a zero-padded copy of dz instead)
    if (!no_direct && !g.bf16 && g.H == 1 && g.W == 1 && g.R == 1 && g.S == 1 &&
        (pass == OWT_PASS_FWD ? dm.Kd % 32 == 0 : dm.Ncols % 4 == 0)) {
        for (int t = 0; t < kNumFcTiles; t++) {
            if (force_tile >= 0 && force_tile != 16 + t) continue;
            const FcTile &ft = kFcTiles[t];
            const long BM = 32 * ft.MB * ft.WM, BN = 32 * ft.NB * ft.WN;
            const long steps = cdiv(dm.Kd, 32), tm = cdiv(dm.M, BM), tn = cdiv(dm.Ncols, BN);
            for (long s0 : split_ladder(tm * tn, 256 * ft.occ)) {
                long s = s0;
                if (force_split > 0) s = force_split < steps ? force_split : steps;
                if (force_split <= 0 && s > 1 && (steps / s < 2 || tm * tn * s > 2048)) break;
                const long per = cdiv(steps, s), splits = cdiv(steps, per);
                Launch l; memset(&l, 0, sizeof(l));
                l.kind = KIND_FCGEMM; l.tile = t; l.splits = (int)splits; l.steps = (int)steps; l.steps_per_split = (int)per;
                l.tiles_m = (int)tm; l.tiles_n = (int)tn;
                if (splits > 1) l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
                if (pass != OWT_PASS_FWD) l.pre_bytes = pad256((size_t)((g.N + 31) & ~31) * ((g.K + 31) & ~31) * 4);     // padded dz
                l.cost = model_cost(tm * tn * splits, 4, ft.occ, (double)BM * BN * 32 * per, 1.6, splits, dm.M, dm.Ncols);
                if (pass != OWT_PASS_FWD) l.cost += 4000.0;               // half of the launch that forms dz
                bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
                for (const Launch &o : out) dup |= o.kind == l.kind && o.tile == l.tile && o.splits == l.splits;
                if (!dup) out.push_back(l);
                if (force_split > 0) break;
            }
        }
    }
    // the shard on the bf16 matrix unit: 64 x 64 tiles, 16-deep steps; only the forward pass splits the reduction over
    // work-groups (its result is small).  32-bit byte offsets, a tile past the end included.
    const bool plain = g.H == 1 && g.W == 1 && g.R == 1 && g.S == 1;
    const long rows64 = g.N + 64 > g.K + 64 ? g.N + 64 : g.K + 64;
    if (plain && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA | OWT_FORCE_FC_ONE_LAUNCH | OWT_FORCE_FC_TWO_LAUNCHES) &&
        (force_tile < 0 || force_tile == kXFcTile) && (double)rows64 * (g.C + 64) * 4 < 2147483647.0 &&
        (double)(g.N + 64) * (g.K + 64) * 4 < 2147483647.0) {
        const long tm = cdiv(dm.M, 64), tn = cdiv(dm.Ncols, 64), steps = cdiv(dm.Kd, 16);
        const double step_clocks = g.bf16 ? 1500.0 : 2000.0;             // a wavefront's step, its loads' latency included
        for (long s0 : split_ladder(tm * tn, 256)) {
            long s = s0;
            if (force_split > 0) s = force_split < steps ? force_split : steps;
            if (pass != OWT_PASS_FWD) s = 1;
            else if (force_split <= 0 && s > 1 && (steps / s < 4 || s > 64)) break;
            const long per = cdiv(steps, s), splits = cdiv(steps, per);
            Launch l; memset(&l, 0, sizeof(l));
            l.kind = KIND_XFC; l.splits = (int)splits; l.steps = (int)steps; l.steps_per_split = (int)per; l.tiles_m = (int)tm; l.tiles_n = (int)tn;
            if (splits > 1) l.partial_bytes = pad256((size_t)splits * dm.M * dm.Ncols * 4);
            l.cost = 0.6 * (6000.0 + cdiv(per, 4) * step_clocks) * (0.5 + 0.5 * cdiv(tm * tn * splits, 256));
            if (splits > 1) l.cost += 5000.0 + (double)(splits + 1) * dm.M * dm.Ncols * 4.0 / 1300.0;
            bool dup = l.partial_bytes > kMaxPartialBytes && force_split <= 0;
            for (const Launch &o : out) dup |= o.kind == l.kind && o.splits == l.splits;
            if (!dup) out.push_back(l);
            if (force_split > 0 || pass != OWT_PASS_FWD) break;
        }
    }
    // Its forward pass in one launch.  Microseconds of both kernels behind a busy device, fitted to 992 launches each of drawn shards of up to
    // 16000 inputs, 0.06 and 0.10 in the logarithm; the other kernels' prices stay, so this one's stands to the cheapest launch above as
    // the microseconds do.  A wavefront's steps are a chain of loads, one behind the other from the reduction's length on that its own
    // sixteenth is longer than what is in flight: bf16, xfc and here: 16 x 5632 -> 19 7.4 and 11.9 us, 8 x 9379 -> 21 9.5 and 16.2, but 128 x 4096
    // -> 512 11.2 and 10.2.  Weighed by 4963 shards near the line, which take 50.7 ms, the faster kernel of each 50.1; with the line at 4500 and
    // 3000 inputs there was before 16 x 5632 -> 19 and the like took up to 1.85 times as long.
    const Launch *split_fc = cheapest_of(out, KIND_XFC);
    if (plain && pass == OWT_PASS_FWD && !no_direct && !forced(OWT_FORCE_NO_BF16_MFMA) && (force_tile < 0 ? split_fc != nullptr : force_tile == kXFcSTile) && force_split <= 1 &&
        (double)(g.N + 16) * g.C * 4 < 2147483647.0 && (double)(g.K + 16) * g.C * 4 < 2147483647.0) {
        Launch l; memset(&l, 0, sizeof(l));
        l.kind = KIND_XFCS; l.splits = 1; l.steps = l.steps_per_split = (int)cdiv(dm.Kd, 16);
        l.tiles_m = (int)cdiv(dm.M, 16); l.tiles_n = (int)cdiv(dm.Ncols, 16);
        const double tiles = (double)l.tiles_m * l.tiles_n, more = (double)cdiv((long)tiles, 256) - 1.0, I = 1e-3 * dm.Kd, odd = dm.Kd % 2;
        const double rows = (std::min(g.N, 16) + std::min(g.K, 16)) / 32.0;      // (rows past the end are no loads)
        // (rows of whole 128-byte lines: 1.2 times as long near the line, 50 x 2600 -> 188 in fp32 9.4 us, 2720 12.0; a tile of few rows, which
        // xfc is a little faster on than its price, 1.05)
        const double weight = dm.Kd * (g.bf16 ? 2 : 4) % 128 == 0 ? 1.1 : g.bf16 ? 1.0 : rows < 1.0 ? 1.03 : 0.98;
        const double here = weight * (g.bf16 ? 2.12 + I * (0.49 + 0.76 * rows + odd * (0.1 + 0.49 * rows) + 1.62 * more + 0.2 * tiles / 256.0) + 0.57 * more
                                           : 2.47 + I * (1.52 + 1.04 * rows + 2.59 * more + 0.6 * tiles / 256.0) + 0.96 * more);
        l.cost = 1260.0 * here;
        if (split_fc) {
            l.pre_bytes = split_fc->ws_bytes();          // asked for though not used: a call that brings less is served, or refused, as without this kernel
            const double steps = (double)cdiv(split_fc->steps_per_split, 4), sp = split_fc->splits > 1, mb = sp * split_fc->splits * dm.M * dm.Ncols * 4e-6;
            const double rows64 = (std::min(g.N, 64) + std::min(g.K, 64)) / 128.0, more64 = (double)cdiv((long)split_fc->tiles_m * split_fc->tiles_n * split_fc->splits, 256) - 1.0;
            l.cost = split_fc->cost * here / (g.bf16 ? 2.6 + steps * (0.21 + rows64 * (0.34 + 1.93 * odd)) + 4.28 * sp + 0.6 * mb + 21.9 * more64
                                                     : 3.77 + steps * (0.34 + 0.86 * rows64) + 3.69 * sp + 0.785 * mb + 3.66 * more64);
        }
        out.push_back(l);
    }
    // the gather kernel is the fallback of the stride-1 forward / backward-data kernel, and an
    // alternative worth timing next to the direct filter-gradient kernel
    const bool have_direct = !out.empty() && (out[0].kind == KIND_DIRECT || out[0].kind == KIND_DIRECT16);
    for (int t = 0; t < NUM_TILES && !have_direct; t++) {
        if (!vec && t != TILE_64x64) continue;
        if (force_tile >= kDFilter2FirstTile && !out.empty()) continue;
        if (vec && force_tile >= 0 && force_tile < NUM_TILES && t != force_tile) continue;
        const TileInfo &ti = kTiles[t];
        const long ksteps = cdiv(dm.Kd, ti.BK);
        const long tiles = cdiv(dm.M, ti.BM) * cdiv(dm.Ncols, 64 * ti.WN);
        const double macs = (double)ti.BM * 64 * ti.WN * ti.BK;
        for (long s : split_ladder(tiles)) {
            if (s > 1 && (ksteps / s < 4 || tiles * s > 4096)) break;
            // (4-byte gathers: 8 images 32x32x3 -> 16, 5x5 forward takes 21 us here, 16.6 with split operands)
            add(KIND_GATHER, t, 0, ksteps, s, macs, t == TILE_128x128 ? 2 : 5, vec ? ti.eff : 0.6 * ti.eff);
            if (force_split > 0) break;
        }
    }
    // bf16 storage: the kinds that know no microseconds, beside those that do.  Each kind's cheapest launch is priced, the order
    // among its launches stays.
    const auto reduce_clocks = [&](const Launch &l) { return l.splits > 1 ? 14000.0 + (double)(l.splits + 1) * dm.M * dm.Ncols * 4.0 / 1300.0 : 0.0; };
    const auto mb = [&](const Launch &l) { return l.splits > 1 ? l.splits * dm.M * dm.Ncols * 4e-6 : 0.0; };
    const Launch *gather = cheapest_of(out, KIND_GATHER);
    if (g.bf16 && pass == OWT_PASS_FWD && blocks && !forced(OWT_FORCE_NO_BF16_MFMA)) {
        // (strided layers, fitted to 2024 and 145 launches, 0.13 and 0.10 in the logarithm.  In clocks alone the gather kernel looked faster
        // than sconv16 on layers of a few us: 13 -> 22 us for 25 images 72x75x16 to 36 filters of 2x2, stride 2)
        if (gather) {
            const double core = (gather->cost - reduce_clocks(*gather)) / 1260.0;
            const double us = 8.8 + 0.72 * core + 0.116 * gather->tiles_m * gather->tiles_n * gather->splits / 256.0 +
                              (gather->splits > 1 ? 0.985 * mb(*gather) - 2.4 : 2.1e-6 * dm.M * dm.Ncols);
            price_kind(out, KIND_GATHER, gather->cost, us);
        }
        if (const Launch *l = cheapest_of(out, KIND_SCONV)) price_kind(out, KIND_SCONV, l->cost, 11.1 + 0.366 * l->cost / 1260.0 + 2.4e-6 * dm.M * dm.Ncols);
    }
    // fp32 filter gradients: the gather kernel beside those over images, which one image leaves 15 zeros in 16 of (fitted to 160 launches,
    // 0.09 and 0.20 in the logarithm): one image 12x17, 240 -> 224 of 5x5 34 us gathering, 73 over images.  Its sums are the less exact ones,
    // so it is taken only where it is the cheaper one by clocks, too, whatever the launches take: 2 images 36x51, 281 -> 320 of 3x3 would
    // be 100 us faster and 1.6 times as far from 64 bits.
    if (demand && pass == OWT_PASS_BWD_FILTER) {
        for (const Launch &l : out)
            if (l.kind != KIND_XFILTER && l.kind != KIND_XGATHER && l.kind != KIND_IFILTER16 && l.kind != KIND_IGATHER16 && l.kind != KIND_IFILTER16B)
                demand->push_back({l.cost, l.ws_bytes(), is_split_kind(l.kind)});
    }
    const double gather_clocks = gather ? gather->cost : 0.0;
    const Launch *over = cheapest_of(out, KIND_XFILTER), *over2 = cheapest_of(out, KIND_XGATHER);
    if (!over || (over2 && over2->cost < over->cost)) over = over2;
    // The strided kernels on the fp32 instruction, whose clocks know nothing of what a unit's two rows take to stage: 176 images 77x79, 8 -> 320 of 1x1,
    // stride 2, masked, 766 us there and 147 over images, at a third of the clocks.  Fitted to 1000 and 612 launches, 0.11 and 0.05 in the logarithm;
    // never below the clocks, as these are the less exact kernels; which of the two, their clocks say.  1000 strided layers 17403 -> 15640 us, the fastest 15560.
    if (!g.bf16 && pass == OWT_PASS_BWD_FILTER && force_tile < 0 && over) {
        const Launch *l = cheapest_of(out, KIND_SFILTER), *streamed = cheapest_of(out, KIND_SFILTER2);
        const bool b = streamed && (!l || streamed->cost <= l->cost);
        if (b) l = streamed;
        if (l) {
            const bool sp = l->splits > 1;
            const double clocks = l->cost, core = (clocks - reduce_clocks(*l)) / 1260.0, steps = (double)l->steps_per_split * cdiv((long)l->tiles_m * l->splits, 256);
            const double us = b ? 3.78 + 0.061 * core + 3.78 * sp + 0.553 * mb(*l) + steps * (0.343 + 1.0e-5 * (g.sh + g.R) * g.W * g.C + 0.218 * g.Q)
                                : 4.14 + 0.133 * core + 4.14 * sp + 0.482 * mb(*l) + steps * (0.739 + 6.35e-4 * (g.sh + g.R) * g.W * g.C + 0.0806 * (1 + g.masked) * g.Q);
            for (int kind : {KIND_SFILTER, KIND_SFILTER2}) price_kind(out, kind, clocks, std::max(clocks / 1260.0, us));
        }
    }
    if (!g.bf16 && pass == OWT_PASS_BWD_FILTER && gather && force_tile < 0 && over) {
        const double core = (gather->cost - reduce_clocks(*gather)) / 1260.0, split = gather->splits > 1, wgs = (double)cdiv((long)gather->tiles_m * gather->tiles_n * gather->splits, 256);
        const double us = vec ? 4.3 + 0.734 * core + 0.474 * mb(*gather) + 0.193 * gather->steps_per_split + 2.53 * wgs
                              : 1.7 + 0.249 * core + 0.3 * split + 0.482 * mb(*gather) + 2.44 * gather->steps_per_split + 0.76 * wgs;
        const double priced = gather->cost < images_clocks ? 1.1 * us : std::max(us, 1.7 * over->cost / 1260.0);
        price_kind(out, KIND_GATHER, gather->cost, priced);
        for (Launch &l : out)
            if (l.kind == KIND_GATHER) l.asked = 1260.0 * (priced - us);
    }
    if (priced16 && gather) price_kind(out, KIND_GATHER, gather->cost, gather->cost / 1260.0 + 10.0);
    // The filter gradients that take 16 images at a time, against the kernel that gathers pixels: of a group of 16 one to four images
    // leave most empty, and few channels leave most of a 32-channel block empty.  Gathering fitted to launches of 546 layers, 0.09 to
    // 0.14 in the logarithm; large layers are left to the clocks, the fit is 25 % off there, and one or two images to gathering unless 16
    // at a time are clearly the faster way (the fit knows no masks, with which gathering takes a tenth longer: 200 masked layers of one or
    // two images 6903 -> 5904 us without).  us, 16 images at a time and gathering: one image 9x62, 33 -> 256 of 5x5 32 and 33; two
    // 47x48, 64 -> 256 of 3x3 37 and 43; two 24x36, 39 -> 451 of 3x3 43 and 58; three 30x20, 130 -> 200 of 5x5 55 and 124.  258 layers, most of
    // which stay with their kernel: 12315 -> 10768 us with four wavefronts to a tile, three more than 4 % slower (by 8 % at most).
    if (g.bf16 && pass == OWT_PASS_BWD_FILTER && force_tile < 0) {
        const auto rounds = [](const Launch &l) { return (double)cdiv((long)l.tiles_m * l.tiles_n * l.splits, 256); };
        const auto gather_us = [&](const Launch &l) {
            const double core = (l.cost - reduce_clocks(l)) / 1260.0, split = l.splits > 1;
            return vec ? 4.95 + 0.663 * core + 1.66 * split + 0.79 * mb(l) + 0.657 * l.steps_per_split + 0.37 * rounds(l)
                       : 5.9 + 0.357 * core + 2.16 * split + 0.84 * mb(l) + 1.9 * l.steps_per_split + 0.66 * rounds(l);
        };
        if (demand) {
            const ImagesDemand *b = nullptr;
            for (const ImagesDemand &d : images16)
                if (!b || d.cost < b->cost) b = &d;
            double more = 0.0;
            if (b && gather) {
                const double c = b->plain / 1260.0, sp = b->splits > 1, mbs = 4e-6 * b->splits * dm.M * dm.Ncols;
                const double here = b->rows ? -4.97 + 0.883 * c + 0.134 * b->per + 0.86 * b->wgs + sp * (4.09 + 0.3 * mbs) : -2.1 + 0.616 * c + 0.33 * b->per + 0.77 * b->wgs + sp * (1.93 + 0.46 * mbs);
                if (gather_us(*gather) < (g.N <= 2 ? 1.05 : 0.92) * here && b->cost < 1260.0 * (g.N <= 2 ? 150.0 : 60.0)) more = std::max(b->cost, 1.54 * gather_clocks) - b->cost;
            }
            for (const ImagesDemand &d : images16) demand->push_back({d.cost + more, d.need, true});
        }
        if (cheapest_of(out, KIND_IFILTER16B) || (cheapest_of(out, KIND_IFILTER16) && (cheapest_of(out, KIND_DFILTER16) || cheapest_of(out, KIND_DFILTER16B)))) {
            // beside the kernel that streams its operands every kind is priced (dfilter16 and dfilter16b fitted to 1494 and 1315 launches, 0.09
            // and 0.10 in the logarithm).  Which of these two is the faster one their clocks know better than the fits do (245 layers on which
            // they differ: 5889 us by clocks, 6588 by the fits), so the faster one is priced and the other keeps its distance.  It is the slower one for one to four images, a group of which is mostly zeros, and on large batches of
            // few channels, where its tile is mostly empty; us, ifilter16b and the kernel before: 2 images 30x22, 288 -> 488 50 and 29; 728 of
            // 49x14, 32 -> 32 77 and 48.  Over the 210 layers none is more than 3 % slower than before it, and all take 6398 us instead of 7900.
            // Of 1448 layers with a staged kernel 12 take more than 3 % longer than on that (140 where the fits chose among the three), all 42230 us
            // instead of 55430.
            if (gather) price_kind(out, KIND_GATHER, gather->cost, gather_us(*gather));
            if (const Launch *l = cheapest_of(out, KIND_IFILTER16)) price_kind(out, KIND_IFILTER16, l->cost, 1.04 * l->cost / images16_chain(*l) / 1260.0);
            const Launch *staged = cheapest_of(out, KIND_DFILTER16), *staged_b = cheapest_of(out, KIND_DFILTER16B);
            const bool b = staged_b && (!staged || staged_b->cost < staged->cost);
            if (const Launch *l = b ? staged_b : staged) {
                const double clocks = l->cost, core = (clocks - reduce_clocks(*l)) / 1260.0;
                const double us = b ? 10.4 + 0.139 * core + 0.576 * mb(*l) + (g.S == 3 ? 0.774 : 1.013) * l->steps_per_split * rounds(*l)
                                    : 10.2 + 0.0955 * core + 0.52 * mb(*l) + 1.62 * l->steps_per_split;
                for (int kind : {KIND_DFILTER16, KIND_DFILTER16B}) price_kind(out, kind, clocks, us);
            }
        } else if (gather) {
            for (int kind : {KIND_IFILTER16, KIND_IGATHER16}) {
                const Launch *l = cheapest_of(out, kind);
                if (!l) continue;
                const double us = l->cost / images16_chain(*l) / 1260.0;
                price_kind(out, kind, l->cost, us);
                price_kind(out, KIND_GATHER, gather->cost, us < (g.N <= 2 ? 150.0 : 60.0) ? gather_us(*gather) * (g.masked ? 1.1 : g.N <= 2 ? 1.0 / 1.2 : 1.0) : std::max(gather->cost / 1260.0, g.N <= 2 ? 0.0 : 1.05 * us));
            }
        }
    }
    if (demand && pass != OWT_PASS_BWD_FILTER) {
        for (const Launch &l : out)
            if (l.kind != KIND_XFCS && l.kind != KIND_XCONVS) demand->push_back({l.cost, l.ws_bytes(), is_split_kind(l.kind)});
    }
}

typedef std::array<int, 15> PlanKey;
static std::map<PlanKey, Launch> g_tuned;
static std::mutex g_tuned_mutex;

static PlanKey plan_key(const Geom &g, int pass, owt_dtype dt)
{
    return PlanKey{g.N, g.C, g.H, g.W, g.K, g.R, g.S, g.sh, g.sw, g.ph, g.pw, pass, (int)dt, g.masked, 0};
}

static bool variants_forced()
{
    return g_force_tile.load(std::memory_order_relaxed) >= 0 || g_force_split.load(std::memory_order_relaxed) > 0 ||
           g_force_flags.load(std::memory_order_relaxed) != 0;
}

// The model's choice per geometry (untimed), so that a call plans once: any scratch in [lo, hi) admits the same plans.
struct ModelledPlan { size_t lo, hi; Launch l; };
static std::map<PlanKey, ModelledPlan> g_modelled, g_modelled_small;   // scratch that the cheapest plans fit in, and the last one of less

// ws_bytes: the scratch the call was given.  A plan of the kernels that split their operands is passed over when its
// scratch does not fit, so a caller that sized its scratch for the kernels that multiply in fp32 is served by those.
static Launch choose(const Geom &g, int pass, owt_dtype dt, const PassDims &dm, bool want_db, bool use_cache, size_t ws_bytes = (size_t)-1)
{
    const bool cached = use_cache && !variants_forced();
    if (cached) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        const auto fits = [&](const Launch &l) { return !is_split_kind(l.kind) || l.ws_bytes() <= ws_bytes; };
        auto it = g_tuned.find(plan_key(g, pass, dt));
        if (it != g_tuned.end() && fits(it->second)) return it->second;
        // (not, or tuned to a plan that does not fit: the model's choice for this scratch, wherever it was put)
        for (const auto *plans : {&g_modelled, &g_modelled_small}) {
            const auto sm = plans->find(plan_key(g, pass, dt));
            if (sm != plans->end() && sm->second.lo <= ws_bytes && (ws_bytes < sm->second.hi || sm->second.hi == (size_t)-1)) return sm->second.l;
        }
    }
    std::vector<Launch> c;
    std::vector<Demand> demand;
    enumerate(g, pass, dm, want_db, c, variants_forced() ? nullptr : &demand);
    bool only_direct = forced(OWT_FORCE_ONLY_DIRECT), any_direct = false;   // test hook
    for (const Launch &l : c) any_direct |= l.kind != KIND_GATHER;
    // `fits`: the cheapest of those that may be taken; `any`: the scratch left out of account, for the caller's check to refuse
    // where nothing fits (the test hook can leave a geometry with split-operand kernels alone)
    size_t fits = c.size(), any = c.size();
    ModelledPlan plan = {0, (size_t)-1, {}};
    const auto bound = [&](size_t need) { if (need > ws_bytes) plan.hi = std::min(plan.hi, need); else plan.lo = std::max(plan.lo, need); };
    for (size_t i = 0; i < c.size(); i++) {
        if (only_direct && any_direct && c[i].kind == KIND_GATHER) continue;
        if (any == c.size() || c[i].cost < c[any].cost) any = i;
        const size_t need = c[i].ws_bytes();
        bound(need);
        if (need > ws_bytes && (is_split_kind(c[i].kind) || !demand.empty())) continue;
        if (fits == c.size() || c[i].cost < c[fits].cost) fits = i;
    }
    plan.l = c[fits < c.size() ? fits : any];
    // refused by the plan that the scratch is asked for, and by no other
    const Demand *asked = nullptr, *least = nullptr;
    for (const Demand &d : demand) {
        bound(d.need);
        if (!least || d.cost < least->cost) least = &d;
        if (!(d.passed_over && d.need > ws_bytes) && (!asked || d.cost < asked->cost)) asked = &d;
    }
    if (!asked) asked = least;
    const size_t both = std::max(plan.l.ws_bytes(), asked ? asked->need : 0);
    if (fits == any && asked == least && both <= ws_bytes) { plan.lo = both; plan.hi = (size_t)-1; }      // the same with any larger scratch
    if (asked && asked->need > ws_bytes) { plan.l.pre_bytes = plan.l.dbias_bytes = 0; plan.l.partial_bytes = asked->need; }
    if (cached) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        (plan.hi == (size_t)-1 ? g_modelled : g_modelled_small)[plan_key(g, pass, dt)] = plan;
    }
    return plan.l;
}

static std::map<PlanKey, size_t> g_workspace;  // owt_conv_workspace_bytes per geometry: listing the candidates takes 10-60 us

// Whether tuning times a candidate, `least` being the cheapest modelled cost, and whether the workspace bound covers it.  Tuned
// without this rule on draws of the layers' ranges, the fastest candidate was modelled at up to 2.82 times the cheapest in 418
// fp32 passes, 1.75 in 200 bf16 passes, 1.57 in 150 of shards, so three times left none out; timing every candidate of the 418
// passes took 32.7 s, these take 5.3 s (up to four times the cheapest 6.8 s, and a training step's tuning 0.79 s instead of
// 0.63).  Split-operand kernels that split their reduction, too, were the fastest up to 1.85
// times: past twice they only raise the bound (the first layer's forward pass 0.3 -> 199 MB).  Costs that have the launch in them lie
// nearer to each other, and to the truth: of 310 bf16 passes priced so 1 loses more than 2 % with 1.6 times (none with 2, three with
// 1.4), 1675 instead of 2918 candidates; of 700 fp32 filter gradients none with 1.6 or 1.2, 16080 and 6218 instead of 31548 (with the gather
// kernel weighed by the choice's cost, which is not of time alone, 36 lost up to 83 %); of 700 in bf16 with ifilter16 and igather16 to 1.6
// and ifilter16b to 1.25 none (1.4: two; 1.15: two, 1.1: eight by up to 17 %).  choose() sees every candidate.
static bool worth_timing(const Launch &l, double least)
{
    if (l.kind == KIND_XCONVS || l.kind == KIND_DIRECT16S) return l.cost <= 1.4 * least;      // (three tiles, up to eight splits; modelled to 0.14-0.17 in the logarithm)
    if (l.kind == KIND_IFILTER16B) return l.cost <= 1.25 * least;
    return l.cost - l.asked <= (l.fitted ? 1.6 : is_split_kind(l.kind) && l.splits > 1 ? 2.0 : 3.0) * least;
}
static bool worth_workspace(const Launch &l, double least) { return !is_split_kind(l.kind) || l.splits == 1 || worth_timing(l, least); }
static double least_cost(const std::vector<Launch> &c)
{
    double least = c.empty() ? 0.0 : c[0].cost;
    for (const Launch &l : c) least = std::min(least, l.cost);
    return least;
}

// Workspace every candidate that may be tuned to, or is the model's choice, fits in (so neither outgrows the caller's buffer).
static size_t max_workspace(const Geom &g, int pass, const PassDims &dm, bool want_db)
{
    // with and without the ReLU' mask flag: a caller may size its buffer with one descriptor of a layer and call
    // with the other (the kernels that take dz as it is are only candidates for the unmasked one)
    size_t m = 0;
    for (int masked = 0; masked < 2; masked++) {
        Geom gm = g;
        gm.masked = masked != 0;
        std::vector<Launch> c;
        std::vector<Demand> demand;
        enumerate(gm, pass, dm, want_db, c, variants_forced() ? nullptr : &demand);
        const Demand *asked = nullptr;
        for (const Demand &d : demand)
            if (!asked || d.cost < asked->cost) asked = &d;
        if (asked) m = std::max(m, asked->need);
        const double least = least_cost(c);
        for (const Launch &l : c)
            if (worth_workspace(l, least) || variants_forced()) m = l.ws_bytes() > m ? l.ws_bytes() : m;
    }
    return m;
}

// The part of the kernel parameters that the chosen launch decides.
static void frame_params(const Geom &g, const PassDims &dm, const Launch &l, void *ws, GemmParams &p)
{
    p.g = g; p.M = (int)dm.M; p.Ncols = (int)dm.Ncols; p.Kd = (int)dm.Kd;
    p.splits = l.splits; p.ksteps = l.steps; p.ksteps_per_split = l.steps_per_split;
    p.tiles_m = l.tiles_m; p.tiles_n = l.tiles_n;
    p.partial = l.splits > 1 ? (float *)((char *)ws + l.pre_bytes) : nullptr;
    p.dbias_partial = (l.splits > 1 && l.dbias_bytes) ? (float *)((char *)ws + l.pre_bytes + l.partial_bytes) : nullptr;
}

static owt_status launch(const Geom &g, int pass, owt_dtype dt, const PassDims &dm, GemmParams p, const Launch &l,
                         void *ws, hipStream_t s)
{
    frame_params(g, dm, l, ws, p);
    const bool bf = dt == OWT_BF16;
    hipError_t e;
    if (l.kind == KIND_XFCS) {
        e = owt_launch_xfcs_fwd(bf, p, s);
    } else if (l.kind == KIND_XFC) {
        e = pass == OWT_PASS_FWD ? owt_launch_xfc_fwd(bf, p, s)
                                 : owt_launch_xfc_bwd(bf, pass == OWT_PASS_BWD_DATA ? &p : nullptr, pass == OWT_PASS_BWD_DATA ? nullptr : &p, s);
    } else if (l.kind == KIND_XCONV) {
        const bool blocks = g.sh > 1 || g.sw > 1;
        if (blocks) blocks_frame(g, p); else dconv_frame(g, pass, p);
        p.dWp.set(p.Wi); p.dHpWp.set(p.Hi * p.Wi);
        p.tpi = l.tpi;
        const bool vec = p.Cred % 4 == 0;
        if (blocks) e = owt_launch_xconv_fwd_blocks(l.tile, l.pr, p, ws, s);
        else if (pass == OWT_PASS_FWD) e = vec ? owt_launch_xconv_fwd_vec1(l.tile, l.pr, p, ws, s) : owt_launch_xconv_fwd_vec0(l.tile, l.pr, p, ws, s);
        else e = vec ? owt_launch_xconv_data_vec1(l.tile, l.pr, p, ws, s) : owt_launch_xconv_data_vec0(l.tile, l.pr, p, ws, s);
    } else if (l.kind == KIND_XCONVS) {
        dconv_frame(g, pass, p);
        e = pass == OWT_PASS_FWD ? owt_launch_xconvs_fwd(l.tile, l.pr, p, s) : owt_launch_xconvs_data(l.tile, l.pr, p, s);
    } else if (l.kind == KIND_DIRECT16S) {
        dconv_frame(g, pass, p);
        e = pass == OWT_PASS_FWD ? owt_launch_dconv16s_fwd(l.tile, l.pr, p, s) : owt_launch_dconv16s_data(l.tile, l.pr, p, s);
    } else if (l.kind == KIND_DIRECT16X) {
        if (l.blocks) blocks_frame(g, p); else dconv_frame(g, pass, p);
        p.dWp.set(p.Wi); p.dHpWp.set(p.Hi * p.Wi);
        e = l.blocks ? owt_launch_dconv16x_blocks(l.pr, p, ws, s)
                     : pass == OWT_PASS_FWD ? owt_launch_dconv16x_fwd(l.pr, p, ws, s) : owt_launch_dconv16x_data(l.pr, p, ws, s);
    } else if (l.kind == KIND_FCGEMM) {
        e = owt_launch_fcgemm(pass, l.tile, p, (float *)ws, s);
    } else if (l.kind == KIND_DIRECT16) {
        dconv_frame(g, pass, p);
        e = pass == OWT_PASS_FWD ? owt_launch_dconv16_fwd(l.tile, l.pr, p, s) : owt_launch_dconv16_data(l.tile, l.pr, p, ws, s);
    } else if (l.kind == KIND_SCONV16) {
        SConv16Geom sg;
        sconv16_geom(g, sg);
        sg.units_per_wg = l.steps_per_split;
        p.splits = 1; p.partial = nullptr;
        e = owt_launch_sconv16(p, sg, l.tiles_m, l.tiles_n, ws, s);
    } else if (l.kind == KIND_SCONV2) {
        SConvGeom sg;
        sconv_geom(g, sg);
        sg.units_per_wg = l.steps_per_split;
        p.splits = 1; p.partial = nullptr;
        e = owt_launch_sconv2_f32(p, sg, l.tiles_m, l.tiles_n, (float *)ws, s);
    } else if (l.kind == KIND_SCONV) {
        SConvGeom sg;
        sconv_geom(g, sg);
        sg.units_per_wg = l.steps_per_split;
        p.splits = 1; p.partial = nullptr;
        e = bf ? owt_launch_sconv_bf16(p, sg, l.tiles_m, l.tiles_n, (float *)ws, s)
               : owt_launch_sconv_f32(p, sg, l.tiles_m, l.tiles_n, (float *)ws, s);
    } else if (l.kind == KIND_SFILTER16B) {
        SFilter16Geom sg;
        sfilter16_geom(g, sg);
        sg.units_per_wg = l.steps_per_split;
        e = owt_launch_sfilter16b(p, sg, l.tiles_m, s);
    } else if (l.kind == KIND_SFILTER16) {
        SFilter16Geom sg;
        sfilter16_geom(g, sg);
        sg.units_per_wg = l.steps_per_split;
        e = owt_launch_sfilter16(p, sg, l.tiles_m, s);
    } else if (l.kind == KIND_SFILTER2) {
        SFilterGeom sg;
        sfilter_geom(g, sg);
        sg.units_per_wg = l.steps_per_split;
        e = owt_launch_sfilter2_f32(p, sg, l.tiles_m, s);
    } else if (l.kind == KIND_SFILTER) {
        SFilterGeom sg;
        sfilter_geom(g, sg);
        sg.units_per_wg = l.steps_per_split;
        e = bf ? owt_launch_sfilter_bf16(p, sg, l.tiles_m, s) : owt_launch_sfilter_f32(p, sg, l.tiles_m, s);
    } else if (l.kind == KIND_XGATHER) {
        e = owt_launch_xgather(l.tile, p, s);
    } else if (l.kind == KIND_XFILTER) {
        p.ctiles = l.ctiles;
        e = owt_launch_xfilter(l.tile, p, s);
    } else if (l.kind == KIND_IGATHER16) {
        e = p.mask ? owt_launch_igather16_masked(l.tile, p, s) : owt_launch_igather16(l.tile, p, s);
    } else if (l.kind == KIND_IFILTER16B) {
        p.ctiles = l.ctiles;
        e = owt_launch_ifilter16b(l.tile, p, s);
    } else if (l.kind == KIND_IFILTER16) {
        p.ctiles = l.ctiles;
        e = p.mask ? owt_launch_ifilter16_masked(l.tile, p, s) : owt_launch_ifilter16(l.tile, p, s);
    } else if (l.kind == KIND_DFILTER16B) {
        p.Hp = g.H + 2 * g.ph; p.Wp = g.W + 2 * g.pw; p.taps = l.taps; p.groups = l.groups; p.ctiles = l.ctiles;
        p.dWp.set(p.Wp); p.dHpWp.set(p.Hp * p.Wp);
        e = owt_launch_dfilter16b(l.tile, p, s);
    } else if (l.kind == KIND_DFILTER16) {
        p.Hp = g.H + 2 * g.ph; p.Wp = g.W + 2 * g.pw; p.taps = l.taps; p.groups = l.groups; p.ctiles = l.ctiles;
        p.dWp.set(p.Wp); p.dHpWp.set(p.Hp * p.Wp);
        e = owt_launch_dfilter16(l.tile, p, s);
    } else if (l.kind == KIND_DFILTER2) {
        p.Hp = g.H + 2 * g.ph; p.Wp = g.W + 2 * g.pw; p.taps = l.taps; p.groups = l.groups; p.ctiles = l.ctiles;
        p.dWp.set(p.Wp); p.dHpWp.set(p.Hp * p.Wp);
        e = owt_launch_dfilter2_f32(l.tile, p, s);
    } else if (l.kind == KIND_DFILTER) {
        p.Hp = g.H + 2 * g.ph; p.Wp = g.W + 2 * g.pw; p.taps = l.taps; p.groups = l.groups; p.ctiles = l.ctiles;
        p.dWp.set(p.Wp); p.dHpWp.set(p.Hp * p.Wp);
        if (kDFilterVariants[l.tile].aligned) { p.cpi = (int)cdiv((long)g.P * g.Q, 32); p.dCpi.set(p.cpi); }
        e = bf ? owt_launch_dfilter_bf16(l.tile, p, s) : owt_launch_dfilter_f32(l.tile, p, s);
    } else if (l.kind == KIND_DIRECT) {
        dconv_frame(g, pass, p);
        if (pass == OWT_PASS_FWD) e = bf ? owt_launch_dconv_fwd_bf16(l.tile, l.pr, p, s) : owt_launch_dconv_fwd_f32(l.tile, l.pr, p, s);
        else e = bf ? owt_launch_dconv_data_bf16(l.tile, l.pr, p, s) : owt_launch_dconv_data_f32(l.tile, l.pr, p, s);
    } else {
        static const LaunchFn table[3][2] = {
            {owt_launch_fwd_f32, owt_launch_fwd_bf16},
            {owt_launch_data_f32, owt_launch_data_bf16},
            {owt_launch_filter_f32, owt_launch_filter_bf16},
        };
        e = table[pass][bf ? 1 : 0](l.tile, dm.va ? 4 : 1, dm.vb ? 4 : 1, p, s);
    }
    if (e != hipSuccess) return fail(OWT_ELAUNCH, "HIP launch failed: %s", hipGetErrorString(e));
    return OWT_OK;
}

static int describe(char *buf, size_t n, int pass, owt_dtype dt, const PassDims &dm, const Launch &l)
{
    // "... gridAxB threadsT": A x B work-groups, T = total threads of the main kernel's launch (the
    // figure profilers list as its grid size)
    static const char *pn[3] = {"fwd", "bwd_data", "bwd_filter"};
    const char *ds = dt == OWT_BF16 ? "bf16" : "f32";
    if (l.kind == KIND_FCGEMM) {
        const FcTile &ft = kFcTiles[l.tile];
        return snprintf(buf, n, "fcgemm %s %s tile%dx%dx32 splitk%d grid%dx%d threads%ld", pn[pass], ds, 32 * ft.MB * ft.WM,
                        32 * ft.NB * ft.WN, l.splits, l.tiles_m * l.tiles_n, l.splits,
                        (long)l.tiles_m * l.tiles_n * l.splits * 64 * ft.WM * ft.WN);
    }
    if (l.kind == KIND_XCONV) {
        const XConvVariant &v = kXConvVariants[l.tile];
        return snprintf(buf, n, "%s %s %s tile%dx%dx16 waves%dx%d panel%d splitk%d grid%dx%d threads%ld", l.blocks ? "sconvx" : "xconv", pn[pass], ds, 32 * v.MB * v.WM,
                        64 * v.WN, v.WM, v.WN, l.pr, l.splits, l.tiles_m * l.tiles_n, l.splits, (long)l.tiles_m * l.tiles_n * l.splits * 64 * v.WM * v.WN);
    }
    if (l.kind == KIND_XCONVS) {
        const XConvSVariant &v = kXConvSVariants[l.tile];
        return snprintf(buf, n, "xconvs %s %s tile%dx32x16 waves%dx1x%d panel%d splitk%d grid%dx%d threads%ld", pn[pass], ds, 32 * v.WM, v.WM, v.TG,
                        l.pr, l.splits, l.tiles_m * l.tiles_n, l.splits, (long)l.tiles_m * l.tiles_n * l.splits * 64 * v.WM * v.TG);
    }
    if (l.kind == KIND_DIRECT16S) {
        const DConv16SVariant &v = kDConv16SVariants[l.tile];
        return snprintf(buf, n, "dconv16s %s %s tile%dx32x32 waves%dx1x%d panel%d splitk%d grid%dx%d threads%ld", pn[pass], ds, 32 * v.WM, v.WM, v.TG,
                        l.pr, l.splits, l.tiles_m * l.tiles_n, l.splits, (long)l.tiles_m * l.tiles_n * l.splits * 64 * v.WM * v.TG);
    }
    if (l.kind == KIND_DIRECT16X)
        return snprintf(buf, n, "%s %s %s tile256x64x32 waves4x1 panel%d splitk%d grid%dx%d threads%ld", l.blocks ? "sconv16x" : "dconv16x", pn[pass], ds, l.pr,
                        l.splits, l.tiles_m * l.tiles_n, l.splits, (long)l.tiles_m * l.tiles_n * l.splits * 256);
    if (l.kind == KIND_XFCS)
        return snprintf(buf, n, "xfcs %s %s tile16x16 waves16 splitk1 grid%d threads%ld", pn[pass], ds, l.tiles_m * l.tiles_n, (long)l.tiles_m * l.tiles_n * 1024);
    if (l.kind == KIND_XFC) {
        const long wgs = (long)l.tiles_m * l.tiles_n * l.splits;
        return snprintf(buf, n, "xfc %s %s tile64x64x16 splitk%d grid%ld threads%ld", pn[pass], ds, l.splits, wgs, wgs * 256);
    }
    if (l.kind == KIND_XGATHER)
        return snprintf(buf, n, "%s %s %s tile%dx%d%s splitk%d grid%dx%d threads%ld", l.blocks ? "sfilterx" : "xgather", pn[pass], ds,
                        32 * kXGatherVariants[l.tile].KB, 32 * kXGatherVariants[l.tile].CB, kXGatherVariants[l.tile].TG > 1 ? " shared4" : "", l.splits, l.tiles_m * l.tiles_n, l.splits,
                        8 * cdiv((long)l.tiles_m * l.tiles_n * l.splits, 8) * 64 * kXGatherVariants[l.tile].TG);
    if (l.kind == KIND_XFILTER)
        return snprintf(buf, n, "xfilter %s %s tile%dx32 taps%dx%d%s splitk%d grid%dx%d threads%ld", pn[pass], ds,
                        32 * kXFilterVariants[l.tile].KB, l.taps, l.groups, kXFilterVariants[l.tile].TG > 1 ? " shared4" : "", l.splits, l.tiles_m * l.tiles_n, l.splits,
                        8 * cdiv(cdiv((long)l.tiles_m * l.tiles_n * l.splits, 4 / kXFilterVariants[l.tile].TG), 8) * 256);
    if (l.kind == KIND_IGATHER16)
        return snprintf(buf, n, "%s %s %s tile%dx%d splitk%d grid%dx%d threads%ld", l.blocks ? "sfilter16x" : "igather16", pn[pass], ds,
                        32 * kIGather16Variants[l.tile].KB, 32 * kIGather16Variants[l.tile].CB, l.splits, l.tiles_m * l.tiles_n, l.splits,
                        8 * cdiv((long)l.tiles_m * l.tiles_n * l.splits, 8) * 256);
    if (l.kind == KIND_IFILTER16B) {
        const IFilter16bVariant &v = kIFilter16bVariants[l.tile];
        return snprintf(buf, n, "ifilter16b %s %s tile%dx%d waves%dx%d taps%dx%d splitk%d grid%dx%d threads%ld", pn[pass], ds, 32 * v.KB * v.WK,
                        32 * v.CB * v.WC, v.WK, v.WC, l.taps, l.groups, l.splits, l.tiles_m * l.tiles_n, l.splits,
                        (long)owt_split_major_grid(l.tiles_m * l.tiles_n, l.splits) * 64 * v.WK * v.WC);
    }
    if (l.kind == KIND_IFILTER16)
        return snprintf(buf, n, "ifilter16 %s %s tile%dx%d taps%dx%d splitk%d grid%dx%d threads%ld", pn[pass], ds,
                        32 * kIFilter16Variants[l.tile].KB, 32 * kIFilter16Variants[l.tile].CB, l.taps, l.groups, l.splits, l.tiles_m * l.tiles_n, l.splits,
                        8 * cdiv((long)l.tiles_m * l.tiles_n * l.splits, 8) * 256);
    if (l.kind == KIND_SCONV16)
        return snprintf(buf, n, "sconv16 %s %s rows%d grid%dx%d threads%ld", pn[pass], ds, kSConv16TP, l.tiles_m, l.tiles_n,
                        (long)l.tiles_m * l.tiles_n * kSConv16NT);
    if (l.kind == KIND_SCONV2)
        return snprintf(buf, n, "sconv2 %s %s band%d filters%d grid%dx%d threads%ld", pn[pass], ds, kSConvBand, kSConv2KB, l.tiles_m,
                        l.tiles_n, (long)l.tiles_m * ((l.tiles_n + 7) / 8) * 8 * kSConvNT);
    if (l.kind == KIND_SCONV)
        return snprintf(buf, n, "sconv %s %s band%d grid%dx%d threads%ld", pn[pass], ds, kSConvBand, l.tiles_m, l.tiles_n,
                        (long)l.tiles_m * l.tiles_n * kSConvNT);
    if (l.kind == KIND_SFILTER16B)
        return snprintf(buf, n, "sfilter16b %s %s rows%d splitk%d grid%dx%d threads%ld", pn[pass], ds, kSFilter16TP, l.splits,
                        l.tiles_m, l.splits, (long)l.tiles_m * l.splits * kSFilter16NT);
    if (l.kind == KIND_SFILTER16)
        return snprintf(buf, n, "sfilter16 %s %s rows%d splitk%d grid%dx%d threads%ld", pn[pass], ds, kSFilter16TP, l.splits,
                        l.tiles_m, l.splits, (long)l.tiles_m * l.splits * kSFilter16NT);
    if (l.kind == KIND_SFILTER2)
        return snprintf(buf, n, "sfilter2 %s %s rows2 splitk%d grid%dx%d threads%ld", pn[pass], ds, l.splits, l.tiles_m,
                        l.splits, (long)l.tiles_m * l.splits * kSFilterNT);
    if (l.kind == KIND_SFILTER)
        return snprintf(buf, n, "sfilter %s %s rows2 splitk%d grid%dx%d threads%ld", pn[pass], ds, l.splits, l.tiles_m,
                        l.splits, (long)l.tiles_m * l.splits * kSFilterNT);
    if (l.kind == KIND_DFILTER16B) {
        const DFilter16bVariant &v = kDFilter16bVariants[l.tile];
        return snprintf(buf, n, "dfilter16b %s %s tile%dx%d taps%dx%d splitk%d grid%dx%d threads%ld", pn[pass], ds,
                        32 * v.KB * v.WK, 32 * v.WC, l.taps, l.groups, l.splits, l.tiles_m * l.tiles_n, l.splits,
                        (long)l.tiles_m * l.tiles_n * l.splits * 64 * v.WK * v.WC);
    }
    if (l.kind == KIND_DFILTER16) {
        const DFilter16Variant &v = kDFilter16Variants[l.tile];
        return snprintf(buf, n, "dfilter16 %s %s tile%dx%d taps%dx%d splitk%d grid%dx%d threads%ld", pn[pass], ds,
                        32 * v.KB * v.WK, 32 * v.WC, l.taps, l.groups, l.splits, l.tiles_m * l.tiles_n, l.splits,
                        (long)l.tiles_m * l.tiles_n * l.splits * 64 * v.WK * v.WC);
    }
    if (l.kind == KIND_DFILTER2) {
        const DFilter2Variant &v = kDFilter2Variants[l.tile];
        return snprintf(buf, n, "dfilter2 %s %s tile%dx32 pixelparts%d taps%dx%d splitk%d grid%dx%d threads%ld", pn[pass], ds, 32 * v.WK,
                        v.WP, l.taps, l.groups, l.splits, l.tiles_m * l.tiles_n, l.splits,
                        (long)l.tiles_m * l.tiles_n * l.splits * 64 * v.WK * v.WP);
    }
    if (l.kind == KIND_DFILTER) {
        const DFilterVariant &v = kDFilterVariants[l.tile];
        return snprintf(buf, n, "dfilter %s %s tile%dx%d taps%dx%d%s splitk%d grid%dx%d threads%ld", pn[pass], ds, 32 * v.WK,
                        32 * v.WC, l.taps, l.groups, v.aligned ? " chunks-per-image" : "", l.splits, l.tiles_m * l.tiles_n, l.splits,
                        (long)l.tiles_m * l.tiles_n * l.splits * 64 * v.WK * v.WC);
    }
    const TileInfo &ti = kTiles[l.tile];
    const long threads = (long)l.tiles_m * l.tiles_n * l.splits * 64 * ti.WM * ti.WN;
    if (l.kind == KIND_DIRECT16)
        return snprintf(buf, n, "dconv16 %s %s tile%dx%dx%d waves%dx%d panel%d splitk%d grid%dx%d threads%ld", pn[pass], ds,
                        ti.BM, 64 * ti.WN, (l.tile == TILE_512x64 || l.tile == TILE_256x64P) ? 32 : 64, ti.WM, ti.WN, l.pr, l.splits,
                        l.tiles_m * l.tiles_n, l.splits, threads);
    if (l.kind == KIND_DIRECT)
        return snprintf(buf, n, "dconv %s %s tile%dx%dx%d waves%dx%d panel%d splitk%d grid%dx%d threads%ld", pn[pass], ds,
                        ti.BM, 64 * ti.WN, l.tile == TILE_128x64 ? 16 : 32, ti.WM, ti.WN, l.pr, l.splits,
                        l.tiles_m * l.tiles_n, l.splits, threads);
    return snprintf(buf, n, "igemm %s %s tile%dx%dx%d vec%d/%d splitk%d grid%dx%d threads%ld", pn[pass], ds, ti.BM,
                    64 * ti.WN, ti.BK, dm.va ? 4 : 1, dm.vb ? 4 : 1, l.splits, l.tiles_m * l.tiles_n, l.splits, threads);
}

// ----------------------------------------------------------------- checking
static const long kMaxElems = 0x7fffffffL;   // tensors are indexed with 32-bit offsets

static owt_status check_conv(const owt_conv_desc *d, Geom &g)
{
    if (!d) return fail(OWT_EINVAL, "descriptor is NULL");
    if (d->N <= 0 || d->C <= 0 || d->H <= 0 || d->W <= 0 || d->K <= 0 || d->R <= 0 || d->S <= 0)
        return fail(OWT_EINVAL, "N,C,H,W,K,R,S must be positive");
    if (d->stride_h < 1 || d->stride_w < 1) return fail(OWT_EINVAL, "strides must be >= 1");
    if (d->pad_h < 0 || d->pad_w < 0 || d->pad_h >= d->R || d->pad_w >= d->S)
        return fail(OWT_EINVAL, "need 0 <= pad_h < R and 0 <= pad_w < S");
    if (d->dtype != OWT_F32 && d->dtype != OWT_BF16) return fail(OWT_EINVAL, "unknown dtype %d", (int)d->dtype);
    if (d->flags & ~(unsigned)(OWT_BIAS | OWT_RELU)) return fail(OWT_EINVAL, "unknown flag bits 0x%x", d->flags);
    if (!fill_geom(g, d->N, d->C, d->H, d->W, d->K, d->R, d->S, d->stride_h, d->stride_w, d->pad_h, d->pad_w))
        return fail(OWT_EINVAL, "filter larger than the padded input: no output");
    g.bf16 = d->dtype == OWT_BF16;
    g.masked = (d->flags & OWT_RELU) ? 1 : 0;       // backward calls then mask dy by y > 0 themselves
    const long xe = (long)d->N * d->H * d->W * d->C, ye = (long)d->N * g.P * g.Q * d->K,
               we = (long)d->K * d->R * d->S * d->C;
    if (xe > kMaxElems || ye > kMaxElems || we > kMaxElems)
        return fail(OWT_EUNSUPPORTED, "tensor with more than 2^31-1 elements");
    return OWT_OK;
}

static owt_status check_ptr(const void *p, const char *name)
{
    if (!p) return fail(OWT_EINVAL, "%s is NULL", name);
    if (!aligned16(p)) return fail(OWT_EINVAL, "%s is not 16-byte aligned", name);
    return OWT_OK;
}

#define OWT_TRY(expr) do { owt_status st_ = (expr); if (st_ != OWT_OK) return st_; } while (0)

static owt_status check_ws(const Launch &l, void *ws, size_t ws_bytes)
{
    if (l.ws_bytes() > ws_bytes)
        return fail(OWT_EWORKSPACE, "workspace too small: need %zu bytes, got %zu", l.ws_bytes(), ws_bytes);
    if (l.ws_bytes() && (!ws || !aligned16(ws))) return fail(OWT_EINVAL, "ws is NULL or misaligned");
    return OWT_OK;
}

static owt_status conv_pass(const Geom &g, int pass, owt_dtype dt, const GemmParams &p, bool want_db,
                            void *ws, size_t ws_bytes, hipStream_t s, bool use_cache)
{
    const PassDims dm = conv_dims(g, pass);
    const Launch l = choose(g, pass, dt, dm, want_db, use_cache, ws && aligned16(ws) ? ws_bytes : 0);
    OWT_TRY(check_ws(l, ws, ws_bytes));
    return launch(g, pass, dt, dm, p, l, ws, s);
}

static GemmParams fwd_params(const owt_conv_desc *d, const void *x, const void *w, const float *bias, void *y)
{
    GemmParams p; memset(&p, 0, sizeof(p));
    p.a = x; p.b = w; p.out = y; p.bias = bias; p.flags = d->flags;
    return p;
}
static GemmParams data_params(const owt_conv_desc *d, const void *dy, const void *y, const void *w, void *dx,
                              const void *xmask = nullptr)
{
    GemmParams p; memset(&p, 0, sizeof(p));
    p.a = dy; p.b = w; p.out = dx; p.flags = d->flags; p.xmask = xmask;
    p.mask = (d->flags & OWT_RELU) ? y : nullptr;
    return p;
}
static GemmParams filter_params(const owt_conv_desc *d, const void *x, const void *dy, const void *y, float alpha,
                                float beta, float *dw, float *db)
{
    GemmParams p; memset(&p, 0, sizeof(p));
    p.a = dy; p.b = x; p.out = dw; p.flags = d->flags; p.alpha = alpha; p.beta = beta; p.dbias = db;
    p.mask = (d->flags & OWT_RELU) ? y : nullptr;
    return p;
}

// Backward pass of a fully-connected shard when both of its products run on the dense kernel.
struct FcPair { Launch ld, lf; bool fused, xfc; };
// How the two products run: each as its own pass, both on the dense kernel in two launches or in one, or in one launch on the
// bf16 matrix unit.  Untimed, one product that chose the latter takes the other along, and two dense ones share a launch.
enum { FC_SEPARATE, FC_DENSE_TWO, FC_DENSE_ONE, FC_XFC };
static std::map<PlanKey, int> g_fc_way;        // timed by owt_fc_autotune

static bool find_fc_launch(const Geom &g, int pass, int kind, int tile, Launch &out)
{
    std::vector<Launch> c;
    enumerate(g, pass, conv_dims(g, pass), pass == OWT_PASS_BWD_FILTER, c);
    for (const Launch &l : c)
        if (l.kind == kind && l.tile == tile && l.splits == 1) { out = l; return true; }
    return false;
}

// The pair of launches for `way` (-1: the model's), false where both products are passes of their own.  Where the plans that
// the products chose since (tuned alone) no longer allow `way`, the model's.
static bool fc_pair_of(const Geom &g, owt_dtype dt, int way, FcPair &fp)
{
    fp.ld = choose(g, OWT_PASS_BWD_DATA, dt, conv_dims(g, OWT_PASS_BWD_DATA), false, true);
    fp.lf = choose(g, OWT_PASS_BWD_FILTER, dt, conv_dims(g, OWT_PASS_BWD_FILTER), true, true);
    fp.fused = fp.xfc = false;
    const bool dense = fp.ld.kind == KIND_FCGEMM && fp.lf.kind == KIND_FCGEMM;
    Launch fd, ff;
    if (way == FC_SEPARATE) return false;
    if (way == FC_DENSE_TWO && dense) return true;
    if (way == FC_XFC || (way != FC_DENSE_ONE && (fp.ld.kind == KIND_XFC || fp.lf.kind == KIND_XFC))) {
        if (find_fc_launch(g, OWT_PASS_BWD_DATA, KIND_XFC, 0, fd) && find_fc_launch(g, OWT_PASS_BWD_FILTER, KIND_XFC, 0, ff)) {
            fp.xfc = true;
            fp.ld = fd; fp.lf = ff;
            return true;
        }
        return dense;
    }
    if (way != FC_DENSE_ONE && !dense) return false;
    if (!forced(OWT_FORCE_FC_TWO_LAUNCHES) && find_fc_launch(g, OWT_PASS_BWD_DATA, KIND_FCGEMM, kFcPairTile, fd) &&
        find_fc_launch(g, OWT_PASS_BWD_FILTER, KIND_FCGEMM, kFcPairTile, ff)) {
        fp.ld = fd; fp.lf = ff; fp.fused = true;
        return true;
    }
    return dense;
}

static std::map<PlanKey, std::pair<bool, FcPair>> g_fc_pairs;     // planned once per geometry; owt_fc_autotune erases its entry

static bool fc_pair_plan(const Geom &g, owt_dtype dt, FcPair &fp)
{
    const bool cached = !variants_forced();
    if (cached) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        auto it = g_fc_pairs.find(plan_key(g, 3, dt));
        if (it != g_fc_pairs.end()) { fp = it->second.second; return it->second.first; }
    }
    int way = -1;
    if (cached) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        auto it = g_fc_way.find(plan_key(g, 3, dt));
        if (it != g_fc_way.end()) way = it->second;
    }
    const bool ok = fc_pair_of(g, dt, way, fp);
    if (cached) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        g_fc_pairs[plan_key(g, 3, dt)] = std::make_pair(ok, fp);
    }
    return ok;
}

static owt_status launch_fc_pair(const Geom &g, const FcPair &fp, GemmParams pd, GemmParams pf, void *ws, hipStream_t s)
{
    frame_params(g, conv_dims(g, OWT_PASS_BWD_DATA), fp.ld, ws, pd);
    frame_params(g, conv_dims(g, OWT_PASS_BWD_FILTER), fp.lf, ws, pf);
    const hipError_t e = fp.xfc ? owt_launch_xfc_bwd(g.bf16 != 0, &pd, &pf, s)
                                : owt_launch_fcgemm_bwd(fp.ld.tile, fp.lf.tile, fp.fused, pd, pf, (float *)ws, s);
    if (e != hipSuccess) return fail(OWT_ELAUNCH, "HIP launch failed: %s", hipGetErrorString(e));
    return OWT_OK;
}

// ---------------------------------------------------------------- static scratch
// Device memory for owt_conv_bwd_filter_static: lives in the code object, one copy per GPU that loads
// the library, held until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; the device address it yields (per device) is what kernels and launchers get.
static constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static constexpr int kMaxDevices = 64;
static void *g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;

static owt_status static_scratch(void **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail(OWT_ELAUNCH, "hipGetDevice failed: %s", hipGetErrorString(e));
    if (dev < 0 || dev >= kMaxDevices) return fail(OWT_EUNSUPPORTED, "device ordinal %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return fail(OWT_ELAUNCH, "hipGetSymbolAddress(scratch) failed on device %d: %s", dev, hipGetErrorString(e));
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return OWT_OK;
}

}  // namespace owt

using namespace owt;

extern "C" {

const char *owt_last_error(void) { return g_err; }
int owt_abi_version(void) { return 3; }

void owt_test_force_variant(int tile, int splitk, unsigned flags)
{
    g_force_tile.store(tile < 0 ? -1 : tile);
    g_force_split.store(splitk > 0 ? splitk : -1);
    g_force_flags.store(flags);
}

int owt_selftest_host(void)
{
    // exact-division constants: every divisor up to 4100 plus large ones, against n around
    // multiples of d, small n and the top of the 31-bit range
    static const uint32_t big[] = {9216, 21632, 93312, 387200, 3097600, 50176, 0x7fffffffu, 0x40000001u};
    for (uint32_t i = 1; i <= 4100 + sizeof(big) / sizeof(big[0]); i++) {
        const uint32_t d = i <= 4100 ? i : big[i - 4101];
        FastDiv f; f.set(d);
        for (uint32_t j = 0; j < 64; j++) {
            const uint64_t mul = (uint64_t)d * (j * 0x01000193u % 100000u);
            const uint32_t cand[] = {j, (uint32_t)(mul & 0x7fffffffu), (uint32_t)((mul + d - 1) & 0x7fffffffu),
                                     0x7fffffffu - j, 0x7fffffffu / (j + 1)};
            for (uint32_t n : cand)
                if (f.div(n) != n / d) { fail(OWT_EINVAL, "FastDiv wrong: %u / %u", n, d); return 1; }
        }
    }
    // every candidate launch covers all reduction steps with no empty split, and fits its workspace bound
    static const int shapes[][7] = {{128, 3, 224, 64, 11, 4, 2}, {128, 64, 27, 192, 5, 1, 2}, {128, 192, 13, 384, 3, 1, 1},
                                    {128, 384, 13, 256, 3, 1, 1}, {8, 3, 32, 16, 5, 1, 2}, {2, 8, 7, 4, 7, 1, 0},
                                    {1024, 256, 13, 256, 3, 1, 1}, {128, 9216, 1, 512, 1, 1, 0}, {1, 1, 3, 1, 3, 1, 1}};
    for (const auto &sh : shapes) {
        Geom g;
        if (!fill_geom(g, sh[0], sh[1], sh[2], sh[2], sh[3], sh[4], sh[4], sh[5], sh[5], sh[6], sh[6])) return 2;
        for (int pass = 0; pass < 3; pass++) {
            const PassDims dm = conv_dims(g, pass);
            std::vector<Launch> c;
            enumerate(g, pass, dm, pass == OWT_PASS_BWD_FILTER, c);
            if (c.empty()) { fail(OWT_EINVAL, "no candidate for shape N=%d C=%d pass %d", sh[0], sh[1], pass); return 3; }
            const size_t bound = max_workspace(g, pass, dm, pass == OWT_PASS_BWD_FILTER);
            const double least = least_cost(c);
            for (const Launch &l : c) {
                const long parts = (l.kind == KIND_SCONV || l.kind == KIND_SCONV2 || l.kind == KIND_SCONV16) ? l.tiles_n : l.splits;   // who shares the steps
                if (l.splits < 1 || parts * l.steps_per_split < l.steps ||
                    (parts - 1) * l.steps_per_split >= l.steps || (l.ws_bytes() > bound && worth_workspace(l, least)) ||
                    ((l.kind == KIND_DIRECT || l.kind == KIND_DIRECT16) && (l.pr > 624 || direct_panel_rows(g, pass, dm, kTiles[l.tile].BM) > l.pr))) {
                    fail(OWT_EINVAL, "bad candidate for shape N=%d C=%d pass %d", sh[0], sh[1], pass); return 4;
                }
            }
        }
    }
    return 0;
}

size_t owt_conv_workspace_bytes(const owt_conv_desc *d, int pass)
{
    Geom g;
    if (pass < 0 || pass > 2) { fail(OWT_EINVAL, "pass must be 0, 1 or 2"); return (size_t)-1; }
    if (check_conv(d, g) != OWT_OK) return (size_t)-1;
    g.masked = 0;                                      // the bound covers calls with and without the mask
    const bool cached = !variants_forced();
    if (cached) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        auto it = g_workspace.find(plan_key(g, pass, d->dtype));
        if (it != g_workspace.end()) return it->second;
    }
    const size_t need = max_workspace(g, pass, conv_dims(g, pass), pass == OWT_PASS_BWD_FILTER);
    if (cached) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        g_workspace[plan_key(g, pass, d->dtype)] = need;
    }
    return need;
}

int owt_conv_plan_describe(const owt_conv_desc *d, int pass, char *buf, size_t buf_bytes)
{
    Geom g;
    if (pass < 0 || pass > 2 || !buf || buf_bytes == 0) { fail(OWT_EINVAL, "bad pass or buffer"); return -1; }
    if (check_conv(d, g) != OWT_OK) return -1;
    const PassDims dm = conv_dims(g, pass);
    return describe(buf, buf_bytes, pass, d->dtype, dm, choose(g, pass, d->dtype, dm, pass == OWT_PASS_BWD_FILTER, true));
}

owt_status owt_conv_fwd(const owt_conv_desc *d, const void *x, const void *w, const float *bias,
                        void *y, void *ws, size_t ws_bytes, void *hip_stream)
{
    Geom g;
    OWT_TRY(check_conv(d, g));
    OWT_TRY(check_ptr(x, "x")); OWT_TRY(check_ptr(w, "w")); OWT_TRY(check_ptr(y, "y"));
    if (d->flags & OWT_BIAS) OWT_TRY(check_ptr(bias, "bias"));
    return conv_pass(g, OWT_PASS_FWD, d->dtype, fwd_params(d, x, w, bias, y), false, ws, ws_bytes,
                     (hipStream_t)hip_stream, true);
}

owt_status owt_conv_bwd_data(const owt_conv_desc *d, const void *dy, const void *y_or_null,
                             const void *w, void *dx, void *ws, size_t ws_bytes, void *hip_stream)
{
    Geom g;
    OWT_TRY(check_conv(d, g));
    OWT_TRY(check_ptr(dy, "dy")); OWT_TRY(check_ptr(w, "w")); OWT_TRY(check_ptr(dx, "dx"));
    if (d->flags & OWT_RELU) OWT_TRY(check_ptr(y_or_null, "y (needed for the ReLU mask)"));
    return conv_pass(g, OWT_PASS_BWD_DATA, d->dtype, data_params(d, dy, y_or_null, w, dx), false, ws, ws_bytes,
                     (hipStream_t)hip_stream, true);
}

owt_status owt_conv_bwd_data_relu_in(const owt_conv_desc *d, const void *dy, const void *y_or_null,
                                     const void *w, const void *x, void *dx, void *ws, size_t ws_bytes,
                                     void *hip_stream)
{
    Geom g;
    OWT_TRY(check_conv(d, g));
    OWT_TRY(check_ptr(dy, "dy")); OWT_TRY(check_ptr(w, "w")); OWT_TRY(check_ptr(dx, "dx")); OWT_TRY(check_ptr(x, "x"));
    if (d->flags & OWT_RELU) OWT_TRY(check_ptr(y_or_null, "y (needed for the ReLU mask)"));
    return conv_pass(g, OWT_PASS_BWD_DATA, d->dtype, data_params(d, dy, y_or_null, w, dx, x), false, ws, ws_bytes,
                     (hipStream_t)hip_stream, true);
}

owt_status owt_conv_bwd_filter(const owt_conv_desc *d, const void *x, const void *dy,
                               const void *y_or_null, float alpha, float beta, float *dw,
                               float *dbias_or_null, void *ws, size_t ws_bytes, void *hip_stream)
{
    Geom g;
    OWT_TRY(check_conv(d, g));
    OWT_TRY(check_ptr(x, "x")); OWT_TRY(check_ptr(dy, "dy")); OWT_TRY(check_ptr(dw, "dw"));
    if (dbias_or_null) OWT_TRY(check_ptr(dbias_or_null, "dbias"));
    if (d->flags & OWT_RELU) OWT_TRY(check_ptr(y_or_null, "y (needed for the ReLU mask)"));
    return conv_pass(g, OWT_PASS_BWD_FILTER, d->dtype, filter_params(d, x, dy, y_or_null, alpha, beta, dw, dbias_or_null),
                     true, ws, ws_bytes, (hipStream_t)hip_stream, true);
}

size_t owt_static_scratch_bytes(void) { return kStaticScratchBytes; }

owt_status owt_conv_bwd_filter_static(const owt_conv_desc *d, const void *x, const void *dy, const void *y_or_null,
                                      float alpha, float beta, float *dw, float *dbias_or_null, void *hip_stream)
{
    Geom g;
    OWT_TRY(check_conv(d, g));
    OWT_TRY(check_ptr(x, "x")); OWT_TRY(check_ptr(dy, "dy")); OWT_TRY(check_ptr(dw, "dw"));
    if (dbias_or_null) OWT_TRY(check_ptr(dbias_or_null, "dbias"));
    if (d->flags & OWT_RELU) OWT_TRY(check_ptr(y_or_null, "y (needed for the ReLU mask)"));
    const PassDims dm = conv_dims(g, OWT_PASS_BWD_FILTER);
    // the variant owt_conv_bwd_filter would run if its partial sums fit the static array, else the
    // cheapest (by the cost model) of those that do
    Launch l = choose(g, OWT_PASS_BWD_FILTER, d->dtype, dm, true, true);
    if (l.ws_bytes() > kStaticScratchBytes) {
        std::vector<Launch> c;
        enumerate(g, OWT_PASS_BWD_FILTER, dm, true, c);
        size_t best = c.size(), least = (size_t)-1;
        for (size_t i = 0; i < c.size(); i++) {
            least = c[i].ws_bytes() < least ? c[i].ws_bytes() : least;
            if (c[i].ws_bytes() <= kStaticScratchBytes && (best == c.size() || c[i].cost < c[best].cost)) best = i;
        }
        if (best == c.size())
            return fail(OWT_EWORKSPACE, "this filter gradient needs at least %zu bytes of scratch; the static buffer holds %zu "
                        "(use owt_conv_bwd_filter with a caller workspace)", least, kStaticScratchBytes);
        l = c[best];
    }
    void *ws = nullptr;
    OWT_TRY(static_scratch(&ws));
    return launch(g, OWT_PASS_BWD_FILTER, d->dtype, dm, filter_params(d, x, dy, y_or_null, alpha, beta, dw, dbias_or_null), l, ws,
                  (hipStream_t)hip_stream);
}

owt_status owt_conv_autotune(const owt_conv_desc *d, int pass, const void *x, const void *w, const float *bias,
                             void *y, const void *dy, void *dx, float *dw, float *dbias_or_null, void *ws,
                             size_t ws_bytes, void *hip_stream)
{
    Geom g;
    if (pass < 0 || pass > 2) return fail(OWT_EINVAL, "pass must be 0, 1 or 2");
    OWT_TRY(check_conv(d, g));
    OWT_TRY(check_ptr(w, "w"));
    GemmParams p;
    if (pass == OWT_PASS_FWD) {
        OWT_TRY(check_ptr(x, "x")); OWT_TRY(check_ptr(y, "y"));
        if (d->flags & OWT_BIAS) OWT_TRY(check_ptr(bias, "bias"));
        p = fwd_params(d, x, w, bias, y);
    } else {
        OWT_TRY(check_ptr(dy, "dy"));
        if (d->flags & OWT_RELU) OWT_TRY(check_ptr(y, "y (needed for the ReLU mask)"));
        if (pass == OWT_PASS_BWD_DATA) { OWT_TRY(check_ptr(dx, "dx")); p = data_params(d, dy, y, w, dx); }
        else { OWT_TRY(check_ptr(x, "x")); OWT_TRY(check_ptr(dw, "dw")); p = filter_params(d, x, dy, y, 1.f, 0.f, dw, dbias_or_null); }
    }
    const PassDims dm = conv_dims(g, pass);
    std::vector<Launch> c;
    enumerate(g, pass, dm, pass == OWT_PASS_BWD_FILTER, c);
    // as a call does (choose()), tuning passes over split-operand plans that the scratch is too small for
    const size_t usable = ws && aligned16(ws) ? ws_bytes : 0;
    c.erase(std::remove_if(c.begin(), c.end(), [&](const Launch &l) { return is_split_kind(l.kind) && l.ws_bytes() > usable; }), c.end());
    for (const Launch &l : c) OWT_TRY(check_ws(l, ws, ws_bytes));
    hipStream_t s = (hipStream_t)hip_stream;
    if (c.empty()) return fail(OWT_EUNSUPPORTED, "no kernel variant for this geometry");
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return fail(OWT_ELAUNCH, "hipEventCreate failed");
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return fail(OWT_ELAUNCH, "hipEventCreate failed"); }
    int best = -1; float best_ms = 0.f;
    owt_status st = OWT_OK;
    const double least = least_cost(c);
    for (size_t i = 0; i < c.size() && st == OWT_OK; i++) {
        if (!worth_timing(c[i], least) && !variants_forced()) continue;
        st = launch(g, pass, d->dtype, dm, p, c[i], ws, s);                       // warm-up
        if (st != OWT_OK) break;
        // 3 launches; a variant that takes under 50 us is timed again over 12 (launch jitter is a few us)
        float ms = 0.f;
        bool ok = true;
        for (int reps = 3; ok && st == OWT_OK; reps = 12) {
            ok = hipEventRecord(e0, s) == hipSuccess;
            for (int r = 0; r < reps && st == OWT_OK; r++) st = launch(g, pass, d->dtype, dm, p, c[i], ws, s);
            if (st != OWT_OK) break;
            ok = ok && hipEventRecord(e1, s) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
                 hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
            ms /= (float)reps;
            if (reps == 12 || ms > 0.05f) break;
        }
        if (st != OWT_OK) break;
        if (!ok) { st = fail(OWT_ELAUNCH, "timing a kernel variant failed: %s", hipGetErrorString(hipGetLastError())); break; }
        if (best < 0 || ms < best_ms) { best = (int)i; best_ms = ms; }
    }
    (void)hipEventDestroy(e0); (void)hipEventDestroy(e1);
    if (st != OWT_OK) return st;
    std::lock_guard<std::mutex> lk(g_tuned_mutex);
    g_tuned[plan_key(g, pass, d->dtype)] = c[best];
    g_fc_pairs.erase(plan_key(g, 3, d->dtype));      // a pair plan built on the old choice is stale
    return OWT_OK;
}

// ------------------------------------------------------- fully-connected shard
static owt_status check_fc(const owt_fc_desc *d, Geom &g, int &o_local)
{
    if (!d) return fail(OWT_EINVAL, "descriptor is NULL");
    if (d->N <= 0 || d->I <= 0 || d->O_total <= 0 || d->workers <= 0)
        return fail(OWT_EINVAL, "N, I, O_total, workers must be positive");
    if (d->rank < 0 || d->rank >= d->workers) return fail(OWT_EINVAL, "need 0 <= rank < workers");
    if (d->O_total % d->workers) return fail(OWT_EINVAL, "O_total must be divisible by workers");
    if (d->dtype != OWT_F32 && d->dtype != OWT_BF16) return fail(OWT_EINVAL, "unknown dtype %d", (int)d->dtype);
    if (d->flags & ~(unsigned)(OWT_BIAS | OWT_RELU)) return fail(OWT_EINVAL, "unknown flag bits 0x%x", d->flags);
    o_local = d->O_total / d->workers;
    if ((long)d->N * d->I > kMaxElems || (long)o_local * d->I > kMaxElems)
        return fail(OWT_EUNSUPPORTED, "tensor with more than 2^31-1 elements");
    fill_geom(g, d->N, d->I, 1, 1, o_local, 1, 1, 1, 1, 0, 0);
    g.bf16 = d->dtype == OWT_BF16;
    return OWT_OK;
}

// Workspace every candidate of the shard's passes fits in, remembered per geometry: the backward call checks
// it on every launch, and listing the candidates costs microseconds on a path whose kernels take ten.
static std::map<PlanKey, size_t> g_fc_ws;

static size_t fc_workspace(const Geom &g, owt_dtype dt, int pass)
{
    const PlanKey key = plan_key(g, 4 + (pass == OWT_PASS_FWD ? 0 : 1), dt);
    if (!variants_forced()) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        auto it = g_fc_ws.find(key);
        if (it != g_fc_ws.end()) return it->second;
    }
    size_t need;
    if (pass == OWT_PASS_FWD) need = max_workspace(g, OWT_PASS_FWD, conv_dims(g, OWT_PASS_FWD), false);
    else {      // the backward call runs the data pass, then the filter pass, on one scratch area
        const size_t a = max_workspace(g, OWT_PASS_BWD_DATA, conv_dims(g, OWT_PASS_BWD_DATA), false);
        const size_t b = max_workspace(g, OWT_PASS_BWD_FILTER, conv_dims(g, OWT_PASS_BWD_FILTER), true);
        need = a > b ? a : b;
    }
    if (!variants_forced()) {
        std::lock_guard<std::mutex> lk(g_tuned_mutex);
        g_fc_ws[key] = need;
    }
    return need;
}

size_t owt_fc_workspace_bytes(const owt_fc_desc *d, int pass)
{
    Geom g; int ol;
    if (pass < 0 || pass > 2) { fail(OWT_EINVAL, "pass must be 0, 1 or 2"); return (size_t)-1; }
    if (check_fc(d, g, ol) != OWT_OK) return (size_t)-1;
    return fc_workspace(g, d->dtype, pass);
}

owt_status owt_fc_shard_fwd(const owt_fc_desc *d, const void *x, const void *w, const float *bias,
                            void *y, void *ws, size_t ws_bytes, void *hip_stream)
{
    Geom g; int ol;
    OWT_TRY(check_fc(d, g, ol));
    OWT_TRY(check_ptr(x, "x")); OWT_TRY(check_ptr(w, "w")); OWT_TRY(check_ptr(y, "y"));
    if (d->flags & OWT_BIAS) OWT_TRY(check_ptr(bias, "bias"));
    GemmParams p; memset(&p, 0, sizeof(p));
    p.a = x; p.b = w; p.out = y; p.bias = bias; p.flags = d->flags;
    return conv_pass(g, OWT_PASS_FWD, d->dtype, p, false, ws, ws_bytes, (hipStream_t)hip_stream, true);
}

owt_status owt_fc_shard_bwd(const owt_fc_desc *d, const void *x, const void *w, const void *y_or_null,
                            const void *dy, float alpha, float beta, void *dx_partial_or_null,
                            float *dw, float *dbias_or_null, void *ws, size_t ws_bytes,
                            void *hip_stream)
{
    Geom g; int ol;
    OWT_TRY(check_fc(d, g, ol));
    OWT_TRY(check_ptr(x, "x")); OWT_TRY(check_ptr(w, "w")); OWT_TRY(check_ptr(dy, "dy"));
    OWT_TRY(check_ptr(dw, "dw"));
    if (dx_partial_or_null) OWT_TRY(check_ptr(dx_partial_or_null, "dx_partial"));
    if (dbias_or_null) OWT_TRY(check_ptr(dbias_or_null, "dbias"));
    if (d->flags & OWT_RELU) OWT_TRY(check_ptr(y_or_null, "y (needed for the ReLU mask)"));
    const size_t need = fc_workspace(g, d->dtype, OWT_PASS_BWD_DATA);
    if (ws_bytes < need) return fail(OWT_EWORKSPACE, "workspace too small: need %zu bytes, got %zu", need, ws_bytes);
    if (need && (!ws || !aligned16(ws))) return fail(OWT_EINVAL, "ws is NULL or misaligned");
    const void *mask = (d->flags & OWT_RELU) ? y_or_null : nullptr;
    GemmParams pd; memset(&pd, 0, sizeof(pd));
    pd.a = dy; pd.b = w; pd.out = dx_partial_or_null; pd.flags = d->flags; pd.mask = mask;
    GemmParams p; memset(&p, 0, sizeof(p));
    p.a = dy; p.b = x; p.out = dw; p.flags = d->flags; p.alpha = alpha; p.beta = beta;
    p.dbias = dbias_or_null; p.mask = mask;
    if (dx_partial_or_null) {
        // both products on the dense kernel: one dz for the two, and one launch for both when that is faster
        FcPair fp;
        if (fc_pair_plan(g, d->dtype, fp)) {
            OWT_TRY(check_ws(fp.ld, ws, ws_bytes)); OWT_TRY(check_ws(fp.lf, ws, ws_bytes));
            return launch_fc_pair(g, fp, pd, p, ws, (hipStream_t)hip_stream);
        }
        OWT_TRY(conv_pass(g, OWT_PASS_BWD_DATA, d->dtype, pd, false, ws, ws_bytes, (hipStream_t)hip_stream, true));
    }
    return conv_pass(g, OWT_PASS_BWD_FILTER, d->dtype, p, true, ws, ws_bytes, (hipStream_t)hip_stream, true);
}

owt_status owt_fc_autotune(const owt_fc_desc *d, const void *x, const void *w, const float *bias, void *y,
                           const void *dy, void *dx_partial, float *dw, float *dbias_or_null, void *ws,
                           size_t ws_bytes, void *hip_stream)
{
    // the shard is the convolution with H = W = R = S = 1 on [N, I] -> [N, O_local]: tune that geometry
    Geom g; int ol;
    OWT_TRY(check_fc(d, g, ol));
    owt_conv_desc c;
    memset(&c, 0, sizeof(c));
    c.N = d->N; c.C = d->I; c.H = c.W = 1; c.K = ol; c.R = c.S = 1; c.stride_h = c.stride_w = 1;
    c.dtype = d->dtype; c.flags = d->flags;
    const size_t need_f = owt_fc_workspace_bytes(d, OWT_PASS_FWD), need_b = owt_fc_workspace_bytes(d, OWT_PASS_BWD_DATA);
    if (ws_bytes < (need_f > need_b ? need_f : need_b))
        return fail(OWT_EWORKSPACE, "workspace too small: need %zu bytes, got %zu", need_f > need_b ? need_f : need_b, ws_bytes);
    OWT_TRY(owt_conv_autotune(&c, OWT_PASS_FWD, x, w, bias, y, nullptr, nullptr, nullptr, nullptr, ws, ws_bytes, hip_stream));
    OWT_TRY(owt_conv_autotune(&c, OWT_PASS_BWD_DATA, nullptr, w, nullptr, y, dy, dx_partial, nullptr, nullptr, ws, ws_bytes,
                              hip_stream));
    OWT_TRY(owt_conv_autotune(&c, OWT_PASS_BWD_FILTER, x, w, nullptr, y, dy, nullptr, dw, dbias_or_null, ws, ws_bytes,
                              hip_stream));
    // the ways to run the two backward products of a call that wants both
    if (variants_forced()) return OWT_OK;
    std::vector<std::pair<int, FcPair>> ways;
    for (int way : {FC_SEPARATE, FC_DENSE_TWO, FC_DENSE_ONE, FC_XFC}) {
        FcPair fp;
        const bool pair = fc_pair_of(g, d->dtype, way, fp);
        const bool dense = fp.ld.kind == KIND_FCGEMM && fp.lf.kind == KIND_FCGEMM;
        if (way == FC_SEPARATE ? !dense && !(fp.ld.kind == KIND_XFC && fp.lf.kind == KIND_XFC)
                               : pair && fp.xfc == (way == FC_XFC) && fp.fused == (way == FC_DENSE_ONE))
            ways.push_back(std::make_pair(way, fp));
    }
    if (ways.empty()) return OWT_OK;
    const void *mask = (d->flags & OWT_RELU) ? y : nullptr;
    GemmParams pd; memset(&pd, 0, sizeof(pd));
    pd.a = dy; pd.b = w; pd.out = dx_partial; pd.flags = d->flags; pd.mask = mask;
    GemmParams pf; memset(&pf, 0, sizeof(pf));
    pf.a = dy; pf.b = x; pf.out = dw; pf.flags = d->flags; pf.alpha = 1.f; pf.beta = 0.f; pf.dbias = dbias_or_null; pf.mask = mask;
    hipStream_t s = (hipStream_t)hip_stream;
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess) return fail(OWT_ELAUNCH, "hipEventCreate failed");
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return fail(OWT_ELAUNCH, "hipEventCreate failed"); }
    float best_ms = 0.f;
    int best = -1;
    owt_status st = OWT_OK;
    const auto run = [&](int way, const FcPair &fp) {
        if (way != FC_SEPARATE) return launch_fc_pair(g, fp, pd, pf, ws, s);
        const owt_status sd = launch(g, OWT_PASS_BWD_DATA, d->dtype, conv_dims(g, OWT_PASS_BWD_DATA), pd, fp.ld, ws, s);
        return sd != OWT_OK ? sd : launch(g, OWT_PASS_BWD_FILTER, d->dtype, conv_dims(g, OWT_PASS_BWD_FILTER), pf, fp.lf, ws, s);
    };
    for (size_t v = 0; v < ways.size() && st == OWT_OK; v++) {
        float ms = 0.f;
        st = run(ways[v].first, ways[v].second);                                   // warm-up
        bool ok = st == OWT_OK && hipEventRecord(e0, s) == hipSuccess;
        for (int r = 0; r < 12 && st == OWT_OK; r++) st = run(ways[v].first, ways[v].second);
        if (st != OWT_OK) break;
        ok = ok && hipEventRecord(e1, s) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
             hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
        if (!ok) st = fail(OWT_ELAUNCH, "timing the backward pair failed: %s", hipGetErrorString(hipGetLastError()));
        if (best < 0 || ms < best_ms) { best = (int)v; best_ms = ms; }
    }
    (void)hipEventDestroy(e0); (void)hipEventDestroy(e1);
    if (st != OWT_OK) return st;
    std::lock_guard<std::mutex> lk(g_tuned_mutex);
    g_fc_way[plan_key(g, 3, d->dtype)] = ways[best].first;
    g_fc_pairs.erase(plan_key(g, 3, d->dtype));
    return OWT_OK;
}

}  // extern "C"
