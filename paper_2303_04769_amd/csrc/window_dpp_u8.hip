// Quantized depthwise 3x3 convolution, stride 1, padding 1, 16-byte channel blocks: the uint8 counterpart of
// window_dpp.hip. uint8 codes in and out, exact int32 sums, the library's requantization rule; HBM traffic is a
// quarter of the fp32 layer's, so the bound is the vector instructions of the requantization, not memory.
//
// The mapping is window_dpp.hip's: a wave owns 16 neighbouring pixels of a strip of at most 3, 5, 7 or 9 rows of one plane
// (or several narrow planes side by side), lane = 16 q + l holding the four channels 4q .. 4q + 3 of pixel l --
// one 32-bit word of the pixel's 16-byte block. Every lane requests its 5 to 11 input words at once (buffer
// addressing: lanes and rows outside the image read as the code zx); the left and right neighbours come from
// lanes l - 1 and l + 1 by lane shifts of the words (zero is shifted in at a band's ends: lanes 0 and 15 produce no
// output there, or the value is replaced). The sums are taken on the matrix cores (see the kernel), go through the
// requantization (HIGH: the form for scales below a half, else the clamped one: the host sends only layers whose scale allows
// it) and into their byte of the output word.
#include "small_internal.h"

namespace small {

namespace {

struct DppU8Args {
    const unsigned char *in;
    const unsigned char *filt;     // [C/16][3][3][16]
    unsigned char *out;
    int H, W, nCb;
    int n_planes;          // N * nCb
    int nb;                // bands per row
    int sp;                // row strips per plane
    int n_units;           // image groups * nCb * sp * nb (FOLD: strip groups * nCb): one per wave
    int ppb;               // planes (FOLD: strips) per band of 16 lanes
    unsigned bytes;        // of the input = of the output tensor (< 2^31)
    FastDiv by_nb, by_sp, by_nCb, by_W;
    int cached;            // CACHED (of HIGH only): stores through the cache, not non-temporal
    QuantParams q;
    int nz;                // NZ where that is kAnyNZ
};

// ROWS: output rows per strip (two more input rows prime the window), at most; a wave computes that many whatever its strip has.

typedef int intx4 __attribute__((ext_vector_type(4)));

// SEG 16: a band is 16 neighbouring pixels of one plane (14 outputs). SEG 8: rows of at most 7 pixels, two planes
// side by side with a lane of padding on their left. SEG 0: rows of at most 5 pixels, floor(16 / W) planes back to
// back without padding lanes (three planes of 5-pixel rows instead of two): the neighbour a plane's
// first and last pixel would take from the plane next to it is replaced by the code zx with a select.
//
// The sums are taken on signed bytes x' = x - 128 and w' = w - 128 (one exclusive-or per word):
//     sum (x - zx)(w - zw) = sum x' w' + b sum x' + a sum w' + 9 a b,   a = 128 - zx, b = 128 - zw,
// over all nine taps, those outside the image carrying the code zx. v_mfma_i32_16x16x64_i8 sums 64 products, 16 of them in each
// group of 16 lanes, and which element a step is only has to be the same in both operands: lane (pixel l, quad q) gives the words
// of its four channels at the left neighbour, the pixel and the right one, as they are in its registers, and a fourth word that
// meets zeros; the other operand has, for output channel m, m's taps of a window row in the bytes of that channel in group m / 4,
// zero elsewhere. A window row is then one instruction for all 16 channels, and its sums come out in the lane that holds their
// pixel. b sum x' is a second instruction per row with b in every tap (NZ = 1; NZ = 2: b = 128, no signed byte, as twice 64);
// it is left out for zw = 128 (NZ = 0). Of 16 products 15 meet a zero, but the matrix cores are idle otherwise: with byte
// permutes into words of one channel's three taps and four-byte dot products, the vector units' way, a word took 6 permutes and
// 12 dot products more (and 16 instructions for the sum of the codes): 1024 images of 64 channels 25x5, zw = 131, 9.4 us / 7.9
// now, 64 of 96 57x43 13.7 / 11.5, 64 of 256 14x14 with zw = 128 4.24 / 3.89. One matrix instruction waits for another
// (about 0.05 us a wave): the smallest layers take as long as with dot products. Over 500 random layers with all of this and the
// rules for rows and stores below, and the requantization by the high word: 0.80 of the time before, none longer.
// The filter operand serves all pixels of the wave: planes side by side in a band (SEG 0, 8) are of one channel block and of
// consecutive images. FOLD: of too few images for that, a band takes strips instead, those of one channel block's planes in order,
// and each lane has its own rows.
constexpr int kAnyNZ = -1;
template <int SEG, int NZ, int ROWS, bool HIGH, bool CACHED, bool FOLD>
__global__ void __launch_bounds__(256) dw16_dpp_u8(DppU8Args a)
{
    constexpr int kSteps = ROWS + 2;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int unit = (int)blockIdx.x * 4 + wave;
    if (unit >= a.n_units) return;
    const int l = lane & 15, q = lane >> 4;

    const int t = FOLD ? unit : a.by_nb.div(unit), band = FOLD ? 0 : unit - t * a.nb;
    const int pg = FOLD ? unit : a.by_sp.div(t), strip = FOLD ? 0 : t - pg * a.sp;
    int r0 = strip * ROWS, r1 = min(r0 + ROWS, a.H);                                   // output rows r0 .. r1 - 1
    int n_in = r1 - r0 + 2;
    const int ig = a.by_nCb.div(pg), cb = pg - ig * a.nCb;                             // images (strips) ig * ppb .., channel block

    // (the rows before the images: behind them the scalar instructions come in another order, 1 % on the audio CNN's layer)
    int image, x;
    bool lane_used = true;
    if (SEG == 16) {
        image = ig;
        x = band * 14 - 1 + l;
    } else if (SEG == 8) {
        image = ig * 2 + (l >> 3);
        x = (l & 7) - 1;
    } else {
        const int pi = a.by_W.div(l);
        image = ig * a.ppb + pi;
        x = l - pi * a.W;
        lane_used = pi < a.ppb;
    }
    if (FOLD) {
        const int slot = image;
        image = a.by_sp.div(slot);
        r0 = (slot - image * a.sp) * ROWS;
        r1 = min(r0 + ROWS, a.H);
        n_in = r1 - r0 + 2;
    }
    const int plane = image * a.nCb + cb;
    const bool col_in = lane_used & (x >= 0) & (x < a.W) & (plane < a.n_planes);
    const bool col_out = col_in & (SEG != 16 || (l >= 1 && l <= 14));
    const bool at_left = x == 0, at_right = x == a.W - 1;          // (SEG 0)
    const int row_bytes = a.W * 16;
    const unsigned at = (unsigned)plane * (unsigned)(a.H * row_bytes) + (unsigned)(x * 16 + q * 4);

    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(a.in), 0, a.bytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, a.bytes, kRawBuffer);

    const unsigned flip = 0x80808080u, zxs = ((unsigned)a.q.zx * 0x01010101u) ^ flip;  // the padding code as signed bytes
    const unsigned *tp = reinterpret_cast<const unsigned *>(a.filt) + cb * 36 + (l >> 2);
    unsigned taps[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) taps[k] = tp[k * 4];
    unsigned raw[kSteps], sign[kSteps];                            // (what is not loaded is zero)
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
        const int r = r0 - 1 + j;
        const bool have = col_in & (r >= 0) & (r < a.H) & (j < n_in);
        raw[j] = __builtin_amdgcn_raw_buffer_load_b32(src, have ? at + (unsigned)(r * row_bytes) : kBeyond, 0, 0);
        sign[j] = have ? flip : zxs;
    }
    // the filter rows' operands, b's, and a sum w' + 9 a b per channel
    const int za = 128 - a.q.zx, zb = 128 - a.q.zw;
    const unsigned mine = q == l >> 2 ? 255u << (8 * (l & 3)) : 0u;
    intx4 w[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
#pragma unroll
        for (int k = 0; k < 3; ++k) w[r][k] = (int)((taps[3 * r + k] ^ flip) & mine);
        w[r][3] = 0;
    }
    const int nz = NZ == kAnyNZ ? a.nz : NZ;
    const int zw4 = (int)((unsigned)((nz == 2 ? zb / 2 : zb) & 255) * 0x01010101u & mine);
    const intx4 wz = {zw4, zw4, zw4, 0};
    intx4 cst = {0, 0, 0, 0};
    if (za != 0) {
        const intx4 ones = {0x01010101, 0x01010101, 0x01010101, 0};
#pragma unroll
        for (int r = 0; r < 3; ++r) cst = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[r], ones, cst, 0, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c) cst[c] = za * cst[c] + 9 * za * zb;
    }
    const long addend = requant_addend<HIGH>(a.q);

    intx4 row[kSteps];                                             // left, centre, right word of an input row
#pragma unroll
    for (int j = 0; j < kSteps; ++j) {
        const unsigned mid = raw[j] ^ sign[j];
        unsigned left = (unsigned)__builtin_amdgcn_update_dpp(0, (int)mid, kRowShr1, 0xf, 0xf, true);
        unsigned right = (unsigned)__builtin_amdgcn_update_dpp(0, (int)mid, kRowShl1, 0xf, 0xf, true);
        // (zero is shifted in at the ends of a row of 16 lanes; where such a lane has an output, it wants zx there)
        if (SEG == 0) {
            left = at_left ? zxs : left;
            right = at_right ? zxs : right;
        } else if (SEG == 8) {
            right = l == 15 ? zxs : right;
        }
        row[j] = intx4{(int)left, (int)mid, (int)right, 0};
        if (j < 2) continue;
        intx4 acc = cst;
#pragma unroll
        for (int r = 0; r < 3; ++r) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(w[r], row[j - 2 + r], acc, 0, 0, 0);
#pragma unroll
        for (int z = 0; z < (NZ == kAnyNZ ? 2 : NZ); ++z)
            if (NZ != kAnyNZ || z < nz)
#pragma unroll
                for (int r = 0; r < 3; ++r) acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(wz, row[j - 2 + r], acc, 0, 0, 0);
        unsigned y = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) y |= (unsigned)requant_code<HIGH>(acc[c], a.q, addend) << (8 * c);
        const unsigned off = (col_out & (j < n_in)) ? at + (unsigned)((r0 + j - 2) * row_bytes) : kBeyond;
        __builtin_amdgcn_raw_buffer_store_b32(y, dst, off, 0, CACHED ? 0 : kNonTemporal);
    }
}

// How a layer is cut: bands of rows (SEG), strips of rows, and what the lanes of a band hold. Images (fold = false) leave lanes idle
// where there are fewer of them than a band holds planes, 15 of 16 for one image of one-pixel rows; strips do not, but a lane's own
// rows cost vector compares. So strips where images fill at most half of the lanes and their shortest strips make more waves than the
// chip has SIMDs. us by images / by strips: one image of 4096 channels 600x1 17.4 / 4.1, 512 2000x2 7.9 / 4.2, 4096 64x5 4.2 / 3.3, 16
// 30000x7 5.1 / 4.2, eight images of 512 300x1 4.4 / 3.5; below that line 0.87 to 1.06 of the time: 128 channels 40x4 2.70 / 2.85. (With
// planes of any channel block side by side, which dot products by the vector unit allowed: 7.0 for the first, 5.7 for the second.)
struct Plan { int seg, ppb, nb, rows, sp; bool fold; long units; };

// Rows per strip: a wave costs about as much as 5 rows and its rows, also those that its strip lacks; up to eight waves a SIMD
// the busiest one counts, beyond that their average, and one more wave's time passes before and after. Over 500 random layers the
// rows taken cost 0.4 % more than the best of 3, 5, 7 and 9 each time; 3 alone 5 %, 5 6 %, 7 9 %, 9 15 %, 13 26 % (13 is the best
// for one layer in ten, by 0.3 % of the whole). us with 7 / with the one taken: one image of 128 channels 2x2 2.77 / 2.41 with 3,
// 8 of 96 7x7 3.22 / 2.83 with 3, 16 of 64 13x4 3.49 / 2.88 with 3.
Plan plan_dw(const LayerGeom &g)
{
    Plan pl;
    pl.seg = g.W <= 5 ? 0 : g.W <= 7 ? 8 : 16;
    pl.ppb = pl.seg == 0 ? 16 / g.W : pl.seg == 8 ? 2 : 1;
    pl.nb = pl.seg == 16 ? (g.W + 13) / 14 : 1;
    pl.fold = false;
    const long nCb = g.Ci / 16;
    const double simds = 4.0 * device_cus();
    auto units = [&](int rows) {
        const long sp = (g.H + rows - 1) / rows;
        return pl.fold ? (g.N * sp + pl.ppb - 1) / pl.ppb * nCb : ((long)g.N + pl.ppb - 1) / pl.ppb * nCb * sp * pl.nb;
    };
    pl.fold = 2 * g.N <= pl.ppb && units(3) > simds;
    auto cost = [&](int rows) {
        const long waves = units(rows), rounds = (waves + (long)simds - 1) / (long)simds;
        return ((rounds <= 8 ? (double)rounds : waves / simds) + 1) * (5 + rows);
    };
    pl.rows = 3;
    for (int rows = 5; rows <= 9; rows += 2)
        if (cost(rows) < cost(pl.rows)) pl.rows = rows;
    pl.sp = (g.H + pl.rows - 1) / pl.rows;
    pl.units = units(pl.rows);
    return pl;
}

template <int ROWS, bool HIGH, bool CACHED, int NZ>
void go3(const DppU8Args &a, int seg, hipStream_t s)
{
    const dim3 grid((unsigned)((a.n_units + 3) / 4)), block(256);
    if (seg == 0) hipLaunchKernelGGL((dw16_dpp_u8<0, NZ, ROWS, HIGH, CACHED, false>), grid, block, 0, s, a);
    else if (seg == 8) hipLaunchKernelGGL((dw16_dpp_u8<8, NZ, ROWS, HIGH, CACHED, false>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((dw16_dpp_u8<16, NZ, ROWS, HIGH, CACHED, false>), grid, block, 0, s, a);
}
template <int ROWS, bool HIGH, bool CACHED>
void go2(const DppU8Args &a, int seg, hipStream_t s)
{
    if (a.q.zw == 128) go3<ROWS, HIGH, CACHED, 0>(a, seg, s);
    else if (a.q.zw == 0) go3<ROWS, HIGH, CACHED, 2>(a, seg, s);
    else go3<ROWS, HIGH, CACHED, 1>(a, seg, s);
}
template <int ROWS>
void go(const DppU8Args &a, int seg, hipStream_t s)
{
    if (a.q.mult32 < 0) go2<ROWS, false, false>(a, seg, s);
    else if (a.cached) go2<ROWS, true, true>(a, seg, s);
    else go2<ROWS, true, false>(a, seg, s);
}
template <int ROWS, bool HIGH>
void go_strips2(const DppU8Args &a, int seg, hipStream_t s)
{
    const dim3 grid((unsigned)((a.n_units + 3) / 4)), block(256);
    if (seg == 0) hipLaunchKernelGGL((dw16_dpp_u8<0, kAnyNZ, ROWS, HIGH, true, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((dw16_dpp_u8<8, kAnyNZ, ROWS, HIGH, true, true>), grid, block, 0, s, a);
}
template <int ROWS>
void go_strips(const DppU8Args &a, int seg, hipStream_t s)
{
    if (a.q.mult32 < 0) go_strips2<ROWS, false>(a, seg, s);
    else go_strips2<ROWS, true>(a, seg, s);
}

}  // namespace

bool dw_dpp_u8_eligible(const LayerGeom &g, const QuantParams &q, const void *in, const void *filt, const void *out)
{
    if (q.amax <= 0) return false;                            // (a scale too large for the clamped requantization)
    if (g.Cib != 16 || g.kh != 3 || g.kw != 3 || g.stride != 1 || g.pt != 1 || g.pl != 1) return false;
    if (g.Ho != g.H || g.Wo != g.W) return false;
    if ((((uintptr_t)in | (uintptr_t)filt | (uintptr_t)out) & 3u) != 0) return false;
    return (size_t)g.N * g.Ci * g.H * g.W < ((size_t)1 << 31);
}

DwForm dw_dpp_u8_form(const LayerGeom &g)
{
    const Plan pl = plan_dw(g);
    return {pl.units, pl.rows, pl.fold};
}

hipError_t launch_dw_dpp_u8(const unsigned char *in, const unsigned char *filt, unsigned char *out, const LayerGeom &g,
                            const QuantParams &q, hipStream_t s)
{
    DppU8Args a = {};
    a.in = in; a.filt = filt; a.out = out;
    a.H = g.H; a.W = g.W; a.nCb = g.Ci / 16;
    a.n_planes = g.N * a.nCb;
    a.bytes = (unsigned)((size_t)g.N * g.Ci * g.H * g.W);
    a.q = q;
    const Plan pl = plan_dw(g);
    a.ppb = pl.ppb; a.nb = pl.nb; a.sp = pl.sp;
    a.n_units = (int)pl.units;
    a.nz = q.zw == 128 ? 0 : q.zw == 0 ? 2 : 1;
    // Outputs of less than 4 MB stay in the cache, 3 to 6 % faster on average; past that the non-temporal stores are (8 to 16 MB: 8 %),
    // except to planes of one pixel a row, which a wave writes in pieces of 16 bytes at as many images: half a cache line each
    // (2000 images of 64 channels 86x1: 22.5 us non-temporal, 13.7). (A branch on it at each store costs 4 to 8 %.) Scales of a half
    // and more have the non-temporal form alone, strips side by side the other alone: one kernel less for each layer that hardly occurs.
    a.cached = a.bytes < (4u << 20) || g.W == 1;
    a.by_nb = make_fastdiv(a.nb);
    a.by_sp = make_fastdiv(a.sp);
    a.by_nCb = make_fastdiv(a.nCb);
    a.by_W = make_fastdiv(g.W);
    if (!pl.fold) {
        if (pl.rows == 3) go<3>(a, pl.seg, s);
        else if (pl.rows == 5) go<5>(a, pl.seg, s);
        else if (pl.rows == 7) go<7>(a, pl.seg, s);
        else go<9>(a, pl.seg, s);
    } else {
        if (pl.rows == 3) go_strips<3>(a, pl.seg, s);
        else if (pl.rows == 5) go_strips<5>(a, pl.seg, s);
        else if (pl.rows == 7) go_strips<7>(a, pl.seg, s);
        else go_strips<9>(a, pl.seg, s);
    }
    return hipGetLastError();
}

}  // namespace small
