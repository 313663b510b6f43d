// Convolution with the reduction split over the waves of a workgroup: layers with few output pixels and a long reduction,
// and, unless their reduction is short, the windows, strides and paddings that conv_same.hip has no tiles for.
//
// Bound: streaming the filter (every value is used for a handful of pixels only) and, per workgroup, a chain of matrix
// instructions. The tiled kernels give a layer of few pixels to a few workgroups that walk the whole reduction one step
// after the other -- 512 channels on one 6 x 6 image are 16 workgroups of 96 steps on a chip of 256 compute units. Here a
// wave owns WM x WN tiles of 16 output pixels x 16 output channels and takes a run of reduction steps, a step being one (input
// block, tap), the WAVES-th part of them. It keeps AHEAD steps of operands in flight in registers (no LDS and no barrier in the
// loop), and the partial sums meet in LDS at the end, in a fixed order. A tap outside the image is an offset beyond the buffer
// descriptor, which reads zero.
#include "small_internal.h"

namespace small {
namespace {

struct SplitArgs {
    const float *in, *filt, *res, *bn;
    float *out;
    int H, W, HoWo, Wo, M;
    int nCib, nCob, taps, kw, stride, pt, pl, steps, run;  // steps; of a wave
    int n_groups;                      // pixel groups of 16
    int epilogue;
    unsigned in_bytes, filt_bytes;
    FastDiv dHoWo, dWo, dCib, dTaps, dKw, dGroups;
};

template <int WAVES, int WM, int WN, bool TAPS_INSIDE, int AHEAD>
__global__ void __launch_bounds__(64 * WAVES) conv16_split(SplitArgs a)
{
    // CH sums per tile, matrix instruction r into sum r % CH: shorter chains round less often. With blocks innermost a wave's run meets
    // the image's border in whole stretches of zeros, so the other runs' sums are longer than if the steps were dealt out in turn; error against
    // 64 bits, 512 channels 3x3 6x6 one image / 7x7 four images: steps in turn 2.12e-7 / 4.02e-7, runs 2.21e-7 / 4.15e-7 with two sums
    // / one, 1.65e-7 / 2.97e-7 with four / two (+0.06 us).
    constexpr int T = WM * WN, CH = T == 1 ? 4 : 2;
    __shared__ floatx4 part[WAVES][T][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int p = lane & 15, q = lane >> 4;
    // pixel groups fastest: the workgroups that read one output block's filter meet in one L2
    const int wg = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    const int ct = quotient(a.dGroups, wg), grp = wg - ct * a.n_groups, cob0 = ct * WN;
    const int HW = a.H * a.W;
    int ih0[WM], iw0[WM], org[WM];                             // window origin; this lane's quad at tap (0, 0) of block 0
#pragma unroll
    for (int i = 0; i < WM; ++i) {
        const int m = min((grp * WM + i) * 16 + p, a.M - 1);
        const int n = quotient(a.dHoWo, m), rem = m - n * a.HoWo, oh = quotient(a.dWo, rem), ow = rem - oh * a.Wo;
        ih0[i] = oh * a.stride - a.pt;
        iw0[i] = ow * a.stride - a.pl;
        org[i] = (n * a.nCib * HW + ih0[i] * a.W + iw0[i]) * 64 + q * 16;
    }
    // matrix instruction r multiplies input channel 4q + r of the step's 16 (both operands): lane (p, q) holds the input
    // quad of pixel p and, in instruction r, the filter value [4q + r][p]
    unsigned f_lane[WN];
#pragma unroll
    for (int j = 0; j < WN; ++j)
        f_lane[j] = cob0 + j < a.nCob ? (unsigned)((cob0 + j) * a.steps) * 1024u + (unsigned)(q * 64 + p) * 4u : kBeyond;

    // This wave's run: from a block to the next only the scalar offsets of the loads change, from a tap to the next the lanes' offsets
    // too, of which the tap's place in the image is part. Behind the run's end the descriptors have no size (and the scalar offsets are
    // zero, for the hardware takes them off the size): such loads read zero.
    const int first = wave * a.run, last = min(first + a.run, a.steps);
    floatx4 x[AHEAD][WM];
    float w[AHEAD][WN][4];
    int outer = quotient(TAPS_INSIDE ? a.dTaps : a.dCib, first), inner = first - outer * (TAPS_INSIDE ? a.taps : a.nCib), s_next = first;
    int &tap = TAPS_INSIDE ? inner : outer, &cib = TAPS_INSIDE ? outer : inner;
    unsigned at[WM];
    auto lanes = [&]() __attribute__((always_inline)) {
        const int y = quotient(a.dKw, tap), z = tap - y * a.kw;
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const bool inside = ((unsigned)(ih0[i] + y) < (unsigned)a.H) & ((unsigned)(iw0[i] + z) < (unsigned)a.W);
            at[i] = inside ? (unsigned)(org[i] + (y * a.W + z) * 64) : kBeyond;
        }
    };
    lanes();
    auto request = [&](floatx4 (&xs)[WM], float (&ws)[WN][4]) __attribute__((always_inline)) {
        const bool more = s_next < last;
        const int x_block = more ? cib * HW * 64 : 0, w_block = more ? (cib * a.taps + tap) * 1024 : 0;
        const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.in), 0, more ? a.in_bytes : 0u, kRawBuffer);
        const __amdgpu_buffer_rsrc_t flt = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.filt), 0, more ? a.filt_bytes : 0u, kRawBuffer);
#pragma unroll
        for (int i = 0; i < WM; ++i) xs[i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, at[i], x_block, 0));
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                ws[j][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(flt, f_lane[j] + 64u * r, w_block, 0));
        ++s_next;
        const bool turn = ++inner == (TAPS_INSIDE ? a.taps : a.nCib);
        if (turn) {
            inner = 0;
            ++outer;
        }
        if (TAPS_INSIDE || turn) lanes();
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) request(x[i], w[i]);
    floatx4 acc[WM][WN][CH];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[i][j][c] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int s = first; s < last; s += AHEAD) {
#pragma unroll
        for (int k = 0; k < AHEAD; ++k) {
            // (steps past the end multiply zeros by zeros)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j)
                        acc[i][j][r % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[k][j][r], x[k][i][r], acc[i][j][r % CH], 0, 0, 0);
            request(x[k], w[k]);
        }
    }
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) {
            floatx4 v = acc[i][j][0] + acc[i][j][1];
            if (CH == 4) v += acc[i][j][CH - 2] + acc[i][j][CH - 1];
            part[wave][i * WN + j][lane] = v;
        }
    __syncthreads();
    for (int t = wave; t < T; t += WAVES) {
        floatx4 v = part[0][t][lane];
#pragma unroll
        for (int k = 1; k < WAVES; ++k) v += part[k][t][lane];
        const int m = (grp * WM + t / WN) * 16 + p, cob = cob0 + t % WN;
        if (m >= a.M || cob >= a.nCob) continue;
        const int n = quotient(a.dHoWo, m), rem = m - n * a.HoWo;
        const size_t o = ((size_t)(n * a.nCob + cob) * a.HoWo + rem) * 16 + q * 4;
        if (a.epilogue & EPI_BN) {
            const float *c = a.bn + cob * 16 + q * 4;
            const floatx4 sc = *reinterpret_cast<const floatx4 *>(c), sh = *reinterpret_cast<const floatx4 *>(c + a.nCob * 16);
            v.x = fmaf(v.x, sc.x, sh.x); v.y = fmaf(v.y, sc.y, sh.y); v.z = fmaf(v.z, sc.z, sh.z); v.w = fmaf(v.w, sc.w, sh.w);
        }
        if (a.epilogue & EPI_ADD) v += *reinterpret_cast<const floatx4 *>(a.res + o);
        if (a.epilogue & EPI_RELU) {
            v.x = v.x > 0.f ? v.x : 0.f; v.y = v.y > 0.f ? v.y : 0.f;
            v.z = v.z > 0.f ? v.z : 0.f; v.w = v.w > 0.f ? v.w : 0.f;
        }
        *reinterpret_cast<floatx4 *>(a.out + o) = v;
    }
}

struct Variant { int waves, wm, wn; const char *name, *name_taps; };
constexpr Variant kVariants[] = {{16, 1, 1, "conv16_split<16,1,1>", "conv16_split<16,1,1,taps>"}, {8, 1, 1, "conv16_split<8,1,1>", "conv16_split<8,1,1,taps>"},
                                 {4, 1, 1, "conv16_split<4,1,1>", "conv16_split<4,1,1,taps>"},    {4, 2, 1, "conv16_split<4,2,1>", "conv16_split<4,2,1,taps>"},
                                 {4, 2, 2, "conv16_split<4,2,2>", "conv16_split<4,2,2,taps>"},    {2, 2, 2, "conv16_split<2,2,2>", "conv16_split<2,2,2,taps>"}};

long split_steps(const LayerGeom &g) { return (long)(g.Ci / 16) * g.kh * g.kw; }
long split_tiles(const LayerGeom &g) { return ((long)g.N * g.Ho * g.Wo + 15) / 16 * (g.Co / 16); }

// Up to about five 16 x 16 tiles per compute unit every tile is a workgroup of its own, split the more ways the longer its
// reduction and the fewer the workgroups; beyond, waves own more tiles (operands serve two of them) and split less. Sweep
// over random layers when steps were dealt out in turn, which took 1.2 of the time, us: 96 tiles of 288 steps 10.4 / 15.9 / 11.9 with 16 / 8 / 4 waves; 90 tiles of 125 steps 7.8 / 7.2 /
// 7.3; 999 tiles of 243 steps 28.1 / 25.9 / 24.7; 3006 tiles of 25 steps 15.6 with <4,1,1>, 11.3 with <4,2,2>; 13128 tiles of
// 25 steps 44.5, 35.3, and 33.7 with <2,2,2>.
int pick_variant(const LayerGeom &g)
{
    const long steps = split_steps(g), tiles = split_tiles(g), cus = device_cus();
    if (2 * tiles <= 3 * cus) return steps >= 200 ? 0 : steps >= 64 ? 1 : 2;
    if (2 * tiles <= 11 * cus) return 2;
    if (g.Co == 16) return 3;
    return tiles <= 24 * cus ? 4 : 5;
}

// Which of block and tap a wave's run has innermost. The block: from step to step only scalar offsets change, which is up to 1.4
// times as fast where the data comes from the caches. But a pixel of a block is 64 bytes, half a cache line, and its neighbour, the
// next tap's, is then read a whole round of blocks later, from memory again once the layer's data is more than the caches hold:
// with the tap innermost it is 0.6 to 0.9 of the time there. The line: the input's bytes times the output blocks (how often they are
// read), 150 MB, or for strides above one, whose taps share less, input and filter, 14 MB. us, block / tap innermost (steps dealt
// out in turn before there were runs): 464 images of 384 channels 3x3 stride 2 7x7 202 / 127 (141), 27 of 464 -> 96 5x5 stride 2
// 49x13 185 / 133 (129), 60 of 192 -> 112 2x2 stride 2 27x80 111 / 74 (80), 136 of 128 3x3 stride 2 10x56 66 / 48 (51); below it 62
// of 384 -> 48 5x5 6x6 26 / 36 (42), 5 of 128 -> 16 3x3 7x47 4.1 / 5.6 (6.3). 2300 random layers of 6 us and more take 0.83 of the
// time with the steps dealt out; 4 are more than 4 % slower, none more than 9, and with the block innermost everywhere up to 63.
// (One output block, <4,2,1>: the block up to the first line, 80 -> 16 channels 3x1 stride 2 63x12, 125 images 6.3 / 7.1.)
bool taps_inside(const LayerGeom &g, int variant)
{
    const double in = (double)g.N * g.Ci * g.H * g.W * 4, filt = (double)g.Co * g.Ci * g.kh * g.kw * 4;
    return g.kh * g.kw > 1 && (in * (g.Co / 16) > 150e6 || (g.stride > 1 && variant != 3 && in + filt > 14e6));
}

// A run is filled up with steps of zeros to a multiple of the steps in flight. Three are enough (with four the layers took 1.04 of the
// time on average, with 6 and 9 1.12 and 1.22: 512 channels 3x3 6x6, one image, 18 steps a wave 8.6 / 9.3 / 9.3 / 9.9 us), but runs
// of 4, 8 and 16 steps come out even with four: two by two tiles 0.85, 0.95 and 0.95 of the time (64 channels 2x2 41x41, 7 images 10.1
// / 8.6), with the tap innermost 0.93, 1.09 and 1.05; waves with a tile of their own have more of them in flight and gain nothing.
template <int WAVES, int WM, int WN>
hipError_t run(const SplitArgs &a, bool taps, hipStream_t s)
{
    const dim3 grid((unsigned)(a.n_groups * ((a.nCob + WN - 1) / WN)));
    constexpr int kEven = WM * WN == 4 ? 4 : 3;
    if (taps && a.run == 4) hipLaunchKernelGGL((conv16_split<WAVES, WM, WN, true, kEven>), grid, dim3(64 * WAVES), 0, s, a);
    else if (taps) hipLaunchKernelGGL((conv16_split<WAVES, WM, WN, true, 3>), grid, dim3(64 * WAVES), 0, s, a);
    else if (a.run == 4 || a.run == 8 || a.run == 16) hipLaunchKernelGGL((conv16_split<WAVES, WM, WN, false, kEven>), grid, dim3(64 * WAVES), 0, s, a);
    else hipLaunchKernelGGL((conv16_split<WAVES, WM, WN, false, 3>), grid, dim3(64 * WAVES), 0, s, a);
    return hipGetLastError();
}

}  // namespace

static bool conv_split_can(const LayerGeom &g)
{
    return g.Cib == 16 && g.Cob == 16 && (long)g.N * g.Ho * g.Wo < (1L << 30) && split_tiles(g) < (1L << 30) && split_steps(g) < (1L << 20) &&
           (size_t)g.N * g.Ci * g.H * g.W * 4 < kBeyond && (size_t)g.Co * g.Ci * g.kh * g.kw * 4 < kBeyond;
}

bool conv_split_beats_gather(const LayerGeom &g)
{
    if (!conv_split_can(g)) return false;
    const long steps = split_steps(g), tiles = split_tiles(g), cus = device_cus();
    // Against the gather kernel of conv.hip, which spends a barrier per step but stages each input value once for a tile: the
    // shorter the reduction, the fewer tiles per compute unit until it wins. 500 random layers, time here over time there, for
    // few / many tiles: 4 steps 0.97 up to one tile a unit, 1.1 to 1.7 beyond (16 -> 32 channels 1x2 48x48 263 images 69 / 26 us,
    // 16 -> 16 1x3 14x14 9633 images 190 / 58); 8 steps 0.78 to 0.96 / 0.93 to 1.24; 9 to 11 steps 0.70 to 1.0 / 1.04 to 1.33;
    // 12 to 15 0.54 to 1.08 / 0.97 to 1.21; from 16 on 0.11 to 1.0, with many tiles 0.7 to 1.1 unless the last round of
    // steps (2 waves of 4, as the kernel was then) or of output blocks (two a tile) is too empty: 18 steps 0.93 to 1.23. (A run is filled
    // up to three steps now and the kernel takes 0.8 of the time; these lines have not been drawn again: 40 images of 32 channels
    // 40x40, unpadded, stay with the gather kernel though their 18 steps waste nothing any more.)
    const double most = steps < 4 ? 0 : steps < 8 ? 1 : steps < 9 ? 2.5 : steps < 12 ? (g.Co == 16 ? 8 : 5.5) : 20;
    const long nCob = g.Co / 16, done = (steps + 7) / 8 * 8 * ((nCob + 1) / 2 * 2);
    return tiles <= most * cus || (steps >= 16 && 100 * steps * nCob >= 78 * done);
}

bool conv_split_eligible(const LayerGeom &g)
{
    if (!conv_same_eligible(g)) return conv_split_beats_gather(g);
    if (!conv_split_can(g)) return false;
    const long steps = split_steps(g), tiles = split_tiles(g), cus = device_cus();
    // Against the tiles of conv_same.hip (their us / here, which was 1.2 times as slow then): up to one tile per compute unit from 7 steps on (189 tiles of 7
    // steps 3.9 / 3.1, 96 of 288 36.0 / 10.4; but 51 of 6 3.4 / 3.8), up to two for reductions of 32 (510 of 45 7.7 / 5.0; but 288
    // of 18 4.6 / 4.5), up to four for 200 (999 of 243 45.7 / 24.7; but 912 of 144 19.5 / 21.5); above that they win (2090 of 45 13.3 / 12.8, 4032 of
    // 63 21.3 / 25.5).
    return tiles <= cus ? steps >= 7 : tiles <= 2 * cus ? steps >= 32 : tiles <= 4 * cus && steps >= 200;
}

const char *conv_split_kernel_name(const LayerGeom &g)
{
    const int v = pick_variant(g);
    return taps_inside(g, v) ? kVariants[v].name_taps : kVariants[v].name;
}

hipError_t launch_conv_split(const float *in, const float *filt, float *out, const float *res, const LayerGeom &g, int epilogue,
                             hipStream_t s, const float *bn)
{
    SplitArgs a;
    a.in = in; a.filt = filt; a.out = out; a.res = res; a.bn = bn;
    a.H = g.H; a.W = g.W; a.Wo = g.Wo; a.HoWo = g.Ho * g.Wo; a.M = g.N * a.HoWo;
    a.nCib = g.Ci / 16; a.nCob = g.Co / 16; a.taps = g.kh * g.kw; a.kw = g.kw;
    a.stride = g.stride; a.pt = g.pt; a.pl = g.pl; a.steps = a.nCib * a.taps;
    const int v = pick_variant(g);
    const bool taps = taps_inside(g, v);
    a.run = (a.steps + kVariants[v].waves - 1) / kVariants[v].waves;
    a.n_groups = (a.M + 16 * kVariants[v].wm - 1) / (16 * kVariants[v].wm);
    a.epilogue = epilogue;
    a.in_bytes = (unsigned)((size_t)g.N * g.Ci * g.H * g.W * 4);
    a.filt_bytes = (unsigned)((size_t)g.Co * g.Ci * a.taps * 4);
    a.dHoWo = make_fastdiv(a.HoWo); a.dWo = make_fastdiv(a.Wo); a.dCib = make_fastdiv(a.nCib); a.dTaps = make_fastdiv(a.taps); a.dKw = make_fastdiv(a.kw);
    a.dGroups = make_fastdiv(a.n_groups);
    switch (v) {
        case 0: return run<16, 1, 1>(a, taps, s);
        case 1: return run<8, 1, 1>(a, taps, s);
        case 2: return run<4, 1, 1>(a, taps, s);
        case 3: return run<4, 2, 1>(a, taps, s);
        case 4: return run<4, 2, 2>(a, taps, s);
        default: return run<2, 2, 2>(a, taps, s);
    }
}

}  // namespace small
