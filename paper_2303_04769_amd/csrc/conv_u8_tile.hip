// Quantized convolution through LDS tiles: any window larger than one pixel, 16-byte blocks, the 8-bit matrix cores.
//
// A workgroup (4 waves) owns TM consecutive output pixels of the flattened (image, row, column) axis and TN output
// channels. What bounds the register-only kernels of quant.hip is vector instructions: every operand is made signed
// (bit 7 flipped) and tested against the image's edge each time it is read, nine times per value under a 3x3 window and
// once per wave. Here a value is brought into LDS once per workgroup, already signed and with the padding filled in, and
// the reduction loop is LDS reads and matrix instructions only:
//   - the input rows under the tile are staged as "virtual" rows: an image has Hv = (Ho - 1) stride + kh of them (its
//     padding included), images are stacked, a row has Wv = (Wo - 1) stride + kw entries, so a tile may cross rows and
//     images and still reads one contiguous range of virtual rows, and the entry of a pixel under filter tap (y, x) is
//     the pixel's own entry plus the constant y Wv + x. Where each entry comes from is worked out once per workgroup.
//   - one v_mfma_i32_16x16x64_i8 takes four 16-byte chunks (lane group g one each): `bpc` input blocks of 4 / bpc
//     neighbouring taps, bpc = 4, 2 or 1, chosen on the host for the fewest instructions (a layer on 16 channels would
//     fill a quarter of an instruction that took blocks alone).
//   - the filter comes in by phases of kTG steps: the next phase's filter and the next chunk's input are requested into
//     registers before the current matrix instructions and written over the current ones behind them. One LDS buffer and
//     two barriers: with two buffers and one barrier half as many workgroups fit a compute unit and nothing covers a
//     wave's waiting (128 channels 28 x 28 x 64 images: 23.5 us, 16.5 with one).
//   - the code is free of branches around loads and LDS writes, and a wave's tile as large as the work allows: the time is
//     issue slots and waiting, not matrix instructions (8.8 of some 30 thousand cycles per SIMD on that layer, now 13.6 us; 15.2
//     with zw != 128).
// The correction sums of the zero points are those of quant.hip; the constant part (K a b and the filter's sums) is the
// accumulators' initial value. Layers whose filter sums the caller did not give (zx != 128) and scales that need the wide
// requantization stay with quant.hip: code that is rarely run would lie between the code that is, and a workgroup that
// lives for some ten microseconds pays for every line of instructions it fetches.
#include "small_internal.h"

#include <type_traits>

namespace small {
namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));

constexpr int kTG = 3;                 // steps of a phase
constexpr int kMaxTaps = 64, kTapSlots = kMaxTaps + 4 * kTG;
constexpr int tile_rounds(int tm) { return tm >= 256 ? 8 : tm >= 128 ? 6 : 5; }     // ... and a chunk, at most

struct QTileArgs {
    const unsigned char *in, *filt;
    unsigned char *out;
    const int *filt_sums;
    int H, W, Ho, Wo, HoWo;
    int Ws, strips, HoWs, M;              // a strip's columns, strips per image, pixels of a strip, pixels of all strips
    int nCib, nCob, taps, kw, kh, pt, pl;
    int l2bpc, phases, F, n_chunks;       // phases of a chunk of bpc input blocks, of all of them
    int Hv, Wv, stride;
    int E, Epad;                          // staged entries: the most any tile needs; room for the whole rounds of a thread
    int n_cot;                            // channel tiles
    unsigned in_bytes, filt_bytes, out_bytes;     // each below 2 GiB
    FastDiv dHoWs, dWs, dWv, dHv, dStrips, dCt, dkw;
    QuantParams q;
};

// The arguments as the kernel finds them in memory. Read again from there, behind a place that the compiler cannot see through,
// they need not be kept in scalar registers (or, spilled, in a vector register's lanes: 50 of them, and 120 lane reads and writes)
// across the reduction: 64 channels 56 x 56 x 64 images 18.9 -> 17.7 us, 128 channels 28 x 28 x 64 14.6 -> 14.1.
typedef const __attribute__((address_space(4))) QTileArgs *QTileKernArgs;
__device__ __forceinline__ QTileKernArgs args_again()
{
    QTileKernArgs ka = (QTileKernArgs)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(ka));
    return ka;
}
__device__ __forceinline__ FastDiv fastdiv_at(const __attribute__((address_space(4))) FastDiv &f)
{
    FastDiv r;
    r.magic = f.magic; r.shift = f.shift; r.d = f.d;
    return r;
}

// STREAM: see streams()
template <int WM, int WN, int WVM, int WVN, int CORR, bool STREAM>
__global__ void __launch_bounds__(256, WM * WN >= 16 ? 2 : WM * WN >= 8 ? 3 : 4) conv_u8_tile(QTileArgs a)
{
    constexpr int TM = 16 * WM * WVM, NCT = WN * WVN;          // pixels, 16-channel blocks of a workgroup
    constexpr int UNITS = kTG * NCT, FI = (UNITS + 3) / 4;     // (step, block) filter operands of a phase, per wave
    constexpr int ROUNDS = tile_rounds(TM);
    static_assert(WVM * WVN == 4, "four waves");
    constexpr bool use_s = CORR == 1;
    static_assert(!STREAM || WM * WN % 4 == 0, "words of a block are not streamed");

    extern __shared__ intx4 lds[];
    int *tapoff = reinterpret_cast<int *>(lds);
    unsigned *etab = reinterpret_cast<unsigned *>(tapoff + kTapSlots);
    intx4 *A = lds + (kTapSlots + a.Epad) / 4;
    intx4 *B = A + 4 * FI * 64;
    const int plane_e = a.E + 1;                               // entries of a staged block; the last one is a dump

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = lane & 15, g = lane >> 4;
    const int wave_m = wave % WVM, wave_n = wave / WVM;
    const int wg = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    const int mt = quotient(a.dCt, wg), cob0 = (wg - mt * a.n_cot) * NCT;
    const int m0 = mt * TM;
    const int bpc = 1 << a.l2bpc;
    const int flip = (int)0x80808080u, pad = (a.q.zx * 0x01010101) ^ flip;
    // Both operands are read through buffer descriptors: what lies outside (padding, channels past the last block, work
    // past the last phase) has an offset beyond the descriptor and reads as zero, and one select gives the word that turns
    // a value read into the signed operand: flip, the padding's code (over zero), or zero. No load and no LDS write sits
    // under a branch (the compiler would wait for each in turn): what has no place goes to the dump entry.
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(a.in), 0, a.in_bytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t flt = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(a.filt), 0, a.filt_bytes, kRawBuffer);

    // ---- filter staging: unit u = (step of the phase, block), a wave's units are wave, wave + 4, ...; lane (p, g) brings
    // the 16 input channels of output channel p that lane group g multiplies.
    const int l2tps = 2 - a.l2bpc, gb = g & (bpc - 1), gt = g >> a.l2bpc;
    struct Filter { intx4 v[FI]; int x[FI]; };
    const unsigned f_lane = (unsigned)((gb * a.taps + gt) * 256 + p * 16);
    auto f_load = [&](int ch, int ph, bool more, Filter &f) __attribute__((always_inline)) {
        const bool lane_ok = more & ((ch << a.l2bpc) + gb < a.nCib);
#pragma unroll
        for (int i = 0; i < FI; ++i) {
            const int u = wave + 4 * i;
            const int st = u / NCT, cob = cob0 + u - st * NCT;
            const int tap0 = (ph * kTG + st) << l2tps;
            const bool ok = lane_ok & (cob < a.nCob) & (tap0 + gt < a.taps);
            const int at = ((cob * a.nCib + (ch << a.l2bpc)) * a.taps + tap0) * 256;      // wave-uniform
            f.v[i] = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(flt, ok ? f_lane + (unsigned)at : kBeyond, 0, 0));
            f.x[i] = ok ? flip : 0;
        }
    };
    auto f_store = [&](const Filter &f) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FI; ++i) A[(wave + 4 * i) * 64 + lane] = f.v[i] ^ f.x[i];
    };
    Filter f0;
    f_load(0, 0, true, f0);

    // ---- the tile's range of virtual rows, and the first chunk: a thread serves block sblk of a chunk, entries
    // se + k * er of round k. Where an entry comes from (byte offset of its pixel in block 0) is kept in LDS.
    const int n0 = quotient(a.dHoWs, m0), vr0 = n0 * a.Hv + quotient(a.dWs, m0 - n0 * a.HoWs) * a.stride;
    const int m1 = min(m0 + TM, a.M) - 1;
    const int n1 = quotient(a.dHoWs, m1), vr1 = n1 * a.Hv + quotient(a.dWs, m1 - n1 * a.HoWs) * a.stride + a.kh - 1;
    const int nE = (vr1 - vr0 + 1) * a.Wv;
    const int sblk = (tid >> 4) & (bpc - 1), se = (tid & 15) + 16 * ((tid >> 4) >> a.l2bpc), er = 256 >> a.l2bpc;
    const unsigned plane = (unsigned)(a.H * a.W) * 16u;
    {
        const bool live = sblk < a.nCib;
        intx4 v[ROUNDS];
        int x[ROUNDS];
        unsigned at[ROUNDS];
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k) {
            const int e = se + k * er;
            const int row = quotient(a.dWv, e), vr = vr0 + row, ns = quotient(a.dHv, vr), iy = vr - ns * a.Hv - a.pt;
            const int n = quotient(a.dStrips, ns), strip = ns - n * a.strips;
            const int ix = e - row * a.Wv + strip * a.Ws * a.stride - a.pl;
            const bool inside = (e < nE) & ((unsigned)iy < (unsigned)a.H) & ((unsigned)ix < (unsigned)a.W);
            at[k] = inside ? (unsigned)((n * a.nCib * a.H + iy) * a.W + ix) * 16u : kBeyond;
            v[k] = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(src, (inside & live) ? at[k] + sblk * plane : kBeyond, 0, 0));
            x[k] = live ? (inside ? flip : pad) : 0;
        }
        if (tid < kTapSlots) {
            const int y = quotient(a.dkw, tid);
            tapoff[tid] = tid < a.taps ? (y * a.Wv + tid - y * a.kw) * 16 : 0;
        }
        intx4 *dst = B + sblk * plane_e;
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k) {
            const int e = se + k * er;
            if (sblk == 0 && e < a.Epad) etab[e] = at[k];
            dst[e < nE ? e : a.E] = v[k] ^ x[k];
        }
    }
    f_store(f0);

    // the chunks after the first
    intx4 iv[ROUNDS];
    auto in_load = [&](int ch) __attribute__((always_inline)) {
        const bool live = (ch << a.l2bpc) + sblk < a.nCib;                               // (false past the last chunk)
        const unsigned lane_at = live ? sblk * plane + (unsigned)(ch << a.l2bpc) * plane : kBeyond;
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k) {
            const unsigned at = etab[min(se + k * er, a.Epad - 1)];
            iv[k] = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(src, max(at, lane_at) >= kBeyond ? kBeyond : at + lane_at, 0, 0));
        }
    };
    auto in_store = [&](int ch) __attribute__((always_inline)) {
        const bool live = (ch << a.l2bpc) + sblk < a.nCib;
        const int x_in = live ? flip : 0, x_out = live ? pad : 0;
        intx4 *dst = B + sblk * plane_e;
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k) {
            const int e = se + k * er;
            const int x = etab[min(e, a.Epad - 1)] != kBeyond ? x_in : x_out;
            dst[e < nE ? e : a.E] = iv[k] ^ x;
        }
    };

    // ---- this lane's pixels
    int base[WM];
#pragma unroll
    for (int wm = 0; wm < WM; ++wm) {
        const int m = min(m0 + (wave_m * WM + wm) * 16 + p, a.M - 1);
        const int n = quotient(a.dHoWs, m), rem = m - n * a.HoWs, oh = quotient(a.dWs, rem);
        base[wm] = (gb * plane_e + (n * a.Hv + oh * a.stride - vr0) * a.Wv + (rem - oh * a.Ws) * a.stride) * 16;
    }

    // ---- accumulators start at K a b - a * (sum of the channel's signed filter bytes)
    const int za = a.q.zx - 128, zb = a.q.zw - 128;
    const int K = a.nCib * 16 * a.taps;
    const __amdgpu_buffer_rsrc_t sum = __builtin_amdgcn_make_buffer_rsrc(const_cast<int *>(a.filt_sums), 0, a.filt_sums ? a.nCob * 64 : 0, kRawBuffer);
    intx4 acc[WM][WN], acc_s[WM];
#pragma unroll
    for (int wn = 0; wn < WN; ++wn) {
        const unsigned kab = (unsigned)K * (unsigned)(za * zb);
        // (without sums zx is 128, za is 0, and the empty descriptor reads zeros)
        const intx4 s = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(sum, ((cob0 + wave_n * WN + wn) * 16 + 4 * g) * 4, 0, 0));
        intx4 c;
#pragma unroll
        for (int r = 0; r < 4; ++r) c[r] = (int)(kab - (unsigned)za * ((unsigned)s[r] - (unsigned)K * 128u));
#pragma unroll
        for (int wm = 0; wm < WM; ++wm) acc[wm][wn] = c;
    }
#pragma unroll
    for (int wm = 0; wm < WM; ++wm) acc_s[wm] = intx4{0, 0, 0, 0};
    __syncthreads();                                       // tables and first operands

    // ---- reduction: chunk ch of input blocks, phase ph of its steps. The filter of the next phase and the input of the
    // next chunk are requested before the matrix instructions and written over the current ones behind them.
    int f = 0;
    for (int ch = 0; ch < a.n_chunks; ++ch) {
        if (ch + 1 < a.n_chunks) in_load(ch + 1);          // (64 channels 56 x 56 x 64 images, one chunk: 17.1 -> 16.6 us)
        for (int ph = 0; ph < a.phases; ++ph, ++f) {
            const bool last_ph = ph + 1 == a.phases;
            f_load(last_ph ? ch + 1 : ch, last_ph ? 0 : ph + 1, f + 1 < a.F, f0);
            __builtin_amdgcn_sched_barrier(0);             // the requests stay ahead of the matrix instructions
            const intx4 *Af = A + wave_n * WN * 64 + lane;
            int off[kTG];
#pragma unroll
            for (int st = 0; st < kTG; ++st) off[st] = tapoff[((ph * kTG + st) << l2tps) + gt];
#pragma unroll
            for (int st = 0; st < kTG; ++st) {
                intx4 fa[WN], fb[WM];
#pragma unroll
                for (int wn = 0; wn < WN; ++wn) fa[wn] = Af[(st * NCT + wn) * 64];
#pragma unroll
                for (int wm = 0; wm < WM; ++wm) fb[wm] = *reinterpret_cast<const intx4 *>(reinterpret_cast<const char *>(B) + base[wm] + off[st]);
                // steps past the chunk's last one and taps past the window multiply zeros (and must not count in the sums)
                const int one = ((ph * kTG + st) << l2tps) + gt < a.taps ? 0x01010101 : 0;
                const intx4 ones = {one, one, one, one};
#pragma unroll
                for (int wm = 0; wm < WM; ++wm) {
#pragma unroll
                    for (int wn = 0; wn < WN; ++wn)
                        acc[wm][wn] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[wn], fb[wm], acc[wm][wn], 0, 0, 0);
                    if (use_s) acc_s[wm] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, fb[wm], acc_s[wm], 0, 0, 0);
                }
            }
            if (f + 1 == a.F) break;
            __syncthreads();
            f_store(f0);
            if (last_ph) in_store(ch + 1);
            __syncthreads();
        }
    }

    // ---- zero-point correction of the pixel, requantization, store. Lane (p, g) has words of four channels (4g ..) of WM
    // pixels and WN blocks; four such words are transposed across the lane groups so that group g holds the whole 16-byte
    // block of the g-th one and a store instruction writes a kilobyte instead of a quarter.
    const QTileKernArgs b = args_again();
    QuantParams q;
    q.zy = b->q.zy; q.mult = b->q.mult; q.shift = b->q.shift; q.lo = b->q.lo; q.hi = b->q.hi; q.amax = b->q.amax; q.mult32 = b->q.mult32;
    const FastDiv dHoWs = fastdiv_at(b->dHoWs), dWs = fastdiv_at(b->dWs), dStrips = fastdiv_at(b->dStrips);
    const int M = b->M, HoWs = b->HoWs, Ws = b->Ws, strips = b->strips, Wo = b->Wo, HoWo = b->HoWo, nCob = b->nCob;
    const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(b->out, 0, b->out_bytes, kRawBuffer);
    auto store = [&](auto high) __attribute__((always_inline)) {
        constexpr bool HIGH = decltype(high)::value;
        const long addend = requant_addend<HIGH>(q);
        auto word = [&](int wm, int wn) __attribute__((always_inline)) {
            const unsigned px = use_s ? (unsigned)(zb * acc_s[wm][0]) : 0u;
            unsigned y[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = (unsigned)requant_code<HIGH>((int)((unsigned)acc[wm][wn][r] - px), q, addend);
            return y[0] | y[1] << 8 | y[2] << 16 | y[3] << 24;
        };
        // byte offset of (pixel wm of this lane, block wn) in the output, or kBeyond
        auto place = [&](int wm, int wn) __attribute__((always_inline)) {
            const int m = m0 + (wave_m * WM + wm) * 16 + p, cob = cob0 + wave_n * WN + wn;
            const int ns = quotient(dHoWs, min(m, M - 1)), rem = m - ns * HoWs, oh = quotient(dWs, rem);
            const int n = quotient(dStrips, ns), ow = rem - oh * Ws + (ns - n * strips) * Ws;
            const bool ok = (m < M) & (ow < Wo) & (cob < nCob);
            return (unsigned)((n * nCob + cob) * HoWo + oh * Wo + ow) * 16u | (kBeyond & ~lane_mask(ok));
        };
        if constexpr (WM * WN % 4 == 0) {
#pragma unroll
            for (int c = 0; c < WM * WN / 4; ++c) {
                unsigned w[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) w[k] = word((4 * c + k) / WN, (4 * c + k) % WN);
                // (swap16: odd rows of 16 lanes of the first with even rows of the second; swap32: halves likewise)
                auto t01 = __builtin_amdgcn_permlane16_swap(w[0], w[1], false, false);
                auto t23 = __builtin_amdgcn_permlane16_swap(w[2], w[3], false, false);
                auto e = __builtin_amdgcn_permlane32_swap(t01[0], t23[0], false, false);
                auto o = __builtin_amdgcn_permlane32_swap(t01[1], t23[1], false, false);
                const uintx4 v = {e[0], o[0], e[1], o[1]};
                const int j = 4 * c + g;
                __builtin_amdgcn_raw_buffer_store_b128(v, dst, place(WN == 4 ? c : j / WN, WN == 4 ? g : j % WN), 0, STREAM ? kNonTemporal : 0);
            }
        } else {
#pragma unroll
            for (int wm = 0; wm < WM; ++wm)
#pragma unroll
                for (int wn = 0; wn < WN; ++wn) __builtin_amdgcn_raw_buffer_store_b32(word(wm, wn), dst, place(wm, wn) + 4u * g, 0, 0);
        }
    };
    if (q.mult32 >= 0) store(std::true_type());
    else store(std::false_type());
}

// Tiles: pixel groups and blocks of a wave, waves along pixels and channels; cycles of a step of one workgroup alone on its
// compute unit, and what a further workgroup beside it adds to that time (both measured, on 384 channels of 29 x 7 images
// and 128 channels of 28 x 28): small tiles wait more than they work, large ones share the time.
struct Tile { int wm, wn, wvm, wvn; double step, beside; };
constexpr Tile kTiles[] = {{4, 4, 4, 1, 890, 0.80}, {4, 4, 2, 2, 990, 0.80}, {2, 4, 4, 1, 650, 0.68}, {2, 4, 2, 2, 740, 0.70},
                           {2, 2, 2, 2, 560, 0.50}, {1, 2, 2, 2, 530, 0.50}, {4, 2, 4, 1, 700, 0.60}, {2, 2, 4, 1, 530, 0.50},
                           {4, 1, 4, 1, 700, 0.60}, {2, 1, 4, 1, 440, 0.45}};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);
constexpr size_t kMaxLds = 160 * 1024;

template <auto Kernel>
hipError_t run(dim3 grid, size_t lds, hipStream_t s, const QTileArgs &a)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(Kernel),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(Kernel, grid, dim3(256), lds, s, a);
    return hipGetLastError();
}

// An image is cut into strips of at most 32 output columns (16 under a stride), as even as can be, so that the rows under a
// tile stay short; strips are laid out one after the other like images.
void strip_split(const LayerGeom &g, int &strips, int &Ws)
{
    const int most = g.stride == 1 ? 32 : 16;
    strips = (g.Wo + most - 1) / most;
    Ws = (g.Wo + strips - 1) / strips;
}

// The most staged entries a tile of tm pixels needs.
long tile_entries(const LayerGeom &g, int tm, int strips, int Ws)
{
    const long pixels = (long)g.N * strips * g.Ho * Ws;
    const long span = (tm < pixels ? tm : pixels) - 1;
    const long rows = (span + Ws - 1) / Ws + 1;                                             // output rows touched
    const long cross = (long)g.N * strips > 1 ? (rows - 1 + g.Ho - 1) / g.Ho : 0;           // boundaries of strips among them
    const long vrows = (rows - 1) * g.stride + g.kh + (g.kh > g.stride ? cross * (g.kh - g.stride) : 0);
    return vrows * ((Ws - 1) * g.stride + g.kw);
}

struct Plan { int tile, l2bpc, phases, n_chunks, strips, Ws; long E, Epad; size_t lds; };

// Tile and reduction order, or tile = -1: the candidate with the shortest time of the fullest compute unit.
Plan plan_tile(const LayerGeom &g)
{
    Plan best;
    best.tile = -1;
    const int taps = g.kh * g.kw, nCib = g.Ci / 16, nCob = g.Co / 16;
    const int Hv = (g.Ho - 1) * g.stride + g.kh;
    int strips, Ws;
    strip_split(g, strips, Ws);
    const long M = (long)g.N * strips * g.Ho * Ws;
    if (taps < 2 || taps > kMaxTaps || ((long)g.N * strips + 1) * Hv >= (1L << 31) || M >= (1L << 31) - 512 ||
        (long)g.N * nCib * g.H * g.W * 16 >= (long)kBeyond || (long)g.N * nCob * g.Ho * g.Wo * 16 >= (long)kBeyond || (long)nCob * nCib * taps * 256 >= (long)kBeyond)
        return best;
    int l2bpc = 2, steps = 0, n_chunks = 0;
    for (int l = 2; l >= 0; --l) {
        const int c = (nCib + (1 << l) - 1) >> l, s = (taps + (4 >> l) - 1) / (4 >> l);
        if (l == 2 || c * s < n_chunks * steps) { l2bpc = l; steps = s; n_chunks = c; }
    }
    const int phases = (steps + kTG - 1) / kTG;
    double best_cost = 0;
    const long cus = device_cus();
    for (int t = 0; t < kNumTiles; ++t) {
        const Tile &k = kTiles[t];
        const int tm = 16 * k.wm * k.wvm, nct = k.wn * k.wvn, er = 256 >> l2bpc;
        const long E = tile_entries(g, tm, strips, Ws);
        const long rounds = (E + er - 1) / er, Epad = rounds * er;
        const size_t lds = (size_t)(kTapSlots + Epad) * 4 + (size_t)((kTG * nct + 3) / 4) * 4096 + ((size_t)(E + 1) << l2bpc) * 16;
        if (lds > kMaxLds || rounds > tile_rounds(tm)) continue;
        const long wgs = ((M + tm - 1) / tm) * ((nCob + nct - 1) / nct);
        const double alone = (double)n_chunks * phases * kTG * k.step + 3000.0 + 200.0 * k.wm * k.wn;
        const double cost = alone * (1.0 + k.beside * (double)((wgs + cus - 1) / cus - 1));
        if (best.tile < 0 || cost < best_cost) {
            best_cost = cost;
            best = Plan{t, l2bpc, phases, n_chunks, strips, Ws, E, Epad, lds};
        }
    }
    return best;
}

// Where the register-only kernels of quant.hip stay the better ones: reductions of at most 20 chunks, which their short form
// holds in registers whole (16 channels 32 x 32 x 100 images 5.3 us there, 6.6 here; 32 channels 16 x 16 x 100 4.0 / 4.9) unless they
// are large (large_short), and where the two models below say so. They are fitted to 3300 measured pairs of layer and tile (us, before both
// sides lost 3 to 12 % of their time by a shorter requantization; 3 to 8 % root mean square for
// the tiles, 7 to 13 for the kernels there), w being the workgroups of the fullest compute unit:
//   here   3.0 + a w + phases (b + c w) + chunks (d + e w)       a phase: kTG steps; a chunk: input brought in and two barriers
//   there  3.5 + a w + steps (b + c w) + d passes               a step: one matrix instruction of four 16-byte chunks per tile;
//          a pass: every megabyte of input beyond four read once more, per window row and group of output blocks
// On 900 fresh random layers the rule leaves 23 more than 3 % slower than there, eight of them by 10 to 31 % (rules on sizes alone
// left 184, by up to 1.9 times: windows of two or three taps on many channels bring in a chunk for a single phase, and few channels out share it
// with few others). us there / here: 128 channels 28 x 28 x 64 images 22.7 / 16.5, 64 channels 56 x 56 x 64 25.9 / 20.8, 240 -> 64
// channels 57 x 57 x 5 28.1 / 14.9, 112 channels 10 x 10 x 76 11.6 / 7.5; not taken: 272 -> 128 2 x 2 14 x 14 x 102 19.3 / 35.3,
// 512 -> 48 1 x 3 35 x 35 x 12 9.2 / 13.4, 128 -> 16 3 x 3 stride 2 47 x 91 x 14 6.7 / 8.8, 512 channels 7 x 7 x 64 23.9 / 25.4.
struct Rate { double a, b, c, d, e; };
constexpr Rate kHere[kNumTiles] = {{2.88, 0.43, 0.38, 0.34, 0.51}, {2.56, 0.47, 0.56, 0.20, 0.40}, {1.42, 0.33, 0.30, 0.43, 0.26},
                                   {1.68, 0.51, 0.35, 0.35, 0.13}, {0.86, 0.32, 0.23, 0.43, 0.15}, {0.67, 0.34, 0.17, 0.48, 0.14},
                                   {1.79, 0.39, 0.25, 0.68, 0.21}, {1.06, 0.31, 0.19, 0.52, 0.16}, {1.07, 0.38, 0.19, 0.67, 0.22},
                                   {0.75, 0.25, 0.13, 0.56, 0.18}};
// [input blocks a multiple of four][output blocks of a workgroup: 1, 2, 4]
constexpr Rate kThere[2][3] = {{{0.74, 0.34, 0.093, 0.016, 0}, {1.10, 0.36, 0.110, 0.013, 0}, {1.97, 0.55, 0.091, 0.042, 0}},
                               {{0.39, 0.086, 0.085, 0.054, 0}, {0.64, 0.062, 0.120, 0.043, 0}, {1.34, 0.060, 0.168, 0.052, 0}}};

// Short reductions, 3x3 windows on 16 or 32 channels, that are better here all the same: there a workgroup has one, two or four
// output blocks, by what divides their number, and reads its window, makes it signed and looks at the edge once more for each such
// group, so the more groups and pixels the more that costs. By pixels x groups of the layer in thousands per compute unit, 210 random
// layers of up to 2 M pixels, us here / there. Three, five, ... blocks (groups of one) on 32 channels: 8.5 / 7.7 at 0.78, 8.1 / 10.1 at
// 1.16 (184 images, 112 channels out, 41x21 stride 2), 14.9 / 20.2 at 2.6, 33.9 / 54.1 at 8.4; on 16 channels 7.9 / 7.1 at 0.92, 10.4 /
// 11.4 at 2.0, 15.9 / 21.8 at 4.0. On 32 channels with stride 1 also groups of four (16.5 / 15.8 at 0.85, 16.7 / 18.0 at 0.96), groups of two
// (11.7 / 11.3 at 0.9, 13.3 / 14.7 at 1.5) and a single block (14.8 / 15.3 at 2.2); with stride 2 those are not (15.6 / 12.9 at 1.2, two
// blocks), and on 16 channels groups of two and four take 1.0 to 1.2 times as long here. Nor are groups of two whose filter has another
// zero point than 128, where the tiles sum up the codes with matrix instructions: 0.95 to 1.07 of the time there (32 channels 43x104, 106
// images 19.1 / 17.8), 0.86 to 0.97 without. 440 random layers that changed: 0.78 of the time, none of the taken ones more than 4 % longer.
bool large_short(const LayerGeom &g, bool plain_filter, long cus)
{
    const int nCob = g.Co / 16, group = nCob % 4 == 0 ? 4 : nCob % 2 == 0 ? 2 : 1;
    if (g.kh != 3 || g.kw != 3) return false;
    const long passes = (long)g.N * g.Ho * g.Wo * (nCob / group);
    if (group == 1 && nCob > 1) return passes >= (g.Ci == 32 ? 940 : 1950) * cus;
    if (g.Ci != 32 || g.stride != 1 || (group == 2 && !plain_filter)) return false;
    return passes >= (group == 4 ? 900 : group == 2 ? 1500 : 1950) * cus;
}

bool better_in_registers(const LayerGeom &g, const Plan &pl, bool plain_filter)
{
    const int nCib = g.Ci / 16, nCob = g.Co / 16, taps = g.kh * g.kw;
    const long cus = device_cus();
    if (nCib * taps <= 20) return !large_short(g, plain_filter, cus);
    // workgroups of the fullest compute unit; many are as good as spread evenly
    auto fullest = [&](long wgs) { return wgs < 4 * cus ? (double)((wgs + cus - 1) / cus) : (double)wgs / cus; };
    const Tile &k = kTiles[pl.tile];
    const int tm = 16 * k.wm * k.wvm, nct = k.wn * k.wvn;
    const double w = fullest(((long)g.N * pl.strips * g.Ho * pl.Ws + tm - 1) / tm * ((nCob + nct - 1) / nct));
    const Rate &h = kHere[pl.tile];
    const double here = 3.0 + h.a * w + pl.n_chunks * (pl.phases * (h.b + h.c * w) + h.d + h.e * w);
    const int wn = nCob % 4 == 0 ? 4 : nCob % 2 == 0 ? 2 : 1;
    const double v = fullest(((long)g.N * g.Ho * g.Wo + 127) / 128 * (nCob / wn));
    const Rate &t = kThere[nCib % 4 == 0][wn / 2];
    const double mb = 1e-6 * (double)g.N * g.Ci * g.H * g.W - 4.0, passes = mb > 0 ? mb * (nCob / wn) * g.kh : 0.0;
    const double there = 3.5 + t.a * v + (double)((nCib * taps + 3) / 4) * (t.b + t.c * v) + t.d * passes;
    return here >= there;
}

// Outputs of 4 MB and more are stored non-temporally: 0.94 to 1.0 of the time over 27 random layers (64 channels 56 x 56 x 64 images
// 16.6 -> 15.6 us, 128 channels 28 x 28 x 64 15.1 -> 14.8); smaller ones 0.97 to 1.06. That is by the tiles whose waves write whole
// 16-byte blocks; the two smallest ones (5 and 9), which write a word of a block per lane, store through the cache.
bool streams(const Tile &t, const LayerGeom &g)
{
    return t.wm * t.wn % 4 == 0 && (size_t)g.N * g.Co * g.Ho * g.Wo >= (4u << 20);
}

}  // namespace

bool conv_u8_tile_eligible(const LayerGeom &g, const QuantParams &q, const int *filt_sums, const void *out)
{
    if (((uintptr_t)out & 15u) != 0 || q.amax <= 0 || (!filt_sums && q.zx != 128)) return false;
    const Plan pl = plan_tile(g);
    return pl.tile >= 0 && !better_in_registers(g, pl, q.zw == 128);
}

TileForm conv_u8_tile_form(const LayerGeom &g)
{
    const Plan pl = plan_tile(g);
    return {pl.tile, pl.tile >= 0 && streams(kTiles[pl.tile], g)};
}

hipError_t launch_conv_u8_tile(const unsigned char *in, const unsigned char *filt, unsigned char *out, const LayerGeom &g,
                               const QuantParams &q, const int *filt_sums, hipStream_t s)
{
    const int corr = q.zw != 128 ? 1 : 0;
    const Plan pl = plan_tile(g);
    if (pl.tile < 0) return hipErrorInvalidValue;
    const Tile &t = kTiles[pl.tile];
    QTileArgs a;
    a.in = in; a.filt = filt; a.out = out; a.filt_sums = filt_sums;
    a.H = g.H; a.W = g.W; a.Ho = g.Ho; a.Wo = g.Wo; a.HoWo = g.Ho * g.Wo;
    a.Ws = pl.Ws; a.strips = pl.strips; a.HoWs = g.Ho * pl.Ws; a.M = g.N * pl.strips * a.HoWs;
    a.nCib = g.Ci / 16; a.nCob = g.Co / 16; a.taps = g.kh * g.kw; a.kh = g.kh; a.kw = g.kw; a.pt = g.pt; a.pl = g.pl;
    a.l2bpc = pl.l2bpc; a.phases = pl.phases; a.n_chunks = pl.n_chunks; a.F = pl.phases * pl.n_chunks;
    a.stride = g.stride;
    a.Hv = (g.Ho - 1) * g.stride + g.kh; a.Wv = (pl.Ws - 1) * g.stride + g.kw;
    a.E = (int)pl.E; a.Epad = (int)pl.Epad;
    a.in_bytes = (unsigned)((size_t)g.N * g.Ci * g.H * g.W); a.filt_bytes = (unsigned)((size_t)g.Co * g.Ci * a.taps);
    a.out_bytes = (unsigned)((size_t)g.N * g.Co * a.HoWo);
    const int tm = 16 * t.wm * t.wvm, nct = t.wn * t.wvn;
    a.n_cot = (a.nCob + nct - 1) / nct;
    a.dHoWs = make_fastdiv(a.HoWs); a.dWs = make_fastdiv(a.Ws); a.dWv = make_fastdiv(a.Wv); a.dHv = make_fastdiv(a.Hv);
    a.dStrips = make_fastdiv(a.strips); a.dCt = make_fastdiv(a.n_cot); a.dkw = make_fastdiv(a.kw);
    a.q = q;
    const dim3 grid((unsigned)((a.M + tm - 1) / tm * a.n_cot));
    const bool stream = streams(t, g);
#define SMALL_TILE_CASE(I_, M_, N_, VM_, VN_)                                                   \
    case I_:                                                                                    \
        if (!stream && corr == 0) return run<conv_u8_tile<M_, N_, VM_, VN_, 0, false>>(grid, pl.lds, s, a);  \
        if (!stream) return run<conv_u8_tile<M_, N_, VM_, VN_, 1, false>>(grid, pl.lds, s, a);  \
        if (corr == 0) return run<conv_u8_tile<M_, N_, VM_, VN_, 0, M_ * N_ % 4 == 0>>(grid, pl.lds, s, a); \
        return run<conv_u8_tile<M_, N_, VM_, VN_, 1, M_ * N_ % 4 == 0>>(grid, pl.lds, s, a);
    switch (pl.tile) {
        SMALL_TILE_CASE(0, 4, 4, 4, 1)
        SMALL_TILE_CASE(1, 4, 4, 2, 2)
        SMALL_TILE_CASE(2, 2, 4, 4, 1)
        SMALL_TILE_CASE(3, 2, 4, 2, 2)
        SMALL_TILE_CASE(4, 2, 2, 2, 2)
        SMALL_TILE_CASE(5, 1, 2, 2, 2)
        SMALL_TILE_CASE(6, 4, 2, 4, 1)
        SMALL_TILE_CASE(7, 2, 2, 4, 1)
        SMALL_TILE_CASE(8, 4, 1, 4, 1)
        SMALL_TILE_CASE(9, 2, 1, 4, 1)
    }
#undef SMALL_TILE_CASE
    return hipErrorInvalidValue;
}

}  // namespace small
