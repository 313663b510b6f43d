// fp32 convolution on the bf16 matrix cores, each value as the sum of three bf16 ones.
//
// A float has 24 significant bits, a bf16 eight: x = h + m + l exactly, with h, m, l the bf16 roundings of x, x - h and
// x - h - m (|m| up to 2^-8 of |x|, |l| up to 2^-17), and six of the nine products of two such sums are taken: hh, hm, mh, mm, hl
// and lh. What is dropped, ml, lm and ll, is up to 2^-24 of a product, as much as rounding it to a float costs. bf16 products are
// exact and the matrix instruction adds them in fp32, 32 at a time. The five small products have sums of their own, added to the
// large ones' once at the end: their roundings are then 2^-8 of what they are in one sum, and the large products are rounded a
// few times per 32 where the fp32 instruction rounds every 4. Error against 64 bits, 2-norm, fp32 instruction / here (64 channels
// 3x3 28x28, 64 images): dense normal filters 4.2e-7 / 1.3e-7 (on rectified inputs 3.1e-7 / 1.0e-7), a tenth of the weights not
// zero 1.4e-7 / 5.5e-8, two weights 3.0e-8 / 2.6e-8, one 2.53e-8 / 2.57e-8 (at most 1.9 instead of 1.0 x 2^-24 of the product: the
// only kind of filter that loses). One sum for all six: 3.7e-7 (3.6e-7 rectified), 2.6e-7, 7.0e-8, 5.4e-8, 2 % faster; with ml and
// lm too 2.53e-8 for one weight and the others unchanged, 11 to 15 % slower.
// The bf16 instruction does sixteen times the work of the fp32 one per cycle, six of them replace it: 2.7 times the matrix rate,
// of which splitting (five and a half vector instructions per value, v_cvt_pk_bf16_f32 rounds two at once) and LDS traffic take
// their share. So every value is split once per workgroup: the tile scheme of conv_u8_tile.hip -- the input rows under TM
// output pixels staged in LDS with their padding, an entry being the 8 channels of half a block, three planes h, m, l of
// each; the filter by steps -- with one matrix instruction per (step, tile, product):
//   a step is one tap of two input blocks, or two taps of one block (a layer on 16 channels, or an odd last block that would
//   leave half of the instruction empty); lane group g takes half g & 1 of the block's channels and block or tap g >> 1.
// Infinities and NaN have no such sum (inf - inf): a workgroup that stages one computes its outputs with the fp32 instruction
// instead, or, where it is a filter value, one by one.
#include "small_internal.h"

namespace small {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr int kMaxTaps = 64, kTapSlots = kMaxTaps + 8;
constexpr int kRounds = 5;             // rounds of staged input entries of a chunk, at most

struct Split3Args {
    const float *in, *filt, *res, *bn;
    float *out;
    int H, W, Ho, Wo, HoWo;
    int Ws, strips, HoWs, M;           // as in conv_u8_tile.hip: columns of a strip, strips per image, pixels of a strip, of all
    int nCib, nCob, taps, kw, kh, pt, pl;
    int l2bpc, steps, n_chunks;        // steps of a chunk of 1 << l2bpc input blocks
    int Hv, Wv, stride;
    int E, Epad, n_cot, epilogue;
    unsigned in_bytes, filt_bytes;     // each below 2 GiB
    FastDiv dHoWs, dWs, dWv, dHv, dStrips, dCt, dkw;
};

// The matrix instruction takes bf16 denormals as zero: without a scale the parts of values below 2^-102 would get lost (2.7e-6
// relative error at 1e-35, 2.7e-4 at 1e-37). Both operands are therefore split at 2^24 times their size, and the sums taken
// back by 2^-48; powers of two, so nothing is rounded by it. Values or sums that overflow at that scale (values above 2^103,
// sums above 2^79) are found and computed like the infinities. (327 us without the scale, 347 with it.)
constexpr float kScale = 16777216.f, kUnscale = 1.f / (16777216.f * 16777216.f);
constexpr float kMost = 0x1.fep127f;   // the largest bf16: a scaled value above may round to an infinity

// Eight values -> their three bf16 parts; `most` becomes their largest magnitude or NaN: a value has no parts if it is not below
// kMost. (One instruction for two values, v_maximum3_f32; seen in the residuals behind the third part it took six.)
__device__ __forceinline__ void split8(floatx4 a, floatx4 b, uintx4 &h, uintx4 &m, uintx4 &l, float &most)
{
    const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        float u = x[2 * k] * kScale, v = x[2 * k + 1] * kScale;
        most = __builtin_elementwise_maximum(most, __builtin_elementwise_maximum(__builtin_fabsf(u), __builtin_fabsf(v)));
        unsigned part[3];
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const bf16x2 r = __builtin_convertvector(floatx2{u, v}, bf16x2);
            part[s] = __builtin_bit_cast(unsigned, r);
            if (s == 2) break;
            u -= __builtin_bit_cast(float, part[s] << 16);
            v -= __builtin_bit_cast(float, part[s] & 0xffff0000u);
        }
        h[k] = part[0]; m[k] = part[1]; l[k] = part[2];
    }
}

template <int WM, int WN, int WVM, int WVN>
__global__ void __launch_bounds__(256, 2) conv16_split3(Split3Args a)
{
    constexpr int TM = 16 * WM * WVM, NCT = WN * WVN;
    constexpr int FI = NCT / 4;                                // filter operands of a step, per wave
    static_assert(WVM * WVN == 4 && NCT % 4 == 0, "four waves, whole filter rounds");

    extern __shared__ uintx4 lds[];
    int *tapoff = reinterpret_cast<int *>(lds);
    int *bad = tapoff + kTapSlots;                             // (four ints)
    unsigned *etab = reinterpret_cast<unsigned *>(bad + 4);
    uintx4 *A = lds + (kTapSlots + 4 + a.Epad) / 4;            // two of [block][part][lane]
    uintx4 *B = A + 2 * NCT * 3 * 64;                          // [part][block, half][entry]
    const int plane_e = a.E + 1;                               // the last entry of a plane is a dump

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = lane & 15, g = lane >> 4;
    const int wave_m = wave % WVM, wave_n = wave / WVM;
    const int wg = (int)xcd_contiguous(blockIdx.x, gridDim.x);
    const int mt = quotient(a.dCt, wg), cob0 = (wg - mt * a.n_cot) * NCT;
    const int m0 = mt * TM;
    const int bpc = 1 << a.l2bpc, planes = 2 * bpc;
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.in), 0, a.in_bytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t flt = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.filt), 0, a.filt_bytes, kRawBuffer);
    float check = 0.f, most = 0.f, most_w = 0.f;               // NaN or infinite: sums; above kMost or NaN: input, filter

    // ---- filter: lane (p, g) brings 8 input channels (half g & 1 of a block) of output channel p, block or tap g >> 1
    const int half = g & 1, sub = g >> 1;
    const int gb = a.l2bpc ? sub : 0, gt = a.l2bpc ? 0 : sub;
    float fv[FI][8];
    auto f_load = [&](int ch, int st, bool more) __attribute__((always_inline)) {
        const int cib = (ch << a.l2bpc) + gb, tap = (st << (1 - a.l2bpc)) + gt;
        const bool lane_ok = more & (cib < a.nCib) & (tap < a.taps);
#pragma unroll
        for (int i = 0; i < FI; ++i) {
            const int cob = cob0 + wave + 4 * i;
            const unsigned at = (lane_ok & (cob < a.nCob)) ? (unsigned)((((cob * a.nCib + cib) * a.taps + tap) * 256 + half * 128 + p) * 4) : kBeyond;
#pragma unroll
            for (int k = 0; k < 8; ++k) fv[i][k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(flt, at + 64u * k, 0, 0));
        }
    };
    auto f_store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < FI; ++i) {
            uintx4 h, m, l;
            split8(floatx4{fv[i][0], fv[i][1], fv[i][2], fv[i][3]}, floatx4{fv[i][4], fv[i][5], fv[i][6], fv[i][7]}, h, m, l, most_w);
            uintx4 *d = A + (buf * NCT + wave + 4 * i) * 3 * 64 + lane;
            d[0] = h; d[64] = m; d[128] = l;
        }
    };
    f_load(0, 0, true);

    // ---- input: a thread serves plane sp (block sp >> 1, half sp & 1), entries se + k er
    const int n0 = quotient(a.dHoWs, m0), vr0 = n0 * a.Hv + quotient(a.dWs, m0 - n0 * a.HoWs) * a.stride;
    const int m1 = min(m0 + TM, a.M) - 1;
    const int n1 = quotient(a.dHoWs, m1), vr1 = n1 * a.Hv + quotient(a.dWs, m1 - n1 * a.HoWs) * a.stride + a.kh - 1;
    const int nE = (vr1 - vr0 + 1) * a.Wv;
    const int sp = (tid >> 4) & (planes - 1), se = (tid & 15) + 16 * ((tid >> 4) >> (a.l2bpc + 1)), er = 128 >> a.l2bpc;
    const unsigned plane_bytes = (unsigned)(a.H * a.W) * 64u;
    floatx4 iv[kRounds][2];
    {
        const int cib = sp >> 1;
#pragma unroll
        for (int k = 0; k < kRounds; ++k) {
            const int e = se + k * er;
            const int row = quotient(a.dWv, e), vr = vr0 + row, ns = quotient(a.dHv, vr), iy = vr - ns * a.Hv - a.pt;
            const int n = quotient(a.dStrips, ns), strip = ns - n * a.strips;
            const int ix = e - row * a.Wv + strip * a.Ws * a.stride - a.pl;
            const bool inside = (e < nE) & ((unsigned)iy < (unsigned)a.H) & ((unsigned)ix < (unsigned)a.W);
            const unsigned at = inside ? (unsigned)((n * a.nCib * a.H + iy) * a.W + ix) * 64u : kBeyond;
            const unsigned mine = (inside & (cib < a.nCib)) ? at + cib * plane_bytes + (sp & 1) * 32u : kBeyond;
            iv[k][0] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, mine, 0, 0));
            iv[k][1] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, mine + 16u, 0, 0));
            if (sp == 0 && e < a.Epad) etab[e] = at;
        }
        if (tid < kTapSlots) {
            const int y = quotient(a.dkw, tid);
            tapoff[tid] = tid < a.taps ? (y * a.Wv + tid - y * a.kw) * 16 : 0;
        }
        if (tid < 4) bad[tid] = 0;
    }
    auto in_load = [&](int ch) __attribute__((always_inline)) {
        const int cib = (ch << a.l2bpc) + (sp >> 1);
        const unsigned lane_at = cib < a.nCib ? cib * plane_bytes + (sp & 1) * 32u : kBeyond;       // (beyond past the last chunk)
#pragma unroll
        for (int k = 0; k < kRounds; ++k) {
            const unsigned at = etab[min(se + k * er, a.Epad - 1)];
            const unsigned mine = max(at, lane_at) >= kBeyond ? kBeyond : at + lane_at;
            iv[k][0] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, mine, 0, 0));
            iv[k][1] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, mine + 16u, 0, 0));
        }
    };
    auto in_store = [&]() __attribute__((always_inline)) {
        uintx4 *d = B + sp * plane_e;
#pragma unroll
        for (int k = 0; k < kRounds; ++k) {
            uintx4 h, m, l;
            asm volatile("" : "+v"(iv[k][0]), "+v"(iv[k][1]));     // (keeps the splitting, and its wait, from moving up to the loads)
            split8(iv[k][0], iv[k][1], h, m, l, most);
            const int e = se + k * er, to = e < nE ? e : a.E;
            d[to] = h; d[planes * plane_e + to] = m; d[2 * planes * plane_e + to] = l;
        }
    };
    in_store();
    f_store(0);

    // ---- this lane's pixels
    int base[WM];
#pragma unroll
    for (int wm = 0; wm < WM; ++wm) {
        const int m = min(m0 + (wave_m * WM + wm) * 16 + p, a.M - 1);
        const int n = quotient(a.dHoWs, m), rem = m - n * a.HoWs, oh = quotient(a.dWs, rem);
        base[wm] = ((gb * 2 + half) * plane_e + (n * a.Hv + oh * a.stride - vr0) * a.Wv + (rem - oh * a.Ws) * a.stride) * 16;
    }
    floatx4 acc[WM][WN], low[WM][WN];                          // sums of hh; of all other products
#pragma unroll
    for (int wm = 0; wm < WM; ++wm)
#pragma unroll
        for (int wn = 0; wn < WN; ++wn) acc[wm][wn] = low[wm][wn] = floatx4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();

    // ---- reduction: the next step's filter and the next chunk's input are requested before the matrix instructions and
    // written over the current ones behind them
    const int part_b = planes * plane_e * 16;                  // bytes between the parts of B
    int buf = 0;
    for (int ch = 0; ch < a.n_chunks; ++ch) {
        in_load(ch + 1);
        for (int st = 0; st < a.steps; ++st, buf ^= 1) {
            const bool last_st = st + 1 == a.steps, end = last_st && ch + 1 == a.n_chunks;
            f_load(last_st ? ch + 1 : ch, last_st ? 0 : st + 1, !end);
            __builtin_amdgcn_sched_barrier(0);                 // the requests stay ahead of the matrix instructions
            const char *Bt = reinterpret_cast<const char *>(B) + tapoff[(st << (1 - a.l2bpc)) + gt];
            const uintx4 *Af = A + (buf * NCT + wave_n * WN) * 3 * 64 + lane;
            bf16x8 fa[WN][3], fb[WM][3];
#pragma unroll
            for (int s = 0; s < 3; ++s) {
#pragma unroll
                for (int wn = 0; wn < WN; ++wn) fa[wn][s] = __builtin_bit_cast(bf16x8, Af[(wn * 3 + s) * 64]);
#pragma unroll
                for (int wm = 0; wm < WM; ++wm) fb[wm][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4 *>(Bt + base[wm] + s * part_b));
            }
            constexpr int kPair[6][2] = {{0, 0}, {1, 0}, {0, 1}, {1, 1}, {2, 0}, {0, 2}};
#pragma unroll
            for (int t = 0; t < 6; ++t)
#pragma unroll
                for (int wm = 0; wm < WM; ++wm)
#pragma unroll
                    for (int wn = 0; wn < WN; ++wn) {
                        floatx4 &c = t == 0 ? acc[wm][wn] : low[wm][wn];
                        c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[wn][kPair[t][0]], fb[wm][kPair[t][1]], c, 0, 0, 0);
                    }
            if (end) break;
            f_store(buf ^ 1);
            if (last_st) {
                __syncthreads();
                in_store();
            }
            __syncthreads();
        }
    }
#pragma unroll
    for (int wm = 0; wm < WM; ++wm)
#pragma unroll
        for (int wn = 0; wn < WN; ++wn)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                acc[wm][wn][r] = (acc[wm][wn][r] + low[wm][wn][r]) * kUnscale;
                check = fmaf(acc[wm][wn][r], 0.f, check);
            }
    if (!(__builtin_fabsf(check) < __builtin_inff()) || !(most <= kMost)) bad[0] = 1;           // (NaN compares false)
    if (!(most_w <= kMost)) bad[1] = 1;
    __syncthreads();

    auto finish = [&](floatx4 v, int cob, size_t o, int q) __attribute__((always_inline)) {
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
    };
    if (bad[1] == 0) {
        if (bad[0] != 0) {
            // ---- some input or sum here is no finite sum of three parts: the fp32 matrix instruction, operands from memory, the
            // next step's on their way (lane (p, g): input channels 4g .. 4g + 3 of its pixels, filter values [4g + r][p])
            int ih0[WM], iw0[WM], at0[WM];
#pragma unroll
            for (int wm = 0; wm < WM; ++wm) {
                const int m = min(m0 + (wave_m * WM + wm) * 16 + p, a.M - 1);
                const int ns = quotient(a.dHoWs, m), rem = m - ns * a.HoWs, oh = quotient(a.dWs, rem);
                const int n = quotient(a.dStrips, ns), ow = rem - oh * a.Ws + (ns - n * a.strips) * a.Ws;
                ih0[wm] = oh * a.stride - a.pt;
                iw0[wm] = ow * a.stride - a.pl;
                at0[wm] = (n * a.nCib * a.H * a.W + ih0[wm] * a.W + iw0[wm]) * 64 + g * 16;
            }
            const int n_steps = a.nCib * a.taps;
            floatx4 x[2][WM];
            float w[2][WN][4];
            auto request = [&](int s, floatx4 (&xs)[WM], float (&ws)[WN][4]) __attribute__((always_inline)) {
                const int sc = min(s, n_steps - 1), cib = sc / a.taps, tap = sc - cib * a.taps, y = quotient(a.dkw, tap), z = tap - y * a.kw;
#pragma unroll
                for (int wm = 0; wm < WM; ++wm) {
                    const bool inside = ((unsigned)(ih0[wm] + y) < (unsigned)a.H) & ((unsigned)(iw0[wm] + z) < (unsigned)a.W);
                    const unsigned at = (unsigned)(at0[wm] + (cib * a.H * a.W + y * a.W + z) * 64);
                    xs[wm] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, inside ? at : kBeyond, 0, 0));
                }
#pragma unroll
                for (int wn = 0; wn < WN; ++wn) {
                    const int cob = cob0 + wave_n * WN + wn;
                    const unsigned at = cob < a.nCob ? (unsigned)((cob * n_steps + sc) * 1024 + (g * 64 + p) * 4) : kBeyond;
#pragma unroll
                    for (int r = 0; r < 4; ++r) ws[wn][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(flt, at + 64u * r, 0, 0));
                }
            };
#pragma unroll
            for (int wm = 0; wm < WM; ++wm)
#pragma unroll
                for (int wn = 0; wn < WN; ++wn) acc[wm][wn] = floatx4{0.f, 0.f, 0.f, 0.f};
            request(0, x[0], w[0]);
            for (int s = 0; s < n_steps; s += 2) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    request(s + k + 1, x[k ^ 1], w[k ^ 1]);
                    if (s + k < n_steps) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int wm = 0; wm < WM; ++wm)
#pragma unroll
                                for (int wn = 0; wn < WN; ++wn)
                                    acc[wm][wn] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[k][wn][r], x[k][wm][r], acc[wm][wn], 0, 0, 0);
                    }
                }
            }
        }
#pragma unroll
        for (int wm = 0; wm < WM; ++wm) {
            const int m = m0 + (wave_m * WM + wm) * 16 + p;
            const int ns = quotient(a.dHoWs, min(m, a.M - 1)), rem = m - ns * a.HoWs, oh = quotient(a.dWs, rem);
            const int n = quotient(a.dStrips, ns), ow = rem - oh * a.Ws + (ns - n * a.strips) * a.Ws;
            if (m < a.M && ow < a.Wo) {
#pragma unroll
                for (int wn = 0; wn < WN; ++wn) {
                    const int cob = cob0 + wave_n * WN + wn;
                    if (cob < a.nCob) finish(acc[wm][wn], cob, (((size_t)n * a.nCob + cob) * a.HoWo + oh * a.Wo + ow) * 16 + g * 4, g);
                }
            }
        }
        return;
    }
    // ---- some filter value is no finite sum of three parts. A tap outside the image does not count, whatever its weight (an
    // infinite one times the zero read there would): plain fp32, four output channels at a time
    for (int it = tid; it < TM * NCT * 4; it += 256) {
        const int q = it & 3, m = m0 + (it >> 2) % TM, cob = cob0 + (it >> 2) / TM;
        if (m >= a.M || cob >= a.nCob) continue;
        const int ns = quotient(a.dHoWs, m), rem = m - ns * a.HoWs, oh = quotient(a.dWs, rem);
        const int n = quotient(a.dStrips, ns), ow = rem - oh * a.Ws + (ns - n * a.strips) * a.Ws;
        if (ow >= a.Wo) continue;
        floatx4 v = {0.f, 0.f, 0.f, 0.f};
        for (int cib = 0; cib < a.nCib; ++cib)
            for (int tap = 0; tap < a.taps; ++tap) {
                const int y = quotient(a.dkw, tap), ih = oh * a.stride + y - a.pt, iw = ow * a.stride + tap - y * a.kw - a.pl;
                if ((unsigned)ih >= (unsigned)a.H || (unsigned)iw >= (unsigned)a.W) continue;
                const float *x = a.in + (((size_t)n * a.nCib + cib) * a.H * a.W + (size_t)ih * a.W + iw) * 16;
                const float *w = a.filt + (((size_t)cob * a.nCib + cib) * a.taps + tap) * 256 + q * 4;
                floatx4 u = {0.f, 0.f, 0.f, 0.f};                  // (sixteen products first: a chain of all would lose more bits)
                for (int c = 0; c < 16; ++c) {
                    const floatx4 wc = *reinterpret_cast<const floatx4 *>(w + c * 16);
                    u.x = fmaf(x[c], wc.x, u.x); u.y = fmaf(x[c], wc.y, u.y); u.z = fmaf(x[c], wc.z, u.z); u.w = fmaf(x[c], wc.w, u.w);
                }
                v += u;
            }
        finish(v, cob, (((size_t)n * a.nCob + cob) * a.HoWo + oh * a.Wo + ow) * 16 + q * 4, q);
    }
}

// The tile: a wave's 32 pixels x 64 channels leave two workgroups per compute unit their LDS and registers; larger and wider
// ones (64 x 64 per wave, 64 x 128 or 64 x 64 per workgroup) measured 1.3 to 2.6 times as long.
constexpr int kWM = 2, kWN = 4, kWVM = 4, kWVN = 1;
constexpr int kTM = 16 * kWM * kWVM, kNCT = kWN * kWVN;
constexpr size_t kMaxLds = 80 * 1024;
constexpr int kStrip = 16;             // output columns of a strip, at most: 128 pixels are then few rows (32 columns: 8 % slower)

struct Plan { bool ok; int l2bpc, steps, n_chunks, strips, Ws; long E, Epad; size_t lds; };

Plan plan_tile(const LayerGeom &g)
{
    Plan o;
    o.ok = false;
    const int taps = g.kh * g.kw, nCib = g.Ci / 16, Hv = (g.Ho - 1) * g.stride + g.kh;
    o.strips = (g.Wo + kStrip - 1) / kStrip;
    o.Ws = (g.Wo + o.strips - 1) / o.strips;
    const long M = (long)g.N * o.strips * g.Ho * o.Ws;
    if (g.Cib != 16 || g.Cob != 16 || taps < 2 || taps > kMaxTaps || ((long)g.N * o.strips + 1) * Hv >= (1L << 31) || M >= (1L << 31) - 512 ||
        (size_t)g.N * g.Ci * g.H * g.W * 4 >= kBeyond || (size_t)g.Co * g.Ci * taps * 4 >= kBeyond)
        return o;
    // two blocks a step, or two taps
    const int s2 = (nCib + 1) / 2 * taps, s1 = nCib * ((taps + 1) / 2);
    o.l2bpc = s2 <= s1 ? 1 : 0;
    o.steps = o.l2bpc ? taps : (taps + 1) / 2;
    o.n_chunks = o.l2bpc ? (nCib + 1) / 2 : nCib;
    // the most staged entries a tile of kTM pixels needs: its rows, and those around the strips that end inside it
    const long span = (kTM < M ? kTM : M) - 1, rows = (span + o.Ws - 1) / o.Ws + 1;
    const long cross = (long)g.N * o.strips > 1 ? (rows - 1 + g.Ho - 1) / g.Ho : 0;
    const long vrows = (rows - 1) * g.stride + g.kh + (g.kh > g.stride ? cross * (g.kh - g.stride) : 0);
    o.E = vrows * ((o.Ws - 1) * g.stride + g.kw);
    const int er = 128 >> o.l2bpc;
    const long rounds = (o.E + er - 1) / er;
    o.Epad = rounds * er;
    o.lds = (size_t)(kTapSlots + 4 + o.Epad) * 4 + (size_t)2 * kNCT * 3 * 1024 + (size_t)3 * (2 << o.l2bpc) * (o.E + 1) * 16;
    o.ok = o.lds <= kMaxLds && rounds <= kRounds;
    return o;
}

}  // namespace

// Where it beats the fp32 matrix instruction: stride 1 (a strided tile stages too many rows), nine steps or more, at least
// 15 / 16 of a workgroup per compute unit, and a time below the other kernels', from a model fitted to 1080 random layers of 150 to
// 1600 workgroups (11 % and 13 % root mean square; of 560 taken then, 20 are slower by more than 3 %, two by more than 10). The
// fullest compute unit counts, with a workgroup alone on it as 1.25; staging a chunk costs a step; work on padded channels, taps or
// columns is done but does not count; an odd number of output blocks costs the other kernels an empty block, or conv_same.hip its
// smaller tile (7 %). At full use the time is 0.62 of that of conv_same.hip's tiles and 0.495 of the others'. us with
// the fp32 instruction / here at the time of the fit (here 5 to 7 % less since, 333 us for the first): 64 -> 64 channels 56 x 56, 256 images (24.5 workgroups a unit) 454 / 355, 28 x 28, 64 images (1.53)
// 41.5 / 31.7, 48 images (1.15; not taken) 29.7 / 30.1, 40 images (0.96) 24.7 / 24.8, 8 x 8, 300 images (0.59; not taken) 18.1 / 23.7;
// 64 -> 112 28 x 28 x 64 66 / 58; 48 -> 64 28 x 28 x 40 (not taken) 20.1 / 23.6; 16 -> 64 (five steps; not taken) 7 x 7 x 500 9.0 /
// 11.5; 48 -> 64 5 x 5 28 x 28 x 64 127 / 60; 256 -> 96 1 x 3 79 x 20 x 12 (1.16; not taken) 36 / 50.
bool conv_split3_eligible(const LayerGeom &g)
{
    if (g.stride != 1) return false;
    const Plan pl = plan_tile(g);
    if (!pl.ok || pl.n_chunks * pl.steps < 9) return false;
    const int nCib = g.Ci / 16, nCob = g.Co / 16, n_cot = (nCob + kNCT - 1) / kNCT;
    const long cus = device_cus(), wgs = ((long)g.N * pl.strips * g.Ho * pl.Ws + kTM - 1) / kTM * n_cot;
    if (wgs * 16 < 15 * cus) return false;
    const bool same = conv_same_eligible(g);
    const double blocks = same ? nCob * (nCob % 2 ? 1.07 : 1.0) : (nCob + 1) / 2 * 2;
    const double useful = nCib * g.kh * g.kw * blocks * g.Wo / (2.0 * pl.n_chunks * (pl.steps + 1) * n_cot * kNCT * pl.strips * pl.Ws);
    const long most = (wgs + cus - 1) / cus;
    return (same ? 0.62 : 0.495) * (most == 1 ? 1.25 : (double)most) * cus < wgs * useful;
}

const char *conv_split3_kernel_name() { return "conv16_split3<2,4,4,1>"; }

hipError_t launch_conv_split3(const float *in, const float *filt, float *out, const float *res, const LayerGeom &g, int epilogue,
                              hipStream_t s, const float *bn)
{
    const Plan pl = plan_tile(g);
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(conv16_split3<kWM, kWN, kWVM, kWVN>),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
    if (attr != hipSuccess) return attr;
    if (!pl.ok) return hipErrorInvalidValue;
    Split3Args a;
    a.in = in; a.filt = filt; a.out = out; a.res = res; a.bn = bn; a.epilogue = epilogue;
    a.H = g.H; a.W = g.W; a.Ho = g.Ho; a.Wo = g.Wo; a.HoWo = g.Ho * g.Wo;
    a.Ws = pl.Ws; a.strips = pl.strips; a.HoWs = g.Ho * pl.Ws; a.M = g.N * pl.strips * a.HoWs;
    a.nCib = g.Ci / 16; a.nCob = g.Co / 16; a.taps = g.kh * g.kw; a.kh = g.kh; a.kw = g.kw; a.pt = g.pt; a.pl = g.pl;
    a.l2bpc = pl.l2bpc; a.steps = pl.steps; a.n_chunks = pl.n_chunks; a.stride = g.stride;
    a.Hv = (g.Ho - 1) * g.stride + g.kh; a.Wv = (pl.Ws - 1) * g.stride + g.kw;
    a.E = (int)pl.E; a.Epad = (int)pl.Epad;
    a.in_bytes = (unsigned)((size_t)g.N * g.Ci * g.H * g.W * 4); a.filt_bytes = (unsigned)((size_t)g.Co * g.Ci * a.taps * 4);
    a.n_cot = (a.nCob + kNCT - 1) / kNCT;
    a.dHoWs = make_fastdiv(a.HoWs); a.dWs = make_fastdiv(a.Ws); a.dWv = make_fastdiv(a.Wv); a.dHv = make_fastdiv(a.Hv);
    a.dStrips = make_fastdiv(a.strips); a.dCt = make_fastdiv(a.n_cot); a.dkw = make_fastdiv(a.kw);
    const dim3 grid((unsigned)((a.M + kTM - 1) / kTM * a.n_cot));
    hipLaunchKernelGGL((conv16_split3<kWM, kWN, kWVM, kWVN>), grid, dim3(256), pl.lds, s, a);
    return hipGetLastError();
}

}  // namespace small
