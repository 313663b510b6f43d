// Image-resident runs of quantized layers: one workgroup takes one image through a run of layers with every tensor, as
// signed bytes, in LDS. A quantized network's tensors are a few kilobytes per image and its layers a microsecond of work, so
// layer by layer its time is launches and their latencies (an 11-layer audio CNN: 12 launches of about 4 us). Bound here:
// the chain of layers -- per layer one barrier and the LDS latency of a few reduction steps.
//
//   - activations keep their layout [C/16][H][W][16]: a pixel's channel block is one matrix operand (quant.hip); bit 7 of
//     every code is flipped once, when the run's input is read and in each layer's requantization.
//   - a tap outside the image is redirected to an entry of the layer's padding code, a chunk past the reduction's end to a
//     zero entry: an address select instead of four selects of the value. Where chunk c = (input block, tap) of a layer lies
//     relative to a pixel is tabled in LDS once per workgroup.
//   - the next layer's filter (and the sums of its channels) is on its way into the other of two LDS buffers while a layer is
//     computed, by the load unit: no registers (of which a thread has 128) and no copy behind the layer. Its bytes are made
//     signed when they are read. (Through registers: audio CNN, 100 images 28.0 us, here 23.6; residual CNN, 256 images 39.0 and
//     33.9.) Filters are at most 64 KB.
//   - depthwise layers run on the matrix cores as well (conv_unit); additions, global average pooling and a closing fully
//     connected layer are plain vector code.
#include "small_internal.h"

#include <type_traits>

namespace small {
namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 16, kThreads = 64 * kWaves;
constexpr int kMaxFilter = 65536;

// One layer, packed so that kRU8MaxLayers of them fit the 4 KB of kernel arguments.
struct RU8Layer {
    const unsigned char *filt;
    const int *sums;               // or null (zx = 128)
    int kind_win;                  // kind | stride << 8 | pt << 16 | pl << 24
    int in_hw, out_hw;             // H | W << 16
    int blocks;                    // input blocks | output blocks << 16
    int taps;                      // taps | kw << 8 | window height << 16
    int src, src2, dst;            // LDS byte offsets
    int table;                     // first chunk-table entry | chunks << 16
    int filt_bytes, sums_bytes;    // sums: the channel sums behind the filter in LDS (convolutions only)
    int z;                         // zx | zw << 8 | zy << 16 | shift << 24   (add: za, zb, zy, shift)
    int clamp;                     // lo | hi << 8 | pixel groups of a unit << 16 | Cob << 24
    int mult, amax;                // (add: mult_a, mult_b)
    unsigned magic, shift;         // division by Wo (average pooling: by the pixel count)
    int inv_unit, inv_taps;        // ceil(2^20 / d) of output blocks, and of taps
    int inv_kw;
    int Co;                        // outputs of a closing fully connected layer
};
struct RU8Args {
    const unsigned char *in;
    unsigned char *out;
    int N, n_layers;
    int in_bytes, in_at;           // bytes of an image of the run's input, its LDS offset
    int out_bytes, out_at;         // ... of its result; out_bytes of a closing fully connected layer: 0 (it writes itself)
    int pads, table, filt0, filt1; // LDS byte offsets
    RU8Layer layer[kRU8MaxLayers];
};
static_assert(sizeof(RU8Args) <= 4096, "kernel arguments");
typedef const __attribute__((address_space(4))) RU8Args *RU8KernArgs;
// all of a layer at once: field by field, where they are used, the scalar loads (some 250 cycles each) stand one behind the other
__device__ __forceinline__ RU8Layer layer_at(RU8KernArgs ka, int l)
{
    RU8Layer L;
    __builtin_memcpy(&L, (const __attribute__((address_space(4))) char *)&ka->layer[l], sizeof(L));
    return L;
}

__device__ __forceinline__ int quotient(unsigned magic, unsigned shift, int n)       // magic = 0: by one
{
    return (int)((__umulhi((unsigned)n, magic) + (magic ? 0u : (unsigned)n)) >> shift);
}
// n / d by inv = ceil(2^20 / d): exact for n < 4096 and d <= 255 (chunks by taps), and for n below the units of a layer and d
// its output blocks, as long as these are at most kMaxUnitBlocks and blocks x pixels at most 4096 (resident_u8_takes; with 1025
// blocks of one pixel the quotient of unit 1024 would be 1)
constexpr int kMaxUnitBlocks = 1024;
__device__ __forceinline__ int short_div(int n, int inv) { return (n * inv) >> 20; }
__device__ __forceinline__ unsigned pack4(const unsigned (&y)[4]) { return y[0] | y[1] << 8 | y[2] << 16 | y[3] << 24; }

// shift 32: mult is the layer's q.mult32 (small_internal.h)
struct Requant { int amax, mult, shift, lo, hi; long bias; };
__device__ __forceinline__ unsigned requant_high(int v, const Requant &q)
{
    return (unsigned)clamp_code((int)(((long)v * (long)q.mult + q.bias) >> 32), q.lo, q.hi);
}
__device__ __forceinline__ unsigned requant_signed(int v, const Requant &q)          // the code, unsigned
{
    if (q.shift == 32) return requant_high(v, q);
    const int c = min(max(v, -q.amax), q.amax);
    const int r = (int)(((long)c * (long)q.mult + q.bias) >> q.shift);
    return (unsigned)min(max(r, q.lo), q.hi);
}

// A unit of a convolution or (DW) depthwise layer: one output block x WM groups of 16 pixels. A depthwise layer is the
// convolution whose filter of a block has channel c's taps on the diagonal: the matrix cores are idle otherwise, and an output
// word costs three matrix instructions and a third of the vector instructions of byte permutes and dot products.
template <int WM, bool DW>
__device__ __forceinline__ void conv_unit(char *lds, const RU8Layer &L, const Requant &q, int u, int lane, int zx, int zw, int filt,
                                          int pads, int table)
{
    const int p = lane & 15, g = lane >> 4;
    const int H = L.in_hw & 0xffff, W = L.in_hw >> 16, Wo = L.out_hw >> 16, P = (L.out_hw & 0xffff) * Wo;
    const int nCob = L.blocks >> 16, chunks = L.table >> 16;
    const int grp = short_div(u, L.inv_unit), cob = u - grp * nCob;
    const int stride = (L.kind_win >> 8) & 255, pt = (L.kind_win >> 16) & 255, pl = L.kind_win >> 24;
    const int za = zx - 128, zb = zw - 128;
    const int src = L.src + (DW ? cob * H * W * 16 : 0);
    int ih0[WM], iw0[WM], base[WM];
#pragma unroll
    for (int i = 0; i < WM; ++i) {
        const int m = min((grp * WM + i) * 16 + p, P - 1), oh = quotient(L.magic, L.shift, m);
        ih0[i] = oh * stride - pt;
        iw0[i] = (m - oh * Wo) * stride - pl;
        base[i] = src + (ih0[i] * W + iw0[i]) * 16;
    }
    const intx4 ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    const int K = DW ? chunks : chunks * 16;
    intx4 acc[WM], acc_s[WM], acc_w = {0, 0, 0, 0};
    intx4 c0 = {K * za * zb, K * za * zb, K * za * zb, K * za * zb};
    if (!DW && za != 0) {
        const intx4 sums = *reinterpret_cast<const intx4 *>(lds + filt + L.filt_bytes + (cob * 16 + 4 * g) * 4);
#pragma unroll
        for (int r = 0; r < 4; ++r) c0[r] = (int)((unsigned)c0[r] - (unsigned)za * ((unsigned)sums[r] - (unsigned)K * 128u));
    }
#pragma unroll
    for (int i = 0; i < WM; ++i) { acc[i] = c0; acc_s[i] = intx4{0, 0, 0, 0}; }
    const int *tab = reinterpret_cast<const int *>(lds + table) + (L.table & 0xffff);
    const char *fl = lds + filt + (DW ? cob * chunks * 16 + p : cob * chunks * 256 + p * 16);
    intx4 diag;                                                // DW: 0xff in byte p of the operand
#pragma unroll
    for (int k = 0; k < 4; ++k) diag[k] = (p >> 2) == k ? 255 << (8 * (p & 3)) : 0;
    // (one step at a time: two or three at once, their reads ahead of the first use, need more than a thread's 128 registers, and
    // what is spilled costs more than the waiting: audio CNN, 100 images 25.2 us, here 23.6)
    for (int t = 0; t < chunks; t += 4) {
        const int c = t + g, e = tab[c];                       // (padded to whole steps)
        intx4 fa;
        int w;
        if (DW) w = *reinterpret_cast<const unsigned char *>(fl + min(c, chunks - 1) * 16);
        else fa = *reinterpret_cast<const intx4 *>(fl + min(c, chunks - 1) * 256) ^ (int)0x80808080u;
        const bool live = c < chunks;
        const int y = e & 63, x = (e >> 6) & 63, off = (e >> 12) * 16, outside = live ? pads : 0;
        intx4 fb[WM];
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const bool in = ((unsigned)(ih0[i] + y) < (unsigned)H) & ((unsigned)(iw0[i] + x) < (unsigned)W) & live;
            fb[i] = *reinterpret_cast<const intx4 *>(lds + (in ? base[i] + off : outside));
        }
        if (DW) {
            const int v = (w ^ 128) * 0x01010101;
            fa = intx4{v, v, v, v} & diag;
            if (za != 0) acc_w = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa & lane_mask(live), ones, acc_w, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa, fb[i], acc[i], 0, 0, 0);
            if (zb != 0) acc_s[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(DW ? diag & ones : ones, fb[i], acc_s[i], 0, 0, 0);
        }
    }
    if (zb != 0) {
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r)                        // (without a diagonal all rows are the same)
                acc[i][r] = (int)((unsigned)acc[i][r] - (unsigned)zb * (unsigned)acc_s[i][DW ? r : 0]);
    }
    if (DW && za != 0) {
#pragma unroll
        for (int i = 0; i < WM; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][r] = (int)((unsigned)acc[i][r] - (unsigned)za * (unsigned)acc_w[r]);
    }
    auto store = [&](auto high) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < WM; ++i) {
            const int m = (grp * WM + i) * 16 + p;
            unsigned y[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) y[r] = decltype(high)::value ? requant_high(acc[i][r], q) : requant_signed(acc[i][r], q);
            if (m < P) *reinterpret_cast<unsigned *>(lds + L.dst + (cob * P + m) * 16 + 4 * g) = pack4(y) ^ 0x80808080u;
        }
    };
    if (q.shift == 32) store(std::true_type());
    else store(std::false_type());
}

template <bool DW>
__device__ __forceinline__ void conv_layer(char *lds, const RU8Layer &L, const Requant &q, int wave, int lane, int zx, int zw, int filt,
                                           int pads, int table)
{
    const int P = (L.out_hw & 0xffff) * (L.out_hw >> 16), wm = (L.clamp >> 16) & 255;
    const int units = ((P + 16 * wm - 1) >> (wm == 1 ? 4 : wm == 2 ? 5 : 6)) * (L.blocks >> 16);
    for (int u = wave; u < units; u += kWaves) {
        if (wm == 1) conv_unit<1, DW>(lds, L, q, u, lane, zx, zw, filt, pads, table);
        else if (wm == 2) conv_unit<2, DW>(lds, L, q, u, lane, zx, zw, filt, pads, table);
        else conv_unit<4, DW>(lds, L, q, u, lane, zx, zw, filt, pads, table);
    }
}

__global__ void __launch_bounds__(kThreads) resident_u8(RU8Args a)
{
    extern __shared__ intx4 lds4[];
    char *lds = reinterpret_cast<char *>(lds4);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int flip = (int)0x80808080u;
    const RU8KernArgs ka = (RU8KernArgs)__builtin_amdgcn_kernarg_segment_ptr();

    // ---- tables: the zero entry, every layer's padding entry, where its chunks lie
    if (tid == 0) lds4[0] = intx4{0, 0, 0, 0};
    if (tid < 4 * a.n_layers) reinterpret_cast<int *>(lds + a.pads)[tid] = ((a.layer[tid >> 2].z & 255) * 0x01010101) ^ flip;
    for (int l = wave; l < a.n_layers; l += kWaves) {
        const RU8Layer &L = a.layer[l];
        const int chunks = L.table >> 16;
        int *tab = reinterpret_cast<int *>(lds + a.table) + (L.table & 0xffff);
        const int taps = L.taps & 255, kw = (L.taps >> 8) & 255, H = L.in_hw & 0xffff, W = L.in_hw >> 16;
        for (int c = lane; c < ((chunks + 3) & ~3); c += 64) {
            const int cib = short_div(c, L.inv_taps), tap = c - cib * taps, y = short_div(tap, L.inv_kw), x = tap - y * kw;
            tab[c] = (cib * H * W + y * W + x) << 12 | x << 6 | y;
        }
    }

    // ---- the filter of a layer (and its channel sums behind it) into LDS, by the load unit: whole kilobytes of a wave, the last
    // one's lanes beyond the end switched off
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) void *)lds;
    auto filter_request = [&](const RU8Layer &L, int at) __attribute__((always_inline)) {
        for (int k = wave * 1024; k < L.filt_bytes; k += kThreads * 16)
            if (k + lane * 16 < L.filt_bytes) dma16(L.filt, (unsigned)(k + lane * 16), lds0 + (unsigned)(at + k));
        if (L.sums != nullptr)
            for (int k = wave * 1024; k < L.sums_bytes; k += kThreads * 16)
                if (k + lane * 16 < L.sums_bytes) dma16(L.sums, (unsigned)(k + lane * 16), lds0 + (unsigned)(at + L.filt_bytes + k));
    };
    filter_request(a.layer[0], a.filt0);
    const intx4 first = reinterpret_cast<const intx4 *>(a.in + (size_t)blockIdx.x * a.in_bytes)[min(tid, a.in_bytes / 16 - 1)];

    int filt = a.filt0, other = a.filt1;
    for (int n = blockIdx.x; n < a.N; n += gridDim.x) {
        const intx4 *src = reinterpret_cast<const intx4 *>(a.in + (size_t)n * a.in_bytes);
        for (int i = tid; i * 16 < a.in_bytes; i += kThreads)
            *reinterpret_cast<intx4 *>(lds + a.in_at + i * 16) = (n == (int)blockIdx.x && i == tid ? first : src[i]) ^ flip;
        wait_vmcnt<0>();
        __syncthreads();
        for (int l = 0; l < a.n_layers; ++l) {
            const RU8Layer L = layer_at(ka, l);
            const RU8Layer next = layer_at(ka, l + 1 < a.n_layers ? l + 1 : 0);
            filter_request(next, other);                       // (its buffer was last read before the barrier)
            const int kind = L.kind_win & 255;
            const int zx = L.z & 255, zw = (L.z >> 8) & 255, pads = a.pads + 16 * l;
            Requant q;
            q.amax = L.amax; q.mult = L.mult; q.shift = (L.z >> 24) & 63; q.lo = L.clamp & 255; q.hi = (L.clamp >> 8) & 255;
            q.bias = (q.shift > 0 ? 1L << (q.shift - 1) : 0L) + ((long)((L.z >> 16) & 255) << q.shift);
            if (kind == RU8_CONV) {
                conv_layer<false>(lds, L, q, wave, lane, zx, zw, filt, pads, a.table);
            } else if (kind == RU8_DW) {
                conv_layer<true>(lds, L, q, wave, lane, zx, zw, filt, pads, a.table);
            } else if (kind == RU8_ADD) {
                const int words = (L.blocks & 0xffff) * (L.in_hw & 0xffff) * (L.in_hw >> 16) * 4;
                for (int i = tid; i < words; i += kThreads) {
                    const unsigned x = *reinterpret_cast<const unsigned *>(lds + L.src + i * 4) ^ 0x80808080u;
                    const unsigned w = *reinterpret_cast<const unsigned *>(lds + L.src2 + i * 4) ^ 0x80808080u;
                    unsigned y[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        long v = (long)((int)((x >> (8 * k)) & 255u) - zx) * (long)L.mult + (long)((int)((w >> (8 * k)) & 255u) - zw) * (long)L.amax;
                        v = (v + q.bias) >> q.shift;
                        v = v < q.lo ? q.lo : v;
                        y[k] = (unsigned)(v > q.hi ? q.hi : v);
                    }
                    *reinterpret_cast<unsigned *>(lds + L.dst + i * 4) = pack4(y) ^ 0x80808080u;
                }
            } else if (kind == RU8_AVG) {
                const int nB = L.blocks & 0xffff, HW = (L.in_hw & 0xffff) * (L.in_hw >> 16), quad = lane & 3;
                for (int blk = wave; blk < nB; blk += kWaves) {
                    unsigned s[4] = {0, 0, 0, 0};
                    for (int m = lane >> 2; m < HW; m += 16) {
                        const unsigned x = *reinterpret_cast<const unsigned *>(lds + L.src + (blk * HW + m) * 16 + quad * 4) ^ 0x80808080u;
#pragma unroll
                        for (int c = 0; c < 4; ++c) s[c] += (x >> (8 * c)) & 255u;
                    }
#pragma unroll
                    for (int c = 0; c < 4; ++c) s[c] = add_quads(s[c]);
                    unsigned y[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c) y[c] = (unsigned)quotient(L.magic, L.shift, (int)(s[c] + (unsigned)HW / 2u));
                    if (lane < 4) *reinterpret_cast<unsigned *>(lds + L.dst + blk * 16 + quad * 4) = pack4(y) ^ 0x80808080u;
                }
            } else {                                           // RU8_DENSE: the closing layer, straight to memory
                const int nB = L.blocks & 0xffff, Cob = (L.clamp >> 24) & 255, za = zx - 128, zb = zw - 128;
                for (int o = wave; o < L.Co; o += kWaves) {
                    const int cob = o / Cob, oi = o - cob * Cob;
                    int v = 0;
                    for (int i = lane; i < nB * 4; i += 64) {
                        const int x = *reinterpret_cast<const int *>(lds + L.src + i * 4);
                        const int w = *reinterpret_cast<const int *>(lds + filt + ((cob * nB + (i >> 2)) * Cob + oi) * 16 + (i & 3) * 4) ^ flip;
                        v = __builtin_amdgcn_sdot4(x, w, v, false) - zb * __builtin_amdgcn_sdot4(x, 0x01010101, 0, false) -
                            za * __builtin_amdgcn_sdot4(w, 0x01010101, 0, false);
                    }
                    v = wave_sum(v);
                    v += nB * 16 * za * zb;
                    if (lane == 0) a.out[(size_t)n * L.Co + o] = (unsigned char)requant_signed(v, q);
                }
            }
            const int t = filt;
            filt = other;
            other = t;
            wait_vmcnt<0>();                                   // this wave's part of the next filter has landed
            __syncthreads();
        }
        for (int i = tid; i * 16 < a.out_bytes; i += kThreads)
            *reinterpret_cast<intx4 *>(a.out + (size_t)n * a.out_bytes + i * 16) = *reinterpret_cast<const intx4 *>(lds + a.out_at + i * 16) ^ flip;
        __syncthreads();
    }
}

constexpr size_t kMaxLds = 160 * 1024;

size_t ru8_chunks(const RU8Group &g)
{
    return g.kind == RU8_CONV ? (size_t)g.Ci / 16 * g.kh * g.kw : g.kind == RU8_DW ? (size_t)g.kh * g.kw : 0;
}

// what filter_request brings into LDS behind a layer's filter: the one statement of it, for the layout and for the kernel
size_t ru8_sums_bytes(const RU8Group &g) { return g.kind == RU8_CONV ? (size_t)g.Co * 4 : 0; }

struct Layout { int pads, table, filt0, filt1, at[kRU8Buffers]; size_t bytes; };

bool lay_out(const RU8Group *g, int n, Layout &o)
{
    size_t at = 16;
    o.pads = (int)at;
    at += 16 * (size_t)n;
    o.table = (int)at;
    size_t filt = 0, entries = 0, size[kRU8Buffers] = {};
    size[g[0].src] = (size_t)g[0].Ci * g[0].H * g[0].W;
    for (int i = 0; i < n; ++i) {
        entries += (ru8_chunks(g[i]) + 3) / 4 * 4;
        const size_t f = (ru8_filter_bytes(g[i]) + 15) / 16 * 16 + ru8_sums_bytes(g[i]);
        filt = f > filt ? f : filt;
        if (g[i].kind == RU8_DENSE) continue;
        const size_t b = (size_t)g[i].Co * g[i].Ho * g[i].Wo;
        if (b > size[g[i].dst]) size[g[i].dst] = b;
    }
    if (entries > 0xffff) return false;
    at += 4 * entries;
    at = (at + 15) / 16 * 16;
    for (int k = 0; k < kRU8Buffers; ++k) {
        o.at[k] = (int)at;
        at += (size[k] + 15) / 16 * 16;
    }
    o.filt0 = (int)at;
    at += filt;
    o.filt1 = (int)at;
    at += filt;
    o.bytes = at;
    return at <= kMaxLds;
}

}  // namespace

size_t ru8_filter_bytes(const RU8Group &g)
{
    return g.kind == RU8_CONV || g.kind == RU8_DENSE ? (size_t)g.Co * g.Ci * g.kh * g.kw : g.kind == RU8_DW ? (size_t)g.Ci * g.kh * g.kw : 0;
}

bool resident_u8_fits(const RU8Group *g, int n)
{
    if (n < 1 || n > kRU8MaxLayers) return false;
    Layout o;
    return lay_out(g, n, o);
}

bool resident_u8_takes(const RU8Group &g)
{
    if (g.Ci % 16 || g.H > 255 || g.W > 255 || g.stride > 255 || (size_t)g.Ci * g.H * g.W > 65536) return false;
    if (g.kind == RU8_ADD || g.kind == RU8_AVG) return true;
    if (ru8_filter_bytes(g) > (size_t)kMaxFilter || ((uintptr_t)g.filt & 15u) || g.q.amax <= 0) return false;
    if (g.kind == RU8_DW)
        return g.kh * g.kw <= 255 && g.kh < 64 && g.kw < 64 && (size_t)g.Ci * g.Ho * g.Wo <= 65536 && g.Ci / 16 <= kMaxUnitBlocks;
    // (channel sums at another address are refused by the layer's own call, also where they are not needed)
    if ((uintptr_t)g.sums & 15u) return false;
    if (g.kind == RU8_DENSE) return g.Cob < 16 && ru8_filter_bytes(g) % 16 == 0;
    return g.Co % 16 == 0 && (size_t)g.Co * g.Ho * g.Wo <= 65536 && g.Co / 16 <= kMaxUnitBlocks && g.kh * g.kw <= 255 && g.kh < 64 && g.kw < 64 &&
           (g.Ci / 16) * g.kh * g.kw < 4096 && (g.sums || g.q.zx == 128);
}

hipError_t launch_resident_u8(const RU8Group *g, int n, const unsigned char *in, unsigned char *out, int N, hipStream_t s)
{
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(resident_u8),
                                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds);
    if (attr != hipSuccess) return attr;
    Layout o;
    if (!lay_out(g, n, o)) return hipErrorInvalidValue;
    RU8Args a;
    a.in = in; a.out = out; a.N = N; a.n_layers = n;
    a.in_bytes = g[0].Ci * g[0].H * g[0].W; a.in_at = o.at[g[0].src];
    const RU8Group &last = g[n - 1];
    a.out_bytes = last.kind == RU8_DENSE ? 0 : last.Co * last.Ho * last.Wo;
    a.out_at = last.kind == RU8_DENSE ? 0 : o.at[last.dst];
    a.pads = o.pads; a.table = o.table; a.filt0 = o.filt0; a.filt1 = o.filt1;
    int entries = 0;
    for (int i = 0; i < n; ++i) {
        const RU8Group &l = g[i];
        RU8Layer &d = a.layer[i];
        const bool add = l.kind == RU8_ADD;
        const int chunks = (int)ru8_chunks(l);
        d.filt = l.filt; d.sums = l.sums;
        d.kind_win = l.kind | l.stride << 8 | l.pt << 16 | l.pl << 24;
        d.in_hw = l.H | l.W << 16; d.out_hw = l.Ho | l.Wo << 16;
        d.blocks = l.Ci / 16 | (chunks ? l.Co / 16 : 0) << 16;
        d.taps = l.kh * l.kw | l.kw << 8 | l.kh << 16;
        if (l.kind == RU8_AVG) d.taps = 0;
        d.src = o.at[l.src]; d.src2 = o.at[l.src2]; d.dst = l.kind == RU8_DENSE ? 0 : o.at[l.dst];
        d.table = entries | chunks << 16;
        entries += (chunks + 3) / 4 * 4;
        d.filt_bytes = (int)ru8_filter_bytes(l);
        d.sums_bytes = (int)ru8_sums_bytes(l);
        d.Co = l.kind == RU8_DENSE ? l.Co : 0;
        d.z = add ? l.qa.za | l.qa.zb << 8 | l.qa.zy << 16 | l.qa.shift << 24 : l.q.zx | l.q.zw << 8 | l.q.zy << 16 | (l.q.mult32 >= 0 ? 32 : l.q.shift) << 24;
        // pixel groups of a unit: a filter operand serves that many, as long as every wave still has a unit
        const int groups = (l.Ho * l.Wo + 15) / 16, units = groups * (l.Co / 16);
        const int wm = units >= 4 * kWaves ? 4 : units >= 2 * kWaves ? 2 : 1;
        d.clamp = (add ? l.qa.lo | l.qa.hi << 8 : l.q.lo | l.q.hi << 8) | wm << 16 | (l.kind == RU8_DENSE ? l.Cob : 0) << 24;
        d.mult = add ? l.qa.mult_a : l.q.mult32 >= 0 ? l.q.mult32 : l.q.mult;
        d.amax = add ? l.qa.mult_b : l.q.amax;
        const FastDiv f = make_fastdiv(l.kind == RU8_AVG ? l.H * l.W : l.Wo > 0 ? l.Wo : 1);
        d.magic = f.magic; d.shift = f.shift;
        auto inv = [](int v) { return v > 0 ? ((1 << 20) + v - 1) / v : 0; };
        d.inv_unit = inv(l.Co / 16); d.inv_taps = inv(l.kh * l.kw); d.inv_kw = inv(l.kw);
    }
    const long slots = (long)device_cus() * (o.bytes * 2 <= kMaxLds ? 2 : 1);
    const long rounds = (N + slots - 1) / slots;
    hipLaunchKernelGGL(resident_u8, dim3((unsigned)((N + rounds - 1) / rounds)), dim3(kThreads), o.bytes, s, a);
    return hipGetLastError();
}

}  // namespace small
