// Quantized pointwise convolution (1x1 window, any stride, no padding), 16-byte blocks, at most 256 input channels.
//
// Bound: vector instructions and, for wide layers, the output stream; the matrix work is a few instructions per tile. The
// kernels of quant.hip give a wave two or four output blocks and read and sign-flip the wave's pixels again for every such
// group (96 -> 160 channels: five times). Here a wave holds 32 pixels, already signed, in registers and walks all output
// blocks of the workgroup's share, whose filter was sign-flipped once into LDS together with the constant term of every
// channel (K a b - a * sum of its signed filter bytes, the accumulators' initial value): per output code about six vector
// instructions instead of twelve. Four blocks at a time are transposed across the lane groups, so that a store writes whole
// 16-byte blocks. Waves walk pixel tiles with the next tile's pixels on their way.
#include "small_internal.h"

namespace small {
namespace {

typedef int intx4 __attribute__((ext_vector_type(4)));

constexpr int kWM = 2;                  // groups of 16 pixels of a wave

struct QPwArgs {
    const unsigned char *in, *filt;
    unsigned char *out;
    const int *filt_sums;
    int W, HW, Wo, HoWo, M, stride;
    int nCib, nCob, share;              // share: output blocks of a workgroup, a multiple of 4
    int n_tiles, n_waves;
    unsigned in_bytes, filt_bytes, out_bytes;      // each below 2 GiB
    FastDiv dHoWo, dWo;
    QuantParams q;
};

// STEPS: matrix instructions of a reduction (four input blocks each); CORR: the pixel sums are needed (zw != 128)
template <int STEPS, bool CORR, bool HIGH, bool STREAM>
__global__ void __launch_bounds__(256) pw_u8_walk(QPwArgs a)
{
    extern __shared__ intx4 lds[];
    intx4 *A = lds;                                            // [block of the share][step][lane]
    int *cst = reinterpret_cast<int *>(lds + a.share * STEPS * 64);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = lane & 15, g = lane >> 4;
    const int cob0 = (int)blockIdx.y * a.share, n_cob = min(a.share, a.nCob - cob0);
    const int za = a.q.zx - 128, zb = a.q.zw - 128;
    const int flip = (int)0x80808080u;
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(a.in), 0, a.in_bytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t flt = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char *>(a.filt), 0, a.filt_bytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t dst = __builtin_amdgcn_make_buffer_rsrc(a.out, 0, a.out_bytes, kRawBuffer);

    // pixels of a tile: lane (p, g) holds input blocks g, 4 + g, ... of pixel p of each group
    auto request = [&](int tile, intx4 (&v)[kWM][STEPS]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < kWM; ++i) {
            const int m = min(tile * (16 * kWM) + i * 16 + p, a.M - 1);
            const int n = quotient(a.dHoWo, m), rem = m - n * a.HoWo, oh = quotient(a.dWo, rem), ow = rem - oh * a.Wo;
            const unsigned at = (unsigned)(n * a.nCib * a.HW + (oh * a.W + ow) * a.stride + g * a.HW) * 16u;
#pragma unroll
            for (int t = 0; t < STEPS; ++t)
                v[i][t] = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(
                              src, 4 * t + g < a.nCib ? at + (unsigned)(4 * t * a.HW) * 16u : kBeyond, 0, 0));
        }
    };
    intx4 cur[kWM][STEPS];
    const int wv = (int)blockIdx.x * 4 + wave;
    request(min(wv, a.n_tiles - 1), cur);

    // the share's filter, signed, zeros beyond the input blocks; and the channels' constants
    for (int u = wave; u < a.share * STEPS; u += 4) {
        const int wn = u / STEPS, t = u - wn * STEPS, cib = 4 * t + g;
        const bool ok = (wn < n_cob) & (cib < a.nCib);
        const intx4 v = __builtin_bit_cast(intx4, __builtin_amdgcn_raw_buffer_load_b128(
                            flt, ok ? (unsigned)((((cob0 + wn) * a.nCib + cib) * 16 + p) * 16) : kBeyond, 0, 0));
        A[u * 64 + lane] = v ^ (ok ? flip : 0);
    }
    for (int c = tid; c < a.share * 16; c += 256) {
        const int K = a.nCib * 16;
        const int sum = a.filt_sums && c < n_cob * 16 ? a.filt_sums[cob0 * 16 + c] - K * 128 : 0;      // (no sums: a is 0)
        cst[c] = K * za * zb - za * sum;
    }
    __syncthreads();
    const long addend = requant_addend<HIGH>(a.q);
    const intx4 ones = {0x01010101, 0x01010101, 0x01010101, 0x01010101};
    for (int tile = wv; tile < a.n_tiles; tile += a.n_waves) {
        intx4 nxt[kWM][STEPS], fb[kWM][STEPS];
        request(min(tile + a.n_waves, a.n_tiles - 1), nxt);
        __builtin_amdgcn_sched_barrier(0);
        int px[kWM];
        unsigned at[kWM];                                      // byte of (pixel, block 0) in the output
#pragma unroll
        for (int i = 0; i < kWM; ++i) {
            intx4 s = {0, 0, 0, 0};
#pragma unroll
            for (int t = 0; t < STEPS; ++t) {
                fb[i][t] = cur[i][t] ^ (4 * t + g < a.nCib ? flip : 0);
                if (CORR) s = __builtin_amdgcn_mfma_i32_16x16x64_i8(ones, fb[i][t], s, 0, 0, 0);
            }
            px[i] = CORR ? zb * s[0] : 0;
            const int m = tile * (16 * kWM) + i * 16 + p, mc = min(m, a.M - 1);
            const int n = quotient(a.dHoWo, mc);
            at[i] = m < a.M ? (unsigned)(n * a.nCob * a.HoWo + mc - n * a.HoWo) * 16u : kBeyond;
        }
        for (int c = 0; c < n_cob; c += 4) {
            unsigned w[kWM][4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const intx4 c0 = *reinterpret_cast<const intx4 *>(cst + (c + k) * 16 + 4 * g);
                intx4 acc[kWM];
#pragma unroll
                for (int i = 0; i < kWM; ++i) acc[i] = c0;
#pragma unroll
                for (int t = 0; t < STEPS; ++t) {
                    const intx4 fa = A[((c + k) * STEPS + t) * 64 + lane];
#pragma unroll
                    for (int i = 0; i < kWM; ++i) acc[i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa, fb[i][t], acc[i], 0, 0, 0);
                }
#pragma unroll
                for (int i = 0; i < kWM; ++i) {
                    unsigned y[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) y[r] = (unsigned)requant_code<HIGH>(acc[i][r] - px[i], a.q, addend);
                    w[i][k] = y[0] | y[1] << 8 | y[2] << 16 | y[3] << 24;
                }
            }
            // word k of lane group g -> word g of lane group k: group g then holds all of block c + g
            const bool ok = c + g < n_cob;
            const unsigned block_at = (unsigned)((cob0 + c + g) * a.HoWo) * 16u;
#pragma unroll
            for (int i = 0; i < kWM; ++i) {
                auto t01 = __builtin_amdgcn_permlane16_swap(w[i][0], w[i][1], false, false);
                auto t23 = __builtin_amdgcn_permlane16_swap(w[i][2], w[i][3], false, false);
                auto e = __builtin_amdgcn_permlane32_swap(t01[0], t23[0], false, false);
                auto o = __builtin_amdgcn_permlane32_swap(t01[1], t23[1], false, false);
                __builtin_amdgcn_raw_buffer_store_b128(uintx4{e[0], o[0], e[1], o[1]}, dst, ok & (at[i] != kBeyond) ? at[i] + block_at : kBeyond, 0,
                                                       STREAM ? kNonTemporal : 0);
            }
        }
#pragma unroll
        for (int i = 0; i < kWM; ++i)
#pragma unroll
            for (int t = 0; t < STEPS; ++t) cur[i][t] = nxt[i][t];
    }
}

template <int STEPS, bool HIGH>
void go2(const QPwArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    // Outputs of 10 MB and more are stored non-temporally: over 27 random layers of 8 to 32 MB 0.78 to 1.0 of the time (400 images of
    // 64 -> 64 channels 28x28 9.7 -> 8.4 us, 64 of 56x56 7.2 -> 6.1); 8 MB are even, and below 4 MB it takes 2 to 4 % longer.
    const bool stream = a.out_bytes >= (10u << 20);
    if (a.q.zw != 128) {
        if (stream) hipLaunchKernelGGL((pw_u8_walk<STEPS, true, HIGH, true>), grid, dim3(256), lds, s, a);
        else hipLaunchKernelGGL((pw_u8_walk<STEPS, true, HIGH, false>), grid, dim3(256), lds, s, a);
    } else {
        if (stream) hipLaunchKernelGGL((pw_u8_walk<STEPS, false, HIGH, true>), grid, dim3(256), lds, s, a);
        else hipLaunchKernelGGL((pw_u8_walk<STEPS, false, HIGH, false>), grid, dim3(256), lds, s, a);
    }
}
template <int STEPS>
void go(const QPwArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    if (a.q.mult32 >= 0) go2<STEPS, true>(a, grid, lds, s);
    else go2<STEPS, false>(a, grid, lds, s);
}

}  // namespace

bool conv_u8_pw_eligible(const LayerGeom &g, const QuantParams &q, const int *filt_sums, const void *out)
{
    if (g.kh != 1 || g.kw != 1 || g.pt != 0 || g.pl != 0 || g.Ci > 256 || q.amax <= 0 || (!filt_sums && q.zx != 128) || ((uintptr_t)out & 15u))
        return false;
    const size_t M = (size_t)g.N * g.Ho * g.Wo;
    // Staging the filter and the constants costs about as much as a tile of pixels, so there has to be enough output. Measured
    // over 100 layers of 16..256 to 48..480 channels (us, before -> here): at 0.8 M codes 3.25 -> 3.5 (128 -> 48) and 3.7 -> 4.4
    // (256 -> 48), at 1.2 to 1.3 M 4.7 -> 4.5 and 4.2 -> 3.5; one input block is cheap to read again: 16 -> 96 at 1.8 M codes
    // 3.6 -> 3.8, 16 -> 224 at 3.1 M 4.2 -> 4.1. Two output blocks or one are a single group of the other kernels, which never
    // read a pixel twice then: 32 -> 32 at 4.8 M codes 5.4 -> 6.5.
    if (g.Co < 48 || g.Co > (1 << 20) || M * g.Co * (g.Ci > 16 ? 2 : 1) < ((size_t)5 << 19)) return false;
    return M < ((size_t)1 << 31) - 64 && (size_t)g.N * g.Ci * g.H * g.W < kBeyond && M * g.Co < kBeyond && (size_t)g.Co * g.Ci < kBeyond;
}

hipError_t launch_conv_u8_pw(const unsigned char *in, const unsigned char *filt, unsigned char *out, const LayerGeom &g,
                             const QuantParams &q, const int *filt_sums, hipStream_t s)
{
    QPwArgs a;
    a.in = in; a.filt = filt; a.out = out; a.filt_sums = filt_sums;
    a.W = g.W; a.HW = g.H * g.W; a.Wo = g.Wo; a.HoWo = g.Ho * g.Wo; a.M = g.N * a.HoWo; a.stride = g.stride;
    a.nCib = g.Ci / 16; a.nCob = g.Co / 16;
    a.in_bytes = (unsigned)((size_t)g.N * g.Ci * g.H * g.W); a.filt_bytes = (unsigned)((size_t)g.Co * g.Ci);
    a.out_bytes = (unsigned)((size_t)a.M * g.Co);
    a.dHoWo = make_fastdiv(a.HoWo); a.dWo = make_fastdiv(a.Wo);
    a.q = q;
    const int steps = (a.nCib + 3) / 4;
    a.n_tiles = (a.M + 16 * kWM - 1) / (16 * kWM);
    // shares of at most 40 KB of filter; with few pixels smaller ones, until every compute unit has a workgroup
    const int wgs_x = (a.n_tiles + 3) / 4;
    int share = 40 / steps / 4 * 4;
    share = share < (a.nCob + 3) / 4 * 4 ? share : (a.nCob + 3) / 4 * 4;
    while (share > 4 && (long)wgs_x * ((a.nCob + share - 1) / share) < device_cus()) share = (share / 2 + 3) / 4 * 4;
    a.share = share;
    const int shares = (a.nCob + share - 1) / share;
    const int resident = 16 * device_cus();                    // waves
    const int per_wave = (a.n_tiles * shares + resident - 1) / resident;
    const int n_wg = ((a.n_tiles + per_wave - 1) / per_wave + 3) / 4;
    a.n_waves = n_wg * 4;
    const dim3 grid((unsigned)n_wg, (unsigned)shares);
    const size_t lds = (size_t)share * steps * 1024 + (size_t)share * 64;
    switch (steps) {
        case 1: go<1>(a, grid, lds, s); break;
        case 2: go<2>(a, grid, lds, s); break;
        case 3: go<3>(a, grid, lds, s); break;
        default: go<4>(a, grid, lds, s); break;
    }
    return hipGetLastError();
}

}  // namespace small
