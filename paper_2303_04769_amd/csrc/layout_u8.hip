// Layout change of uint8 tensors at the network's boundary: plain [N][C][H][W] <-> blocked [N][C/Cb][H][W][Cb].
// Bound: HBM and, below some 20 MB, launch and first access (a byte is read and a byte written).
#include "small_internal.h"

namespace small {
namespace {

// Memory words at any byte address (a channel's row of pixels starts wherever C * H * W puts it): the hardware takes
// unaligned global accesses, the type tells the compiler that these are.
struct __attribute__((packed)) Word { unsigned v; };
__device__ __forceinline__ unsigned load_word(const unsigned char *p) { return reinterpret_cast<const Word *>(p)->v; }
__device__ __forceinline__ void store_word(unsigned char *p, unsigned v) { reinterpret_cast<Word *>(p)->v = v; }

// 4 x 4 bytes: byte i of word j <-> byte j of word i
__device__ __forceinline__ void transpose4(unsigned (&w)[4])
{
    const unsigned a = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u), b = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    const unsigned c = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u), d = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    w[0] = __builtin_amdgcn_perm(c, a, 0x05040100u);
    w[1] = __builtin_amdgcn_perm(c, a, 0x07060302u);
    w[2] = __builtin_amdgcn_perm(d, b, 0x05040100u);
    w[3] = __builtin_amdgcn_perm(d, b, 0x07060302u);
}

// CB channels of four neighbouring pixels, w[c] = channel c's word of four pixels, as the 4 * CB bytes of the four
// pixels in memory order (o[k] = bytes 4k .. 4k + 3), and back.
template <int CB>
__device__ __forceinline__ void to_pixels(const unsigned (&w)[CB], unsigned (&o)[CB])
{
    if constexpr (CB % 4 == 0) {
#pragma unroll
        for (int q = 0; q < CB / 4; ++q) {
            unsigned t[4] = {w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
            transpose4(t);
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j * (CB / 4) + q] = t[j];
        }
    } else {
#pragma unroll
        for (int k = 0; k < CB; ++k) {
            o[k] = 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) o[k] |= ((w[(4 * k + t) % CB] >> (8 * ((4 * k + t) / CB))) & 255u) << (8 * t);
        }
    }
}
template <int CB>
__device__ __forceinline__ void to_channels(const unsigned (&o)[CB], unsigned (&w)[CB])
{
    if constexpr (CB % 4 == 0) {
#pragma unroll
        for (int q = 0; q < CB / 4; ++q) {
            unsigned t[4] = {o[q], o[CB / 4 + q], o[2 * (CB / 4) + q], o[3 * (CB / 4) + q]};
            transpose4(t);
#pragma unroll
            for (int j = 0; j < 4; ++j) w[4 * q + j] = t[j];
        }
    } else {
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            w[c] = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) w[c] |= ((o[(j * CB + c) / 4] >> (8 * ((j * CB + c) % 4))) & 255u) << (8 * j);
        }
    }
}

// A lane owns four neighbouring pixels of one (image, channel block) plane: one word of four pixels per channel on the
// plain side, 4 * CB contiguous bytes on the blocked side, the transposition between them in registers (byte permutes,
// no LDS). The plain side is 256 contiguous bytes per wave and access; the CB accesses of either side are independent,
// so a lane has its whole share of the tensor in flight at once. Where a plane's pixels are no multiple of four its last lane
// takes the last four, some of which the lane before it writes too, with the same bytes (moving the rest byte by byte took
// that lane up to 48 memory round trips: 32 channels 63x1, 43 images 8.3 us, 2.8 this way). Planes of at least four pixels.
template <int CB, bool UNPACK>
__global__ void __launch_bounds__(256) pack_u8_words(const unsigned char *src, unsigned char *dst, int HW, int groups,
                                                     FastDiv div_groups, int total)
{
    const int i = (int)(blockIdx.x * 256u + threadIdx.x);
    if (i >= total) return;
    const int plane = div_groups.div(i), group = i - plane * groups;          // plane = n * nCb + cb
    const int pix = group + 1 < groups ? group * 4 : HW - 4;
    const size_t base = (size_t)plane * HW * CB;                              // of the plane, in either layout
    const unsigned char *in = src + base + (UNPACK ? (size_t)pix * CB : (size_t)pix);
    unsigned char *out = dst + base + (UNPACK ? (size_t)pix : (size_t)pix * CB);
    unsigned w[CB], o[CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) w[c] = load_word(UNPACK ? in + 4 * c : in + (size_t)c * HW);
    if (UNPACK) to_channels<CB>(w, o);
    else to_pixels<CB>(w, o);
#pragma unroll
    for (int c = 0; c < CB; ++c) store_word(UNPACK ? out + (size_t)c * HW : out + 4 * c, o[c]);
}

// Any block size: one lane per byte of the blocked tensor.
__global__ void __launch_bounds__(256) pack_u8_kernel(const unsigned char *src, unsigned char *dst, int C, int HW, int Cb,
                                                      size_t total, int unpack)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;   // index into the blocked tensor
    if (i >= total) return;
    const int c_in = (int)(i % Cb);
    const size_t t = i / Cb;
    const int pix = (int)(t % HW);
    const size_t t2 = t / HW;          // n * nCb + cb
    const int nCb = C / Cb;
    const int cb = (int)(t2 % nCb);
    const size_t n = t2 / nCb;
    const size_t j = (n * C + (size_t)cb * Cb + c_in) * HW + pix;
    if (unpack) dst[j] = src[i];
    else dst[i] = src[j];
}

template <int CB>
void launch_words(const unsigned char *src, unsigned char *dst, long planes, int HW, bool unpack, hipStream_t s)
{
    const int groups = (int)((HW + 3L) / 4);
    const int total = (int)(planes * groups);
    const dim3 grid((unsigned)((total + 255) / 256));
    if (unpack) hipLaunchKernelGGL((pack_u8_words<CB, true>), grid, dim3(256), 0, s, src, dst, HW, groups, make_fastdiv(groups), total);
    else hipLaunchKernelGGL((pack_u8_words<CB, false>), grid, dim3(256), 0, s, src, dst, HW, groups, make_fastdiv(groups), total);
}

}  // namespace

// The word kernel for the block sizes of the networks' inputs (1, 3) and of their tensors (4, 8, 16), a lane per byte for the
// others, for planes of fewer than four pixels, and for small tensors in 16-byte blocks whose planes are small or no multiple of
// four pixels, where sixteen scattered accesses in a row are the lane's time. Kernel us, a lane per byte / words: 64x128x28x28
// packed 19.4 / 4.7, back 20.3 / 3.5; 256x3x32x32 in one block 3.9 / 2.3; 1x16x83x83 (not taken) 2.4 / 2.7; 3000 planes of 2x2
// (not taken) 2.6 / 4.0; 300 thousand codes of 5x5 planes 2.9 / 3.1, a million 4.6 / 3.3; a million of 2x2 ones 4.6 / 4.1.
hipError_t launch_pack_u8(const unsigned char *src, unsigned char *dst, int N, int C, int H, int W, int Cb, bool unpack,
                          hipStream_t s)
{
    const size_t total = (size_t)N * C * H * W;
    const int HW = H * W;
    const long planes = (long)N * (C / Cb);
    const bool scattered = Cb == 16 && total < (HW == 4 ? 800000u : 300000u) && (HW < 64 || HW % 4 != 0);
    if (HW >= 4 && !scattered && planes * ((HW + 3L) / 4) < (1L << 31) - 256) {
        switch (Cb) {
            case 1: launch_words<1>(src, dst, planes, HW, unpack, s); return hipGetLastError();
            case 3: launch_words<3>(src, dst, planes, HW, unpack, s); return hipGetLastError();
            case 4: launch_words<4>(src, dst, planes, HW, unpack, s); return hipGetLastError();
            case 8: launch_words<8>(src, dst, planes, HW, unpack, s); return hipGetLastError();
            case 16: launch_words<16>(src, dst, planes, HW, unpack, s); return hipGetLastError();
            default: break;
        }
    }
    hipLaunchKernelGGL(pack_u8_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, src, dst, C, HW, Cb, total,
                       unpack ? 1 : 0);
    return hipGetLastError();
}

}  // namespace small
