// fp32 convolution on the bf16 matrix cores, each value as the sum of three bf16 ones: 3x3 windows at stride 1, an even number of input
// blocks, layers of about half a 256-pixel x 64-channel tile per compute unit or more. conv_split3.hip says which products, at which
// scale, and with what error; here two more of them where the fp32 instruction is the other choice (products()). A matrix
// instruction's 32 products are of another 32 channels than there (lane group g holds channels 4g .. 4g + 3 of two blocks, there
// eight of one), so results differ in the last bits (1.7e-7 of the result, 2-norm); their error is the same.
//
// Bound: the matrix cores' power. conv16_split3 spends 3570 cycles of a compute unit on what is 1536 cycles of matrix instructions:
// its waves own 32 pixels x 64 channels, whose operands take LDS 94 of its 128 bytes a cycle, and its two workgroups meet at two
// barriers a step with the splitting between them. Here a wave owns 64 x 64, one wave on a SIMD, so 62 bytes a cycle; and as the
// bf16 instruction of 16 cycles leaves room for two vector instructions behind it (measured: one or two cost nothing, a third four
// to six cycles; beside the fp32 instruction every one costs its time), everything else is cut into pieces of one or two vector
// instructions or one LDS or memory instruction, and one piece stands in every gap between two matrix instructions:
//   step s (a tap of two input blocks): operands of the next pixels and of step s + 1's filter from LDS; the filter of step s + 2 is
//   split and written to the slot that step s has read, that of step s + 3 requested; of the next chunk of two input blocks a
//   sixth of the input is requested (steps 0, 1) or split and written (2 .. 7: the parts h and m, which have two places; the
//   third parts, which have one, in the last step, whose own are in registers by then). One barrier a step.
// The workgroup stays and walks over tiles, so that the pipeline runs on across them. The instructions are pinned where they stand:
// the accumulators are tied operands of an asm statement, and empty asm statements keep the pieces from being moved together.
// 1536 cycles of matrix instructions take some 2000 here, and the clock falls from 2.2 to 2.05 GHz and less, by the device: fewer cycles
// (2300 to 2000 a step) brought nothing any more at the largest layers. us, conv16_split3 / here, several devices: 64 channels 56 x 56, 256
// images 339 to 343 / 305 to 316 (188 to 194 TFLOP/s of fp32 work), 128 channels 28 x 28, 64 images 96 / 79 to 82, 32 images 50 /
// 40; with the fp32 instruction / here (eight products): 160 channels 24 x 24, 27 images 62 / 56, 192 channels 106 x 14, 10 images 90 / 65.
#include "small_internal.h"

#include <algorithm>

namespace small {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

constexpr float kScale = 16777216.f, kUnscale = 1.f / (16777216.f * 16777216.f);      // as in conv_split3.hip
constexpr int kTaps = 9;
constexpr float kMost = 0x1.fep127f;   // the largest bf16: a scaled value above may round to an infinity

struct WideArgs {
    const float *in, *filt, *res, *bn;
    float *out;
    int H, W, HoWo, Wo;
    int Ws, strips, HoWs, M;           // as in conv_u8_tile.hip: columns of a strip, strips per image, pixels of a strip, of all
    int nCib, nCob, pt, pl;
    int Hv, Wv, nCibH, n_chunks, n_cot, n_tiles, epilogue;
    unsigned in_bytes, filt_bytes;
    FastDiv dHoWs, dWs, dWv, dHv, dStrips, dCt;
};

template <int N> struct Num { static constexpr int value = N; };
template <int... I> struct Seq {};
template <int N, int... I> struct MakeSeq : MakeSeq<N - 1, N - 1, I...> {};
template <int... I> struct MakeSeq<0, I...> { typedef Seq<I...> type; };
template <int... I, class F>
__device__ __forceinline__ void each_of(Seq<I...>, F &&f) { (f(Num<I>{}), ...); }
template <int N, class F>
__device__ __forceinline__ void each(F &&f) { each_of(typename MakeSeq<N>::type{}, f); }

// Two values on their way to three bf16 parts each, in eight pieces of one or two vector instructions. The empty statements keep
// a piece where it stands: the compiler would move it to where its result is needed.
struct Pair { float u, v, a, b; unsigned part[3]; };
__device__ __forceinline__ void stay(float x, float y) { asm volatile("" :: "v"(x), "v"(y)); }
template <int PIECE>
__device__ __forceinline__ void split_piece(Pair &s)
{
    constexpr int n = PIECE / 3;
    if constexpr (PIECE == 0) {
        s.u *= kScale; s.v *= kScale;
        stay(s.u, s.v);
    } else if constexpr (PIECE % 3 == 1) {
        s.part[n] = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{s.u, s.v}, bf16x2));
        asm volatile("" :: "v"(s.part[n]));
    } else if constexpr (PIECE % 3 == 2) {
        s.a = __builtin_bit_cast(float, s.part[n] << 16);
        s.b = __builtin_bit_cast(float, s.part[n] & 0xffff0000u);
        stay(s.a, s.b);
    } else {
        s.u -= s.a; s.v -= s.b;
        stay(s.u, s.v);
    }
}

// The compiler does not see matrix instructions in the asm statements and puts in no wait states round them: what writes their operands
// or reads their results stands on the other side of one of these, whose operands keep it there. 1: two wait states, from a vector
// instruction to a matrix instruction; 15: sixteen, from a result to its use, which needs at most eleven.
template <int STATES>
__device__ __forceinline__ void wait_states(floatx4 (&u)[4], floatx4 (&v)[4])
{
    asm volatile("s_nop %8" : "+a"(u[0]), "+a"(u[1]), "+a"(u[2]), "+a"(u[3]), "+a"(v[0]), "+a"(v[1]), "+a"(v[2]), "+a"(v[3]) : "n"(STATES));
}

// A workgroup's tile is kTM pixels by kNCT output blocks, a wave's part of it WM x WN groups of 16.
constexpr int WM = 4, WN = 4, kWavesM = 4, kWavesN = 1;
constexpr int kTM = 16 * WM * kWavesM, kNCT = WN * kWavesN;
constexpr int kEntries = 384;          // staged input entries of a tile, at most

template <int PRODUCTS>
__global__ void __launch_bounds__(256, 1) conv16_split3_wide(WideArgs a)
{
    constexpr int R = kEntries / 64, EC = kEntries + 1;        // (an entry more: planes four banks apart)
    static_assert(kWavesM * kWavesN == 4 && kNCT == 4 && kEntries % 64 == 0 && R == 6, "a block of the filter for each wave; six parts of a chunk's input");
    constexpr int PLANE = EC * 16, PART_B = 4 * PLANE;         // bytes

    extern __shared__ uintx4 lds[];
    uintx4 *const A = lds;                                     // two of [block][part][lane]
    char *const B = reinterpret_cast<char *>(lds + 2 * kNCT * 3 * 64);      // [quad][entry]: l; then two times h, m

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p = lane & 15, g = lane >> 4;
    const int wave_m = wave % kWavesM, wave_n = wave / kWavesM;
    const int sp = (tid >> 4) & 3, se = (tid & 15) + 16 * (tid >> 6);      // staged: quad sp, entries se + 64 k
    const unsigned plane_bytes = (unsigned)(a.H * a.W) * 64u;

    // ---- the tile whose input and filter are requested next
    int cob_aim, vr0_aim, nE_aim, ok_aim;
    int row[R], col[R];
    unsigned at[R] = {};
    each<R>([&](auto k) { row[k.value] = quotient(a.dWv, se + 64 * k.value); col[k.value] = se + 64 * k.value - row[k.value] * a.Wv - a.pl; });
    auto aim = [&](int t) __attribute__((always_inline)) {
        ok_aim = t < a.n_tiles;
        t = min(t, a.n_tiles - 1);
        const int mt = quotient(a.dCt, t), m0 = mt * kTM;
        cob_aim = (t - mt * a.n_cot) * kNCT;
        const int n0 = quotient(a.dHoWs, m0);
        vr0_aim = n0 * a.Hv + quotient(a.dWs, m0 - n0 * a.HoWs);
        const int m1 = min(m0 + kTM, a.M) - 1;
        const int n1 = quotient(a.dHoWs, m1), vr1 = n1 * a.Hv + quotient(a.dWs, m1 - n1 * a.HoWs) + 2;
        nE_aim = ok_aim ? (vr1 - vr0_aim + 1) * a.Wv : 0;
    };
    // where entry se + 64 k of that tile lies, in ten pieces
    int p_vr = 0, p_ns = 0, p_iy = 0, p_n = 0, p_ix = 0;
    unsigned p_hi = 0;
    const unsigned one_v = a.dHv.d == 1 ? ~0u : 0u, one_s = a.dStrips.d == 1 ? ~0u : 0u;       // (quotient() in two halves)
    auto place = [&](auto K, auto PIECE) __attribute__((always_inline)) {
        constexpr int k = K.value, piece = PIECE.value;
        if constexpr (piece == 0) {
            p_vr = vr0_aim + row[k];
            p_hi = __umulhi((unsigned)p_vr, a.dHv.magic);
        } else if constexpr (piece == 1) {
            p_ns = (int)((p_hi + ((unsigned)p_vr & one_v)) >> a.dHv.shift);
        } else if constexpr (piece == 2) {
            p_iy = p_vr - p_ns * a.Hv - a.pt;
        } else if constexpr (piece == 3) {
            p_hi = __umulhi((unsigned)p_ns, a.dStrips.magic);
        } else if constexpr (piece == 4) {
            p_n = (int)((p_hi + ((unsigned)p_ns & one_s)) >> a.dStrips.shift);
        } else if constexpr (piece == 5) {
            p_ix = p_ns - p_n * a.strips;
        } else if constexpr (piece == 6) {
            p_ix = col[k] + p_ix * a.Ws;
        } else if constexpr (piece == 7) {
            at[k] = (unsigned)(p_n * a.nCibH + p_iy);
        } else if constexpr (piece == 8) {
            at[k] = at[k] * (unsigned)a.W + (unsigned)p_ix;
        } else {
            const bool inside = (se + 64 * k < nE_aim) & ((unsigned)p_iy < (unsigned)a.H) & ((unsigned)p_ix < (unsigned)a.W);
            at[k] = inside ? at[k] * 64u + sp * 16u : kBeyond;
        }
        asm volatile("" :: "v"(at[k]), "v"(p_vr), "v"(p_ns), "v"(p_iy), "v"(p_n), "v"(p_ix), "v"(p_hi));
    };
    floatx4 iv[R][2];
    const __amdgpu_buffer_rsrc_t src = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.in), 0, a.in_bytes, kRawBuffer);
    const __amdgpu_buffer_rsrc_t flt = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.filt), 0, a.filt_bytes, kRawBuffer);
    auto in_load = [&](int k, int half, unsigned chunk) __attribute__((always_inline)) {       // chunk: the byte its first block starts at
        iv[k][half] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, at[k], chunk + half * plane_bytes, 0));
    };
    // ---- filter: wave w brings output block w of the tile's; lane (p, g) of it the input channels 4g .. 4g + 3 of two blocks
    float fr[8];
    // (an output block that the layer does not have: beyond the descriptor)
    auto f_lanes = [&](int cob, bool more) __attribute__((always_inline)) { return (more & (cob + wave < a.nCob)) ? (unsigned)(g * 256 + p * 4) : kBeyond; };
    auto f_block = [&](int cob, int ch) __attribute__((always_inline)) { return (unsigned)((min(cob + wave, a.nCob - 1) * a.nCib + 2 * ch) * kTaps) * 1024u; };
    auto f_load = [&](int k, unsigned lanes, unsigned block, int tap) __attribute__((always_inline)) {      // channel 4g + (k & 3) of block k >> 2
        fr[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(flt, lanes + 64u * (k & 3), block + ((k >> 2) * kTaps + tap) * 1024u, 0));
    };
    Pair fp[4], ip[4];
    uintx4 pl[R];

    uintx4 *const a_write = A + wave * 3 * 64 + lane;
    const uintx4 *const a_read = A + wave_n * WN * 3 * 64 + lane;
    int par = 0;                                               // slot of the chunk's step 0
    constexpr int SLOT = kNCT * 3 * 64;
    auto f_write = [&](int slot, int s) __attribute__((always_inline)) {
        a_write[slot * SLOT + s * 64] = uintx4{fp[0].part[s], fp[1].part[s], fp[2].part[s], fp[3].part[s]};
    };
    auto f_take = [&](int q) __attribute__((always_inline)) { fp[q].u = fr[2 * q]; fp[q].v = fr[2 * q + 1]; };
    auto i_take = [&](int k, int q) __attribute__((always_inline)) { ip[q].u = iv[k][q >> 1][2 * (q & 1)]; ip[q].v = iv[k][q >> 1][2 * (q & 1) + 1]; };
    auto i_put = [&](int k) __attribute__((always_inline)) { pl[k] = uintx4{ip[0].part[2], ip[1].part[2], ip[2].part[2], ip[3].part[2]}; };
    int bpar = 0;                                              // which h, m are the current chunk's
    char *const b_here = B + sp * PLANE + se * 16;
    auto b_write = [&](int k, int s, int buf) __attribute__((always_inline)) {
        const uintx4 v = s == 2 ? pl[k] : uintx4{ip[0].part[s], ip[1].part[s], ip[2].part[s], ip[3].part[s]};
        *reinterpret_cast<uintx4 *>(b_here + (s == 2 ? 0 : (1 + 2 * buf + s) * PART_B) + k * 1024) = v;
    };
    auto arrive = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0xc07f);                    // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    // ---- first tile
    int tile = (int)xcd_contiguous(blockIdx.x, gridDim.x), ch = 0;
    aim(tile);
    int cob0 = cob_aim, vr0 = vr0_aim;
    unsigned lanes = f_lanes(cob0, true), block = f_block(cob0, 0);
    each<R>([&](auto k) {
        each<10>([&](auto piece) { place(k, piece); });
        in_load(k.value, 0, 0); in_load(k.value, 1, 0);
    });
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        each<8>([&](auto k) { f_load(k.value, lanes, block, s); });
        each<4>([&](auto q) { f_take(q.value); each<8>([&](auto piece) { split_piece<piece.value>(fp[q.value]); }); });
        each<3>([&](auto part) { f_write(s, part.value); });
    }
    each<8>([&](auto k) { f_load(k.value, lanes, block, 2); });
    each<R>([&](auto k) {
        each<4>([&](auto q) { i_take(k.value, q.value); each<8>([&](auto piece) { split_piece<piece.value>(ip[q.value]); }); });
        i_put(k.value);
        each<3>([&](auto s) { b_write(k.value, s.value, 0); });
    });
    arrive();

    const char *base[WM];
    auto rebase = [&]() __attribute__((always_inline)) {
        const int m0 = quotient(a.dCt, tile) * kTM;
#pragma unroll
        for (int wm = 0; wm < WM; ++wm) {
            const int m = min(m0 + (wave_m * WM + wm) * 16 + p, a.M - 1);
            const int n = quotient(a.dHoWs, m), rem = m - n * a.HoWs, oh = quotient(a.dWs, rem);
            base[wm] = B + g * PLANE + ((n * a.Hv + oh - vr0) * a.Wv + (rem - oh * a.Ws)) * 16;
        }
    };
    rebase();
    const int row_b = a.Wv * 16;

    floatx4 acc[WM][WN], low[WM][WN];
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int wm = 0; wm < WM; ++wm) {
#pragma unroll
            for (int wn = 0; wn < WN; ++wn) acc[wm][wn] = low[wm][wn] = floatx4{0.f, 0.f, 0.f, 0.f};
            wait_states<1>(acc[wm], low[wm]);
        }
    };
    clear();

    bf16x8 fa[2][WN][3], fb[2][3], fl[WM];                     // fl: the last parts of a chunk's last step
    auto a_get = [&](int set, int slot, int wn, int s) __attribute__((always_inline)) { fa[set][wn][s] = __builtin_bit_cast(bf16x8, a_read[slot * SLOT + (wn * 3 + s) * 64]); };
    auto b_get = [&](int wm, int tap, int s, int buf) __attribute__((always_inline)) {
        const int y = tap / 3, z = tap - 3 * y;
        const char *from = s == 2 ? base[wm] + y * row_b : base[wm] + (y * row_b + (1 + 2 * buf) * PART_B) + s * PART_B;
        return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uintx4 *>(from + z * 16));
    };
    each<WN>([&](auto wn) { each<3>([&](auto s) { a_get(0, 0, wn.value, s.value); }); });
    each<3>([&](auto s) { fb[0][s.value] = b_get(0, 0, s.value, 0); });

    // ---- results of this wave's part of tile t
    auto put = [&](int t, const floatx4 (&v)[WM][WN]) __attribute__((always_inline)) {
        const int mt = quotient(a.dCt, t), m0 = mt * kTM + wave_m * WM * 16, cob_w = (t - mt * a.n_cot) * kNCT + wave_n * WN;
#pragma unroll
        for (int wm = 0; wm < WM; ++wm) {
            const int m = m0 + wm * 16 + p;
            const int ns = quotient(a.dHoWs, min(m, a.M - 1)), rem = m - ns * a.HoWs, oh = quotient(a.dWs, rem);
            const int n = quotient(a.dStrips, ns), ow = rem - oh * a.Ws + (ns - n * a.strips) * a.Ws;
            if (m < a.M && ow < a.Wo) {
#pragma unroll
                for (int wn = 0; wn < WN; ++wn) {
                    const int cob = cob_w + wn;
                    if (cob >= a.nCob) break;
                    const size_t o = (((size_t)n * a.nCob + cob) * a.HoWo + oh * a.Wo + ow) * 16 + g * 4;
                    floatx4 y = v[wm][wn];
                    if (a.epilogue & EPI_BN) {
                        const float *c = a.bn + cob * 16 + g * 4;
                        const floatx4 sc = *reinterpret_cast<const floatx4 *>(c), sh = *reinterpret_cast<const floatx4 *>(c + a.nCob * 16);
                        y.x = fmaf(y.x, sc.x, sh.x); y.y = fmaf(y.y, sc.y, sh.y); y.z = fmaf(y.z, sc.z, sh.z); y.w = fmaf(y.w, sc.w, sh.w);
                    }
                    if (a.epilogue & EPI_ADD) y += *reinterpret_cast<const floatx4 *>(a.res + o);
                    if (a.epilogue & EPI_RELU) {
                        y.x = y.x > 0.f ? y.x : 0.f; y.y = y.y > 0.f ? y.y : 0.f;
                        y.z = y.z > 0.f ? y.z : 0.f; y.w = y.w > 0.f ? y.w : 0.f;
                    }
                    *reinterpret_cast<floatx4 *>(a.out + o) = y;
                }
            }
        }
    };
    unsigned long long bad = 0;                                // rounds of tiles whose sums here are not finite (kMaxRounds bits)
    int round = 0;

    // the chunk behind the current one: of this tile or the first of the next
    auto behind = [&](int &t, int &c) __attribute__((always_inline)) {
        const bool ends = c + 1 == a.n_chunks;
        t += ends ? (int)gridDim.x : 0;
        c = ends ? 0 : c + 1;
    };
    int t2 = tile, ch2 = 0;
    behind(t2, ch2);
    aim(t2);
    for (;;) {
        const int cob2 = cob_aim, vr2 = vr0_aim, ok2 = ok_aim;
        const unsigned lanes2 = f_lanes(cob2, ok2), block2 = f_block(cob2, ch2), chunk2 = 2 * ch2 * plane_bytes;
        int t3 = t2, ch3 = ch2;
        behind(t3, ch3);

        each<kTaps>([&](auto S) {
            constexpr int s = S.value, cur = s & 1, nxt = cur ^ 1;
            const int my_slot = cur ^ par;                     // filter of this step, whose slot step s + 2 takes
            auto filter_work = [&](auto I) __attribute__((always_inline)) {        // 0 .. 35: splits step s + 2's
                constexpr int i = I.value, q = i / 8;
                if constexpr (i < 32) {
                    if constexpr (i % 8 == 0) f_take(q);
                    split_piece<i % 8>(fp[q]);
                } else if constexpr (i < 35) f_write(my_slot, i - 32);
            };
            auto input_work = [&](auto I) __attribute__((always_inline)) {         // 0 .. 35: the next chunk's input
                constexpr int i = I.value;
                if constexpr (s < 2) {                         // requested in two steps,
                    constexpr int k = s * (R / 2) + i / 12, piece = i % 12;
                    if constexpr (k < (s + 1) * (R / 2)) {
                        if constexpr (piece < 10) place(Num<k>{}, Num<piece>{});
                        else in_load(k, piece - 10, chunk2);
                    }
                } else if constexpr (s - 2 < R) {              // split in the next six; h and m have room beside the current ones
                    constexpr int k = s - 2, q = i / 8;
                    if constexpr (i < 32) {
                        if constexpr (i % 8 == 0) i_take(k, q);
                        split_piece<i % 8>(ip[q]);
                    } else if constexpr (i < 34) b_write(k, i - 32, bpar ^ 1);
                    else if constexpr (i == 34) i_put(k);
                } else if constexpr (i % 4 == 0 && i / 4 < R) b_write(i / 4, 2, 0);           // l takes the current one's place
                if constexpr (s == 2 && i == 35) aim(t3);
            };
            each<WM>([&](auto W) {
                constexpr int wm = W.value;
                each<PRODUCTS * WN>([&](auto TN) {
                    constexpr int t = TN.value / WN, wn = TN.value % WN;
                    constexpr int pa[8] = {0, 1, 0, 1, 2, 0, 1, 2}, pb[8] = {0, 0, 1, 1, 0, 2, 2, 1};
                    floatx4 &c = t == 0 ? acc[wm][wn] : low[wm][wn];
                    const bf16x8 x = s == kTaps - 1 && pb[t] == 2 ? fl[wm] : fb[wm & 1][pb[t]];
                    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "a"(fa[cur][wn][pa[t]]), "v"(x));
                    // every fourth gap reads an operand, of the next pixels or of the next step's filter, and requests some of the
                    // filter of step s + 3; the others take turns at the filter's and the input's splitting
                    if constexpr (wn == 0) {
                        if constexpr (t < 3) {
                            if constexpr (wm + 1 < WM) {
                                if constexpr (s < kTaps - 1 || t < 2) fb[(wm + 1) & 1][t] = b_get(wm + 1, s, t, bpar);
                            } else if constexpr (s < kTaps - 1) {
                                if constexpr (s < kTaps - 2 || t < 2) fb[0][t] = b_get(0, s + 1, t, bpar);
                            }
                        } else if constexpr (t < 6) {
                            constexpr int n = wm * 3 + t - 3;
                            if constexpr (n < 3 * WN) a_get(nxt, my_slot ^ 1, n / 3, n % 3);
                        }
                        // (values 2q and 2q + 1 are taken in piece 8q of the filter's, before)
                        if constexpr (t == 1 || t == 3) {
                            constexpr int k = 2 * wm + t / 2, ahead = s + 3;
                            if constexpr (ahead < kTaps) f_load(k, lanes, block, ahead);
                            else f_load(k, lanes2, block2, ahead - kTaps);
                        }
                        if constexpr (s == kTaps - 2 && t == 5) fl[wm] = b_get(wm, s + 1, 2, bpar);
                    } else {
                        constexpr int r = (wm * PRODUCTS + t) * (WN - 1) + wn - 1;
                        if constexpr (r % 2 == 0) filter_work(Num<r / 2>{});
                        else input_work(Num<r / 2>{});
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
            arrive();
        });
        par ^= 1;
        bpar ^= 1;
        if (t2 != tile) {
            wait_states<15>(acc[0], low[0]);
#pragma unroll
            for (int wm = 1; wm < WM; ++wm) wait_states<0>(acc[wm], low[wm]);      // (behind it, as volatile statements stay in order)
            float most = 0.f;                                  // the largest magnitude, or NaN
#pragma unroll
            for (int wm = 0; wm < WM; ++wm)
#pragma unroll
                for (int wn = 0; wn < WN; ++wn) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc[wm][wn][r] = (acc[wm][wn][r] + low[wm][wn][r]) * kUnscale;
                    most = __builtin_elementwise_maximum(most, __builtin_elementwise_maximum(__builtin_fabsf(acc[wm][wn].x), __builtin_fabsf(acc[wm][wn].y)));
                    most = __builtin_elementwise_maximum(most, __builtin_elementwise_maximum(__builtin_fabsf(acc[wm][wn].z), __builtin_fabsf(acc[wm][wn].w)));
                }
            if (__ballot(!(most < __builtin_inff()))) bad |= 1ull << round;
            else put(tile, acc);
            ++round;
            if (!ok2) break;
            clear();
            tile = t2; cob0 = cob2; vr0 = vr2;
            rebase();
        }
        ch = ch2; t2 = t3; ch2 = ch3; lanes = lanes2; block = block2;
        each<3>([&](auto s) { fb[0][s.value] = b_get(0, 0, s.value, bpar); });
        each<WN>([&](auto wn) { each<3>([&](auto s) { fa[0][wn.value][s.value] = fa[1][wn.value][s.value]; }); });
#pragma unroll
        for (int wn = 0; wn < WN; ++wn) asm volatile("s_nop 1" : "+a"(fa[0][wn][0]), "+a"(fa[0][wn][1]), "+a"(fa[0][wn][2]));
    }

    // ---- the tiles whose sums were not all finite: some value there, or a sum, is not finite or not so at the scale of the parts.
    // The fp32 instruction, operands from memory, the next step's on their way (lane (p, g): input channels 4g .. 4g + 3 of its
    // pixels, filter values [4g + r][p]), or, with such a value in the filter, plain fp32: a tap outside the image does not count,
    // whatever its weight (an infinite one times the zero read there would).
    for (int t = (int)xcd_contiguous(blockIdx.x, gridDim.x), rnd = 0; bad && t < a.n_tiles; t += (int)gridDim.x, ++rnd) {
        if (!(bad >> rnd & 1)) continue;
        const int steps = a.nCib * kTaps, mt = quotient(a.dCt, t), m0 = mt * kTM + wave_m * WM * 16;
        const int cob_w = (t - mt * a.n_cot) * kNCT + wave_n * WN;
        int ih0[WM], iw0[WM], at0[WM];
        floatx4 v[WM][WN];
#pragma unroll
        for (int wm = 0; wm < WM; ++wm) {
            const int m = min(m0 + wm * 16 + p, a.M - 1);
            const int ns = quotient(a.dHoWs, m), rem = m - ns * a.HoWs, oh = quotient(a.dWs, rem);
            const int n = quotient(a.dStrips, ns), ow = rem - oh * a.Ws + (ns - n * a.strips) * a.Ws;
            ih0[wm] = oh - a.pt;
            iw0[wm] = ow - a.pl;
            at0[wm] = n * a.nCib * a.H * a.W + ih0[wm] * a.W + iw0[wm];
#pragma unroll
            for (int wn = 0; wn < WN; ++wn) v[wm][wn] = floatx4{0.f, 0.f, 0.f, 0.f};
        }
        auto inside = [&](int wm, int y, int z) __attribute__((always_inline)) {
            return ((unsigned)(ih0[wm] + y) < (unsigned)a.H) & ((unsigned)(iw0[wm] + z) < (unsigned)a.W);
        };
        auto request = [&](int s, floatx4 (&xs)[WM], float (&ws)[WN][4]) __attribute__((always_inline)) {
            const int sc = min(s, steps - 1), cib = sc / kTaps, tap = sc - cib * kTaps, y = tap / 3, z = tap - 3 * y;
#pragma unroll
            for (int wm = 0; wm < WM; ++wm) {
                const unsigned from = (unsigned)(at0[wm] + cib * a.H * a.W + y * a.W + z) * 64u + g * 16u;
                xs[wm] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(src, inside(wm, y, z) ? from : kBeyond, 0, 0));
            }
#pragma unroll
            for (int wn = 0; wn < WN; ++wn) {
                const unsigned from = cob_w + wn < a.nCob ? (unsigned)((cob_w + wn) * steps + sc) * 1024u + g * 256u + p * 4u : kBeyond;
#pragma unroll
                for (int r = 0; r < 4; ++r) ws[wn][r] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(flt, from + 64u * r, 0, 0));
            }
        };
        float worst = 0.f;
        for (unsigned i = lane; i < (unsigned)(min(WN, a.nCob - cob_w) * steps * 256); i += 64)
            worst = __builtin_elementwise_maximum(worst, __builtin_fabsf(a.filt[(size_t)cob_w * steps * 256 + i] * kScale));
        if (!__ballot(!(worst <= kMost))) {
            floatx4 x[2][WM];
            float w[2][WN][4];
            request(0, x[0], w[0]);
            for (int s = 0; s < steps; s += 2) {
#pragma unroll
                for (int k = 0; k < 2; ++k) {
                    request(s + k + 1, x[k ^ 1], w[k ^ 1]);
                    if (s + k < steps) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int wm = 0; wm < WM; ++wm)
#pragma unroll
                                for (int wn = 0; wn < WN; ++wn)
                                    v[wm][wn] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[k][wn][r], x[k][wm][r], v[wm][wn], 0, 0, 0);
                    }
                }
            }
        } else {
            for (int s = 0; s < steps; ++s) {
                const int tap = s % kTaps, y = tap / 3, z = tap - 3 * y;
                floatx4 x[WM];
                float w[WN][4];
                request(s, x, w);
#pragma unroll
                for (int wm = 0; wm < WM; ++wm)
#pragma unroll
                    for (int wn = 0; wn < WN; ++wn) {
                        floatx4 u = {0.f, 0.f, 0.f, 0.f};      // (sixteen products first: a chain of all would lose more bits)
#pragma unroll
                        for (int c = 0; c < 16; ++c) {
                            const float xc = __shfl(x[wm][c & 3], (c >> 2) * 16 + p);
#pragma unroll
                            for (int r = 0; r < 4; ++r) u[r] = fmaf(xc, __shfl(w[wn][c & 3], (c >> 2) * 16 + g * 4 + r), u[r]);
                        }
                        if (inside(wm, y, z)) v[wm][wn] += u;
                    }
            }
        }
        put(t, v);
    }
}

constexpr size_t kLds = (size_t)2 * kNCT * 3 * 1024 + (size_t)20 * (kEntries + 1) * 16;
constexpr int kStrip = 16;             // output columns of a strip, at most
// Tiles that a workgroup walks over, at most: one bit of `bad` for each. A tile that is not finite must be computed again on its own,
// not with others that are stored already, for its result may stand in the residual's place. Layers of more rounds get a second,
// third, ... set of workgroups, which start where others end (64 channels 56x56, 1400 images: 34 + 34 rounds instead of 67).
constexpr int kMaxRounds = 64;

struct WidePlan { bool ok; int strips, Ws; long tiles; };

WidePlan plan_wide(const LayerGeom &g)
{
    WidePlan o;
    o.ok = false;
    const int nCib = g.Ci / 16, Hv = g.Ho + 2;
    if (g.Cib != 16 || g.Cob != 16 || g.kh != 3 || g.kw != 3 || g.stride != 1 || nCib % 2 || (size_t)g.N * g.Ci * g.H * g.W * 4 >= kBeyond ||
        (size_t)g.Co * g.Ci * 36 >= kBeyond)
        return o;
    o.strips = (g.Wo + kStrip - 1) / kStrip;
    o.Ws = (g.Wo + o.strips - 1) / o.strips;
    const long M = (long)g.N * o.strips * g.Ho * o.Ws;
    if (((long)g.N * o.strips + 1) * Hv >= (1L << 31) || M >= (1L << 31) - 1024) return o;
    // the most staged entries a tile needs: its rows, and those around the strips that end inside it
    const long span = (kTM < M ? kTM : M) - 1, rows = (span + o.Ws - 1) / o.Ws + 1;
    const long cross = (long)g.N * o.strips > 1 ? (rows - 1 + g.Ho - 1) / g.Ho : 0;
    const long E = (rows + 2 + 2 * cross) * (o.Ws + 2);
    o.tiles = (M + kTM - 1) / kTM * ((g.Co / 16 + kNCT - 1) / kNCT);
    o.ok = E <= kEntries && o.tiles < (1L << 30);
    return o;
}

}  // namespace

// Products of the parts that are taken. Where conv_split3.hip is the other choice, six, as there. Layers that the fp32 instruction would
// compute keep ml and lm too: without them a product is off by up to 1.9 x 2^-24 of it, which shows in filters of one weight, and with
// them by the 2^-24 of that instruction. 160 channels 24x24, 27 images, six / eight / fp32: one weight, 2-norm 2.60e-8 / 2.53e-8 / 2.53e-8,
// worst 1.56 / 1.00 / 1.00 x 2^-24; dense filters 2.2e-7 / 2.2e-7 / 6.7e-7. They cost a fifth: 46.8 / 55.6 / 62.3 us.
static int products(const LayerGeom &g) { return conv_split3_eligible(g) ? 6 : 8; }

const char *conv_split3_wide_kernel_name(const LayerGeom &g)
{
    return products(g) == 6 ? "conv16_split3_wide<6>" : "conv16_split3_wide<8>";
}

// Where it beats the others: times in us of both sides, here by rounds of tiles. With six products (120 random layers, 4 % root mean
// square): 6.9 a chunk and 2.8 a tile, 1.7 more a chunk when all compute units work, and 6 once, against 2 and the layer's work at
// 178 TFLOP/s, which conv16_split3 reaches with one layer in ten. (Near the line this kernel is ahead by some 5 % where both run in turns
// and no more where each runs for itself, for it draws the clocks down further: 64 channels 56x56, 64 images 94.5 / 88 and 92.9 / 93.5. Of
// 220 random layers 133 are taken, at 0.82 to 0.97 of the time in turns.) With eight (140 random layers, 2.1 %): 8.9, 2.5, 0.7 and 6.2, against 2 and
// the work at 125 TFLOP/s, which the best ones on the fp32 instruction reach: of the 140 it takes 37, at 0.87 of their time, and leaves 12
// that would gain 5 % or more; 60 others that it takes 0.74 to 1.00 of theirs.
bool conv_split3_wide_eligible(const LayerGeom &g)
{
    const WidePlan pl = plan_wide(g);
    if (!pl.ok) return false;
    const long cus = device_cus(), rounds = (pl.tiles + cus - 1) / cus;
    const double chunks = g.Ci / 32, fill = pl.tiles < cus ? (double)pl.tiles / cus : 1.0;
    const double mflop = 18e-6 * g.N * g.Ho * g.Wo * (double)g.Ci * g.Co;
    if (products(g) == 6) return rounds * (6.88 * chunks + 2.75 + 1.73 * fill * chunks) + 5.94 < 2.0 + mflop / 178.0;
    return rounds * (8.93 * chunks + 2.50 + 0.73 * fill * chunks) + 6.22 < 2.0 + mflop / 125.0;
}

template <int PRODUCTS>
static hipError_t run_wide(const WideArgs &a, unsigned groups, hipStream_t s)
{
    const auto kernel = conv16_split3_wide<PRODUCTS>;
    static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
    if (attr != hipSuccess) return attr;
    hipLaunchKernelGGL(kernel, dim3(groups), dim3(256), kLds, s, a);
    return hipGetLastError();
}

hipError_t launch_conv_split3_wide(const float *in, const float *filt, float *out, const float *res, const LayerGeom &g, int epilogue,
                                   hipStream_t s, const float *bn)
{
    const WidePlan pl = plan_wide(g);
    if (!pl.ok) return hipErrorInvalidValue;
    WideArgs a;
    a.in = in; a.filt = filt; a.out = out; a.res = res; a.bn = bn; a.epilogue = epilogue;
    a.H = g.H; a.W = g.W; a.Wo = g.Wo; a.HoWo = g.Ho * g.Wo;
    a.Ws = pl.Ws; a.strips = pl.strips; a.HoWs = g.Ho * pl.Ws; a.M = g.N * pl.strips * a.HoWs;
    a.nCib = g.Ci / 16; a.nCob = g.Co / 16; a.pt = g.pt; a.pl = g.pl;
    a.Hv = g.Ho + 2; a.Wv = pl.Ws + 2; a.nCibH = a.nCib * g.H;
    a.n_chunks = (a.nCib + 1) / 2; a.n_cot = (a.nCob + kNCT - 1) / kNCT; a.n_tiles = (int)pl.tiles;
    a.in_bytes = (unsigned)((size_t)g.N * g.Ci * g.H * g.W * 4); a.filt_bytes = (unsigned)((size_t)g.Co * g.Ci * 36);
    a.dHoWs = make_fastdiv(a.HoWs); a.dWs = make_fastdiv(a.Ws); a.dWv = make_fastdiv(a.Wv); a.dHv = make_fastdiv(a.Hv);
    a.dStrips = make_fastdiv(a.strips); a.dCt = make_fastdiv(a.n_cot);
    const long cus = device_cus(), sets = (pl.tiles + kMaxRounds * cus - 1) / (kMaxRounds * cus);
    const unsigned groups = (unsigned)std::min(pl.tiles, sets * cus);
    return products(g) == 6 ? run_wide<6>(a, groups, s) : run_wide<8>(a, groups, s);
}

}  // namespace small
