// A run of depthwise-separable blocks (dwpw_run.hip says what that is) on one or a few images: a team of workgroups per
// image, one for each 16-channel block of the widest tensor.
//
// What bounds it: latency. One workgroup per image streams every filter of the run through one compute unit and does every
// stage there, some 4 us a block, while the rest of the chip idles. Here workgroup t owns channel block t: it computes the
// pointwise result of that block (its share of the filters is one sixteenth), then, as a depthwise layer maps channel
// blocks on their own, the next block's depthwise layer on it, and hands the result to the team. So a block costs one
// hand-over through memory, one reduction of at most 16 steps and one window pass, a wave per 16 pixels. All sums are those of
// dwpw_run, in its order: the results are the same bits, however many images there are.
// The depthwise-separable CNN, one image, without the packing of its input: 64.3 -> 42.9 us, two images 64.4 -> 43.8, the launch in
// front (2 us) among it; the kernel 29. Some 1.3 us a block are the way of a value to memory and back. Whether all values that a wave
// waits for are there is the maximum of their words: asked one by one, a branch each, it cost 239 spilled scalar registers and 2.4 us.
// With the reduction split over the four waves it was faster by 6 (at the time), but sums in another order: after 26 layers two logits
// near zero can then differ by more than a few 1e-6 of them between an image on its own and in a batch.
// All of a team on one of the chip's eight dies gained nothing (30.1 against 28.9 us for the kernel at the time), nor did waiting
// before the first look (0.07 to 2.9 us slower): values are looked at past the dies' caches either way. What a wave needs for its
// next stage besides results -- taps, window entries, the layer's numbers -- it gets ready while it would be waiting (28.9 -> 26.0).
//
// The hand-over has no flags and no barrier: a word of the exchange area is "not there yet" while it holds kNotYet, a NaN
// with all bits set, which no result is stored as, and the launch in front fills the area with it. A consumer reads the
// values it needs, each in agent scope (which goes past the L2s, of which the chip has eight), until none is kNotYet; a
// value that is there is final. Nothing else is communicated, so nothing has to be ordered.
//
// Every wait ends: a workgroup needs only results of its own team, and the launch is small enough for all teams to be on the chip
// together where one process with its four hardware queues uses it (dwpw_team_exchange). Nothing guarantees that -- several
// processes share a device, a captured run can be replayed on a stream of a few compute units -- so a workgroup that has looked for
// some milliseconds does the whole image by itself, the parts of all of the team in turn, and hands everything on on the way. The
// words and the outputs it stores are the bits that the others store there, so it does not matter who comes first, and one that
// finds its place late finds all it needs.
#include "small_internal.h"

#include <algorithm>

namespace small {
namespace {

constexpr int kTeamWaves = 4;
constexpr int kTeamThreads = kTeamWaves * 64;
constexpr int kTeamMax = 16;              // workgroups of a team = channel blocks of the widest tensor
constexpr int kTeamHeadMost = 16;         // outputs of a head (plan_fusion allows no more)
constexpr int kTeamItems = 16;            // (input block, pixel group) pairs that a wave has in registers
constexpr unsigned kNotYet = ~0u;
constexpr unsigned kOwnTries = 1u << 21;  // for what is known to come: a workgroup's own stores

struct TeamBlock {
    const float *dw, *pw;
    int dw_relu, pw_relu;
    int nCbi, nCbo;
    int Hi, Wi, Ho, Wo, stride, pt, pl;
    FastDiv by_Wo;
};

struct TeamArgs {
    const float *in;
    float *out;
    char *exchange;
    unsigned exchange_bytes;              // per image
    int n_blocks, team, plane_bytes, part_bytes;
    unsigned tries;                       // looks at values that are not there yet, before a wave gives up
    FastDiv by_team;
    const float *head;                    // as in dwpw_run.hip
    int head_Co, head_Cob;
    TeamBlock block[kDwpwChainMaxBlocks];
};

typedef const __attribute__((address_space(4))) TeamArgs *TeamKernArgs;
typedef __attribute__((address_space(1))) char *GlobalBytes;
typedef __attribute__((address_space(1))) unsigned long long *GlobalPairs;
typedef __attribute__((address_space(1))) unsigned *GlobalWords;

__device__ __forceinline__ unsigned long long team_load(GlobalBytes p)
{
    return __hip_atomic_load((GlobalPairs)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned team_word(float v)
{
    const unsigned u = __builtin_bit_cast(unsigned, v);
    return u == kNotYet ? 0x7fffffffu : u;              // that one NaN as another
}
__device__ __forceinline__ void team_store(GlobalBytes p, floatx4 v)
{
    const unsigned x = team_word(v.x), y = team_word(v.y), z = team_word(v.z), u = team_word(v.w);
    __hip_atomic_store((GlobalPairs)p, (unsigned long long)y << 32 | x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store((GlobalPairs)(p + 8), (unsigned long long)u << 32 | z, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned team_most(unsigned m, unsigned long long v)
{
    return max(max(m, (unsigned)v), (unsigned)(v >> 32));
}
__device__ __forceinline__ floatx4 team_relu(floatx4 v)
{
    v.x = v.x > 0.f ? v.x : 0.f; v.y = v.y > 0.f ? v.y : 0.f;
    v.z = v.z > 0.f ? v.z : 0.f; v.w = v.w > 0.f ? v.w : 0.f;
    return v;
}

// A wave's part of a pointwise layer: NI items, the J input blocks of pixel groups g0, g0 + kTeamWaves, ... Filters and values are all
// requested at once; the sums of a pixel group, in the order of dwpw_run, go to part[group][lane].
template <int NI>
__device__ __forceinline__ void team_reduce(const float *filt, GlobalBytes x, int HW, int p, int q, int lane, int J, int g0,
                                            floatx4 *part, TeamKernArgs ka, bool &lost)
{
    float a[NI][4];
    unsigned off[NI];
    {
        int ci = 0, g = g0;
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const float *f = filt + (size_t)ci * 256 + q * 64 + p;
#pragma unroll
            for (int r = 0; r < 4; ++r) a[n][r] = f[r * 16];
            off[n] = (unsigned)(ci * HW + min(g * 16 + p, HW - 1)) * 64 + q * 16;      // lanes past the image: its last pixel again
            if (++ci == J) { ci = 0; g += kTeamWaves; }
        }
    }
    unsigned long long v[NI][2];
    for (unsigned tries = 0;; ++tries) {
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            v[n][0] = team_load(x + off[n]);
            v[n][1] = team_load(x + off[n] + 8);
        }
        unsigned most = 0;                // kNotYet is the largest word (and a maximum of three is one instruction, without branches)
#pragma unroll
        for (int n = 0; n < NI; ++n) most = team_most(team_most(most, v[n][0]), v[n][1]);
        if (__ballot(most == kNotYet) == 0) break;
        if (tries >= ka->tries) { lost = true; break; }
    }
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    int g = g0, j = 0;
#pragma unroll
    for (int n = 0; n < NI; ++n) {
        const unsigned b[4] = {(unsigned)v[n][0], (unsigned)(v[n][0] >> 32), (unsigned)v[n][1], (unsigned)(v[n][1] >> 32)};
#pragma unroll
        for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[n][r], __builtin_bit_cast(float, b[r]), acc, 0, 0, 0);
        if (++j == J) {
            part[g * 64 + lane] = acc;
            acc = floatx4{0.f, 0.f, 0.f, 0.f};
            j = 0; g += kTeamWaves;
        }
    }
}

// The head, a channel block's part of it: the sum over the pixels by the weights, to the exchange area. Lane: a channel of one of four
// outputs, which go round the waves.
__device__ __forceinline__ void team_head_part(TeamKernArgs ka, const float *head, GlobalBytes x, const floatx4 *plane, int c, int w, int lane)
{
    const int last = ka->n_blocks - 1, C = ka->block[last].nCbo * 16, HW = ka->block[last].Ho * ka->block[last].Wo;
    const int Co = ka->head_Co, Cob = ka->head_Cob;
    const int ch = c * 16 + (lane & 15);
    const float *act = reinterpret_cast<const float *>(plane) + (lane & 15);
    float sum = 0.f;
    for (int m = 0; m < HW; ++m) sum += act[m * 16];
    for (int o = w * 4 + (lane >> 4); o < Co; o += kTeamWaves * 4) {
        const float v = fmaf(sum, head[((size_t)(o / Cob) * C + ch) * Cob + o % Cob], 0.f);
        __hip_atomic_store((GlobalWords)(x + (unsigned)(o * C + ch) * 4), team_word(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ... and the outputs, one after the other round the waves, a wave's all requested at once; lane: a channel of 64, summed as dwpw_run does.
__device__ __forceinline__ void team_head_sum(TeamKernArgs ka, float *out, int img, GlobalBytes x, int w, int lane, unsigned most, bool &lost)
{
    constexpr int U = kTeamHeadMost / kTeamWaves, K = kTeamMax / 4;
    const int last = ka->n_blocks - 1, C = ka->block[last].nCbo * 16, HW = ka->block[last].Ho * ka->block[last].Wo, Co = ka->head_Co;
    if (w >= Co) return;
    unsigned v[U][K];
    for (unsigned tries = 0;; ++tries) {
        unsigned most_word = 0;
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k)
                v[u][k] = __hip_atomic_load((GlobalWords)(x + (unsigned)(min(w + kTeamWaves * u, Co - 1) * C + min(k * 64 + lane, C - 1)) * 4),
                                            __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < K; ++k) most_word = max(most_word, v[u][k]);
        if (__ballot(most_word == kNotYet) == 0) break;
        if (tries >= most) { lost = true; break; }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int o = w + kTeamWaves * u;
        if (o >= Co) break;
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            float y = k * 64 + lane < C ? __builtin_bit_cast(float, v[u][k]) : 0.f;
#pragma unroll
            for (int d = 32; d > 0; d >>= 1) y += __shfl_xor(y, d, 64);
            sum += y;
        }
        if (lane == 0) out[(size_t)img * Co + o] = sum * (1.f / (float)HW);
    }
}

// A workgroup that has given up its team: the parts of all of the team one after the other, from the run's input on, and every output.
// Waits for nothing but its own stores. Not inlined, so that the kernel's registers are those of its usual way.
__device__ __attribute__((noinline)) void team_alone(TeamKernArgs ka, int img, floatx4 *lds)
{
    const int lane = threadIdx.x & 63, p = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n_blocks = ka->n_blocks;
    const float *head = ka->head;
    floatx4 *plane = lds + 4;
    GlobalBytes x = (GlobalBytes)(ka->exchange + (size_t)img * ka->exchange_bytes);       // what the pointwise layer reads
    for (int b = 0; b <= n_blocks; ++b) {
        // block b's input, a channel block at a time: to plane, then what the block's depthwise layer makes of it
        const int last = max(b - 1, 0), J = ka->block[last].nCbi;
        const int HW = ka->block[last].Ho * ka->block[last].Wo;
        GlobalBytes behind = x + (b ? (unsigned)(J * HW) * 64 : 0u);
        const int n_c = b ? ka->block[last].nCbo : J;
        for (int c = 0; c < n_c; ++c) {
            __syncthreads();                                    // plane has been read
            if (b == 0) {
                const int quads = ka->block[0].Hi * ka->block[0].Wi * 4;
                const floatx4 *src = reinterpret_cast<const floatx4 *>(ka->in) + ((size_t)img * n_c + c) * quads;
                for (int k = threadIdx.x; k < quads; k += kTeamThreads) plane[k] = src[k];
            }
            for (int g = w; b > 0 && g * 16 < HW; g += kTeamWaves) {
                const int m = g * 16 + p;
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                for (int ci = 0; ci < J; ++ci) {
                    const float *f = ka->block[last].pw + ((size_t)c * J + ci) * 256 + q * 64 + p;
                    const GlobalBytes from = x + ((unsigned)(ci * HW + min(m, HW - 1)) * 64 + q * 16);
                    unsigned long long u = 0, v = 0;
                    for (unsigned tries = 0; tries < kOwnTries; ++tries) {
                        u = team_load(from);
                        v = team_load(from + 8);
                        if (__ballot(team_most(team_most(0, u), v) == kNotYet) == 0) break;
                    }
                    const unsigned y[4] = {(unsigned)u, (unsigned)(u >> 32), (unsigned)v, (unsigned)(v >> 32)};
#pragma unroll
                    for (int r = 0; r < 4; ++r) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(f[r * 16], __builtin_bit_cast(float, y[r]), acc, 0, 0, 0);
                }
                if (ka->block[last].pw_relu) acc = team_relu(acc);
                if (m < HW) {
                    if (b == n_blocks && head == nullptr) reinterpret_cast<floatx4 *>(ka->out)[((size_t)img * n_c + c) * HW * 4 + m * 4 + q] = acc;
                    else plane[m * 4 + q] = acc;
                }
            }
            __syncthreads();
            if (b < n_blocks) {
                const floatx4 *taps = reinterpret_cast<const floatx4 *>(ka->block[b].dw + (size_t)c * 144) + q;
                const int Hi = ka->block[b].Hi, Wi = ka->block[b].Wi, Wo = ka->block[b].Wo, d_HW = ka->block[b].Ho * Wo;
                for (int m = w * 16 + p; m < d_HW; m += kTeamWaves * 16) {
                    const int oy = m / Wo, ox = m - oy * Wo;
                    const int iy0 = oy * ka->block[b].stride - ka->block[b].pt, ix0 = ox * ka->block[b].stride - ka->block[b].pl;
                    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
                    for (int k = 0; k < 9; ++k) {               // (taps outside the image multiply zeros, as in the kernel)
                        const int iy = iy0 + k / 3, ix = ix0 + k % 3;
                        const bool on = (unsigned)iy < (unsigned)Hi && (unsigned)ix < (unsigned)Wi;
                        const floatx4 v = plane[(on ? iy * Wi + ix : -1) * 4 + q], u = taps[k * 4];
                        acc.x = fmaf(v.x, u.x, acc.x); acc.y = fmaf(v.y, u.y, acc.y);
                        acc.z = fmaf(v.z, u.z, acc.z); acc.w = fmaf(v.w, u.w, acc.w);
                    }
                    if (ka->block[b].dw_relu) acc = team_relu(acc);
                    team_store(behind + (unsigned)(c * d_HW + m) * 64 + q * 16, acc);
                }
            } else if (head != nullptr) {
                team_head_part(ka, head, behind, plane, c, w, lane);
            }
        }
        x = behind;
    }
    bool lost = false;
    if (head != nullptr) team_head_sum(ka, ka->out, img, x, w, lane, kOwnTries, lost);
}

__global__ void __launch_bounds__(kTeamThreads) dwpw_team(TeamArgs args)
{
    (void)args;
    const TeamKernArgs ka = (TeamKernArgs)__builtin_amdgcn_kernarg_segment_ptr();
    const int n_blocks = ka->n_blocks, team = ka->team;
    const FastDiv by_team = {ka->by_team.magic, ka->by_team.shift, ka->by_team.d};
    const int img = by_team.div((int)blockIdx.x), t = (int)blockIdx.x - img * team;
    const int lane = threadIdx.x & 63, p = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const float *in = ka->in, *head = ka->head;
    float *out = ka->out;
    GlobalBytes x = (GlobalBytes)(ka->exchange + (size_t)img * ka->exchange_bytes);

    // LDS: [a pixel of zeros][this workgroup's channel block of the present tensor: pixel, quad][sums of the next, two sets in turn]
    extern __shared__ floatx4 lds[];
    __shared__ int gave_up[2];            // with the sets of sums, in turn: a wave ahead of the others, past at most one barrier, sets the other
    floatx4 *plane = lds + 4;
    const int part_set = ka->part_bytes >> 4;
    floatx4 *const part0 = plane + (ka->plane_bytes >> 4);
    floatx4 *part = part0;
    bool lost = false;

    // What this workgroup's next depthwise layer needs and what does not depend on results: the taps, the window's entries in
    // plane for the wave's first pixel group (those outside the image are the zeros) and the layer's numbers. It is got ready
    // while the wave would be waiting for the block before.
    floatx4 wt[9];
    int at[9];
    int d_ng, d_HW, d_relu, d_Hi, d_Wi, d_Wo, d_stride, d_pt, d_pl;
    FastDiv d_by_Wo;
    auto window = [&](int g) __attribute__((always_inline)) {
        const int m = min(g * 16 + p, d_HW - 1);
        const int oy = d_by_Wo.div(m), ox = m - oy * d_Wo;
        const int iy0 = oy * d_stride - d_pt, ix0 = ox * d_stride - d_pl;
#pragma unroll
        for (int k = 0; k < 9; ++k) {
            const int iy = iy0 + k / 3, ix = ix0 + k % 3;
            const bool on = (unsigned)iy < (unsigned)d_Hi && (unsigned)ix < (unsigned)d_Wi;
            at[k] = (on ? iy * d_Wi + ix : -1) * 4 + q;
        }
    };
    auto get_ready = [&](int b) __attribute__((always_inline)) {
        const floatx4 *taps = reinterpret_cast<const floatx4 *>(ka->block[b].dw + (size_t)t * 144) + q;
#pragma unroll
        for (int k = 0; k < 9; ++k) wt[k] = taps[k * 4];
        d_Hi = ka->block[b].Hi; d_Wi = ka->block[b].Wi; d_Wo = ka->block[b].Wo;
        d_stride = ka->block[b].stride; d_pt = ka->block[b].pt; d_pl = ka->block[b].pl;
        d_relu = ka->block[b].dw_relu;
        d_HW = ka->block[b].Ho * d_Wo;
        d_ng = (d_HW + 15) >> 4;
        d_by_Wo.magic = ka->block[b].by_Wo.magic; d_by_Wo.shift = ka->block[b].by_Wo.shift; d_by_Wo.d = ka->block[b].by_Wo.d;
        window(w);
    };
    if (threadIdx.x < 2) gave_up[threadIdx.x] = 0;
    if (threadIdx.x < 4) lds[threadIdx.x] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (t < ka->block[0].nCbi) {
        const int quads = ka->block[0].Hi * ka->block[0].Wi * 4;
        const floatx4 *src = reinterpret_cast<const floatx4 *>(in) + ((size_t)img * ka->block[0].nCbi + t) * quads;
        for (int k = threadIdx.x; k < quads; k += kTeamThreads) plane[k] = src[k];
        get_ready(0);
    }
    __syncthreads();

    for (int b = 0; b < n_blocks; ++b) {
        const int nCbi = ka->block[b].nCbi, nCbo = ka->block[b].nCbo;
        const int HW = ka->block[b].Ho * ka->block[b].Wo;
        const int ng = (HW + 15) >> 4;

        // ---------------- depthwise: plane -> exchange area, pixel groups round the waves
        if (t < nCbi) {
            for (int g = w; g < d_ng; g += kTeamWaves) {
                if (g != w) window(g);
                floatx4 v[9];
#pragma unroll
                for (int k = 0; k < 9; ++k) v[k] = plane[at[k]];
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int k = 0; k < 9; ++k) {
                    acc.x = fmaf(v[k].x, wt[k].x, acc.x); acc.y = fmaf(v[k].y, wt[k].y, acc.y);
                    acc.z = fmaf(v[k].z, wt[k].z, acc.z); acc.w = fmaf(v[k].w, wt[k].w, acc.w);
                }
                if (d_relu) acc = team_relu(acc);
                const int m = g * 16 + p;
                if (m < d_HW) team_store(x + (unsigned)(t * d_HW + m) * 64 + q * 16, acc);
            }
        }
        if (b + 1 < n_blocks && t < nCbo) get_ready(b + 1);

        // ---------------- pointwise: exchange area -> partial sums -> plane
        if (t < nCbo) {
            const int items = w < ng ? nCbi * ((ng - w + kTeamWaves - 1) / kTeamWaves) : 0;
            const float *filt = ka->block[b].pw + (size_t)t * nCbi * 256;
            switch (items) {
#define SMALL_TEAM_CASE(NI_) case NI_: team_reduce<NI_>(filt, x, HW, p, q, lane, nCbi, w, part, ka, lost); break;
                SMALL_TEAM_CASE(1) SMALL_TEAM_CASE(2) SMALL_TEAM_CASE(3) SMALL_TEAM_CASE(4) SMALL_TEAM_CASE(5) SMALL_TEAM_CASE(6)
                SMALL_TEAM_CASE(7) SMALL_TEAM_CASE(8) SMALL_TEAM_CASE(9) SMALL_TEAM_CASE(10) SMALL_TEAM_CASE(11) SMALL_TEAM_CASE(12)
                SMALL_TEAM_CASE(13) SMALL_TEAM_CASE(14) SMALL_TEAM_CASE(15) SMALL_TEAM_CASE(16)
#undef SMALL_TEAM_CASE
                default: break;
            }
            int *const flag = gave_up + (part != part0);
            if (lost && lane == 0) *flag = 1;
            __syncthreads();                            // plane has been read
            lost = __builtin_amdgcn_readfirstlane(*flag) != 0;
            if (lost) break;
            const int pw_relu = ka->block[b].pw_relu;
            const bool to_memory = b + 1 == n_blocks && head == nullptr;
            for (int g = w; g < ng; g += kTeamWaves) {
                floatx4 v = part[g * 64 + lane];
                if (pw_relu) v = team_relu(v);
                const int m = g * 16 + p;
                if (m < HW) {
                    if (to_memory) reinterpret_cast<floatx4 *>(out)[((size_t)img * nCbo + t) * HW * 4 + m * 4 + q] = v;
                    else plane[m * 4 + q] = v;
                }
            }
            // One pixel group, here and in the next block: wave 0 wrote plane and alone reads it. The other set of sums is next, so
            // a wave that runs ahead, past at most one more barrier, writes nothing that is still read.
            if (ng > 1 || (b + 1 < n_blocks && d_ng > 1)) __syncthreads();
            else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
            part = part == part0 ? part0 + part_set : part0;
        }
        x += (unsigned)(nCbi * HW) * 64;
    }

    // ---------------- the network's head: mean over the pixels, fully connected layer; every workgroup its channels' part
    if (head != nullptr && !lost) {
        const int last = n_blocks - 1;
        if (t < ka->block[last].nCbo) {
            __syncthreads();                            // (a single pixel group's plane is wave 0's)
            team_head_part(ka, head, x, plane, t, w, lane);
        }
        if (t == 0) {
            team_head_sum(ka, out, img, x, w, lane, ka->tries, lost);
            int *const flag = gave_up + (part != part0);
            if (lost && lane == 0) *flag = 1;
            __syncthreads();
            lost = __builtin_amdgcn_readfirstlane(*flag) != 0;
        }
    }
    if (lost) team_alone(ka, img, lds);
}

__global__ void __launch_bounds__(kTeamThreads) team_clear(uint4 *p, unsigned n)
{
    const unsigned i = blockIdx.x * kTeamThreads + threadIdx.x;
    if (i < n) p[i] = uint4{kNotYet, kNotYet, kNotYet, kNotYet};
}

int team_size(const DwpwRunBlock *b, int n)
{
    int most = b[0].Cin;
    for (int i = 0; i < n; ++i) most = std::max(most, b[i].Cout);
    return most / 16;
}
int team_groups(const DwpwRunBlock &b) { return (b.Ho * b.Wo + 15) / 16; }
size_t team_exchange_bytes(const DwpwRunBlock *b, int n, int head_Co)
{
    size_t words = (size_t)b[n - 1].Cout * head_Co;
    for (int i = 0; i < n; ++i) words += (size_t)b[i].Cin * b[i].Ho * b[i].Wo;
    return words * 4;
}
void team_lds(const DwpwRunBlock *b, int n, int &plane, int &part)
{
    plane = b[0].Hi * b[0].Wi * 64;
    part = 0;
    for (int i = 0; i < n; ++i) {
        plane = std::max(plane, b[i].Ho * b[i].Wo * 64);
        part = std::max(part, team_groups(b[i]) << 10);
    }
}

}  // namespace

// A workgroup of a team waits for the others, and where they find no place on the chip beside it, it has waited in vain. A compute unit
// holds two (registers); kernels that wait for nobody make room in the end; and with an eighth of the compute units' number per
// launch, 16 launches that wait fit together, four times the hardware queues that a process has unless told otherwise. A stream may
// be confined to some of the compute units: those count. Within that a team is faster however short the run: 200 random ones of 2 to
// 12 blocks, 2 to 16 workgroups an image, 1 to 16 images, with and without a head, take 0.43 to 0.97 of dwpw_run's time (2 blocks, 64
// channels, 32 pixels 7.4 / 7.2 us; 12 blocks, 160 channels, 49 pixels, 3 images 76 / 36).
size_t dwpw_team_exchange(const DwpwRunBlock *blocks, int n_blocks, int N, int head_Co, hipStream_t s)
{
    const int T = team_size(blocks, n_blocks);
    if (T > kTeamMax || T < 2 || head_Co > kTeamHeadMost || 8L * N * T > device_cus()) return 0;
    uint32_t mask[32] = {};
    if (hipExtStreamGetCUMask(s, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    int cus = 0;
    for (uint32_t m : mask) cus += __builtin_popcount(m);
    if (8L * N * T > cus) return 0;
    for (int i = 0; i < n_blocks; ++i) {
        if (blocks[i].Cin / 16 * ((team_groups(blocks[i]) + kTeamWaves - 1) / kTeamWaves) > kTeamItems) return 0;
    }
    int plane, part;
    team_lds(blocks, n_blocks, plane, part);
    if (plane + 2 * part > 52 * 1024) return 0;
    return (size_t)N * team_exchange_bytes(blocks, n_blocks, head_Co);
}

hipError_t launch_dwpw_team(const float *in, float *out, const DwpwRunBlock *blocks, int n_blocks, int N, const DwpwRunHead &head,
                            void *exchange, hipStream_t s, unsigned tries, int absent)
{
    TeamArgs a;
    a.tries = tries;
    a.in = in; a.out = out; a.exchange = (char *)exchange;
    a.head = head.filt; a.head_Co = head.Co; a.head_Cob = head.Cob;
    a.n_blocks = n_blocks;
    a.team = team_size(blocks, n_blocks);
    a.by_team = make_fastdiv(a.team);
    a.exchange_bytes = (unsigned)team_exchange_bytes(blocks, n_blocks, head.filt ? head.Co : 0);
    team_lds(blocks, n_blocks, a.plane_bytes, a.part_bytes);
    for (int i = 0; i < kDwpwChainMaxBlocks; ++i) {
        const DwpwRunBlock &b = blocks[i < n_blocks ? i : n_blocks - 1];
        TeamBlock &d = a.block[i];
        d.dw = b.dw; d.pw = b.pw; d.dw_relu = b.dw_relu; d.pw_relu = b.pw_relu;
        d.nCbi = b.Cin / 16; d.nCbo = b.Cout / 16;
        d.Hi = b.Hi; d.Wi = b.Wi; d.Ho = b.Ho; d.Wo = b.Wo; d.stride = b.stride; d.pt = b.pt; d.pl = b.pl;
        d.by_Wo = make_fastdiv(b.Wo);
    }
    const unsigned quads = (unsigned)((size_t)N * a.exchange_bytes / 16);
    hipLaunchKernelGGL(team_clear, dim3((quads + kTeamThreads - 1) / kTeamThreads), dim3(kTeamThreads), 0, s, (uint4 *)exchange, quads);
    hipLaunchKernelGGL(dwpw_team, dim3((unsigned)(N * a.team - absent)), dim3(kTeamThreads), 64 + (size_t)a.plane_bytes + 2 * (size_t)a.part_bytes, s, a);
    return hipGetLastError();
}

}  // namespace small
