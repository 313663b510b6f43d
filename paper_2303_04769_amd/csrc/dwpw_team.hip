// A run of depthwise-separable blocks (dwpw_run.hip says what that is) on one or a few images: a team of workgroups per
// image, one for each 16-channel block of the widest tensor.
//
// What bounds it: latency. One workgroup per image streams every filter of the run through one compute unit and does every
// stage there, some 4 us a block, while the rest of the chip idles. Here workgroup t owns channel block t: it computes the
// pointwise result of that block (its share of the filters is one sixteenth), then, as a depthwise layer maps channel
// blocks on their own, the next block's depthwise layer on it, and hands the result to the team. So a block costs one
// hand-over through memory, one reduction of at most 16 steps split over the workgroup's four waves, and one window pass.
// The eleven blocks and the head of the depthwise-separable CNN, one image: 50 -> 26.0 us and 2 for the launch in front, of which
// some 1.3 us a block are the way of a value to memory and back; the network's call 66.8 -> 42.2 (two images 65.3 -> 40.9 without
// the packing of its input). All of a team on one of the chip's eight dies gains nothing (30.1 against 28.9 us at the time), nor
// does waiting before the first look (0.07 to 2.9 us slower): values are looked at past the dies' caches either way. What a wave
// needs for its next stage besides results -- taps, window entries, the layer's numbers -- it gets ready while it would be
// waiting (28.9 -> 26.0 us).
//
// The hand-over has no flags and no barrier: a word of the exchange area is "not there yet" while it holds kNotYet, a NaN
// with all bits set, which no result is stored as, and the launch in front fills the area with it. A consumer reads the
// values it needs, each in agent scope (which goes past the L2s, of which the chip has eight), until none is kNotYet; a
// value that is there is final. Nothing else is communicated, so nothing has to be ordered.
//
// Every wait ends: a workgroup needs only results of its own team, and the launch is small enough for all teams to be on
// the chip together (dwpw_team_eligible). Should they not get there all the same, a wave gives up after some seconds, hands
// nothing on, and the outputs of that image are NaN.
#include "small_internal.h"

#include <algorithm>

namespace small {
namespace {

constexpr int kTeamWaves = 4;
constexpr int kTeamThreads = kTeamWaves * 64;
constexpr int kTeamMax = 16;              // workgroups of a team = channel blocks of the widest tensor
constexpr int kTeamItems = 8;             // (input block, pixel group) pairs that a wave has in registers
constexpr unsigned kNotYet = ~0u;
constexpr unsigned kMaxTries = 1u << 21;  // a try takes at least a round trip to memory, some 0.6 us

struct TeamBlock {
    const float *dw, *pw;
    int dw_relu, pw_relu;
    int nCbi, nCbo;
    int Hi, Wi, Ho, Wo, stride, pt, pl;
    int log_kw;                           // the pointwise reduction is split over 1 << log_kw waves, the pixel groups over the rest
    FastDiv by_Wo;
};

struct TeamArgs {
    const float *in;
    float *out;
    char *exchange;
    unsigned exchange_bytes;              // per image
    int n_blocks, team, plane_bytes, part_bytes;
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
__device__ __forceinline__ bool team_there(unsigned long long v)
{
    return (unsigned)v != kNotYet && (unsigned)(v >> 32) != kNotYet;
}
__device__ __forceinline__ floatx4 team_relu(floatx4 v)
{
    v.x = v.x > 0.f ? v.x : 0.f; v.y = v.y > 0.f ? v.y : 0.f;
    v.z = v.z > 0.f ? v.z : 0.f; v.w = v.w > 0.f ? v.w : 0.f;
    return v;
}

// A wave's part of the pointwise reduction: NI items, input blocks k0, k0 + kw, ... (J of them) of pixel groups g0, g0 + gw, ...
// Filters and values are all requested at once; the sums of a pixel group go to part[group][lane].
template <int NI>
__device__ __forceinline__ void team_reduce(const float *filt, GlobalBytes x, int HW, int p, int q, int lane, int k0, int kw, int J,
                                            int g0, int gw, floatx4 *part, bool &lost)
{
    float a[NI][4];
    unsigned off[NI];
    {
        int ci = k0, g = g0, j = 0;
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            const float *f = filt + (size_t)ci * 256 + q * 64 + p;
#pragma unroll
            for (int r = 0; r < 4; ++r) a[n][r] = f[r * 16];
            off[n] = (unsigned)(ci * HW + min(g * 16 + p, HW - 1)) * 64 + q * 16;      // lanes past the image: its last pixel again
            ci += kw;
            if (++j == J) { j = 0; ci = k0; g += gw; }
        }
    }
    unsigned long long v[NI][2];
    for (unsigned tries = 0;; ++tries) {
#pragma unroll
        for (int n = 0; n < NI; ++n) {
            v[n][0] = team_load(x + off[n]);
            v[n][1] = team_load(x + off[n] + 8);
        }
        bool there = true;
#pragma unroll
        for (int n = 0; n < NI; ++n) there = there && team_there(v[n][0]) && team_there(v[n][1]);
        if (__ballot(!there) == 0) break;
        if (lost || tries >= kMaxTries) { lost = true; break; }
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
            j = 0; g += gw;
        }
    }
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

    // LDS: [a pixel of zeros][this workgroup's channel block of the present tensor: pixel, quad][partial sums, two sets in turn]
    extern __shared__ floatx4 lds[];
    __shared__ int gave_up;
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
    if (threadIdx.x == 0) gave_up = 0;
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
        if (t < nCbi && !lost) {
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
            const int log_kw = ka->block[b].log_kw, kw = 1 << log_kw, gw = kTeamWaves >> log_kw;
            const int k0 = w & (kw - 1), g0 = w >> log_kw;
            const int J = (nCbi - k0 + kw - 1) >> log_kw;
            const int items = g0 < ng ? J * ((ng - g0 + gw - 1) >> (2 - log_kw)) : 0;
            const float *filt = ka->block[b].pw + (size_t)t * nCbi * 256;
            floatx4 *mine = part + k0 * ng * 64;
            switch (items) {
                case 1: team_reduce<1>(filt, x, HW, p, q, lane, k0, kw, J, g0, gw, mine, lost); break;
                case 2: team_reduce<2>(filt, x, HW, p, q, lane, k0, kw, J, g0, gw, mine, lost); break;
                case 3: team_reduce<3>(filt, x, HW, p, q, lane, k0, kw, J, g0, gw, mine, lost); break;
                case 4: team_reduce<4>(filt, x, HW, p, q, lane, k0, kw, J, g0, gw, mine, lost); break;
                case 5: team_reduce<5>(filt, x, HW, p, q, lane, k0, kw, J, g0, gw, mine, lost); break;
                case 6: team_reduce<6>(filt, x, HW, p, q, lane, k0, kw, J, g0, gw, mine, lost); break;
                case 7: team_reduce<7>(filt, x, HW, p, q, lane, k0, kw, J, g0, gw, mine, lost); break;
                case 8: team_reduce<8>(filt, x, HW, p, q, lane, k0, kw, J, g0, gw, mine, lost); break;
                default: break;
            }
            if (lost && lane == 0) gave_up = 1;
            __syncthreads();                            // the partial sums are complete, and plane has been read
            lost = __builtin_amdgcn_readfirstlane(gave_up) != 0;
            const int pw_relu = ka->block[b].pw_relu;
            const bool to_memory = b + 1 == n_blocks && head == nullptr;
            for (int g = w; g < ng; g += kTeamWaves) {
                floatx4 v = part[g * 64 + lane];
                for (int k = 1; k < kw; ++k) v += part[(k * ng + g) * 64 + lane];
                if (pw_relu) v = team_relu(v);
                const int m = g * 16 + p;
                if (m < HW) {
                    if (to_memory) {
                        const float nan = __builtin_nanf("");
                        reinterpret_cast<floatx4 *>(out)[((size_t)img * nCbo + t) * HW * 4 + m * 4 + q] = lost ? floatx4{nan, nan, nan, nan} : v;
                    } else {
                        plane[m * 4 + q] = v;
                    }
                }
            }
            // One pixel group, here and in the next block: wave 0 wrote plane and alone reads it. The other set of partial sums is
            // next, so a wave that runs ahead, past at most one more barrier, writes nothing that is still read.
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
    if (head != nullptr && w == 0) {
        const int nCb = ka->block[n_blocks - 1].nCbo, C = nCb * 16;
        const int HW = ka->block[n_blocks - 1].Ho * ka->block[n_blocks - 1].Wo;
        const int Co = ka->head_Co, Cob = ka->head_Cob;
        if (t < nCb && !lost) {
            const float *act = reinterpret_cast<const float *>(plane);
            float sum = 0.f;
            for (int m = q; m < HW; m += 4) sum += act[m * 16 + p];
            sum += __shfl_xor(sum, 16, 64);
            sum += __shfl_xor(sum, 32, 64);             // lane: channel p
            float mine = 0.f;
#pragma unroll
            for (int o = 0; o < 16; ++o) {
                if (o < Co) {
                    float v = sum * head[((size_t)(o / Cob) * C + t * 16 + p) * Cob + o % Cob];
#pragma unroll
                    for (int d = 8; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
                    mine = lane == o ? v : mine;
                }
            }
            if (lane < Co)
                __hip_atomic_store((GlobalWords)(x + (unsigned)(t * 16 + lane) * 4), team_word(mine), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (t == 0) {
            const int o = min(p, Co - 1);
            unsigned v[4];
            for (unsigned tries = 0;; ++tries) {
                bool there = true;
#pragma unroll
                for (int k = 0; k < 4; ++k)             // lane: output p, channel blocks q, q + 4, ...
                    v[k] = __hip_atomic_load((GlobalWords)(x + (unsigned)(min(q + 4 * k, nCb - 1) * 16 + o) * 4), __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int k = 0; k < 4; ++k) there = there && v[k] != kNotYet;
                if (__ballot(!there) == 0) break;
                if (lost || tries >= kMaxTries) { lost = true; break; }
            }
            float sum = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) sum += q + 4 * k < nCb ? __builtin_bit_cast(float, v[k]) : 0.f;
            sum += __shfl_xor(sum, 16, 64);
            sum += __shfl_xor(sum, 32, 64);
            if (lane < Co) out[(size_t)img * Co + lane] = lost ? __builtin_nanf("") : sum * (1.f / (float)HW);
        }
    }
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
int team_log_kw(int nCbi) { return nCbi >= 4 ? 2 : (nCbi >= 2 ? 1 : 0); }
int team_groups(const DwpwRunBlock &b) { return (b.Ho * b.Wo + 15) / 16; }
size_t team_exchange_bytes(const DwpwRunBlock *b, int n, bool head)
{
    size_t words = head ? (size_t)kTeamMax * 16 : 0;
    for (int i = 0; i < n; ++i) words += (size_t)b[i].Cin * b[i].Ho * b[i].Wo;
    return words * 4;
}
void team_lds(const DwpwRunBlock *b, int n, int &plane, int &part)
{
    plane = b[0].Hi * b[0].Wi * 64;
    part = 0;
    for (int i = 0; i < n; ++i) {
        plane = std::max(plane, b[i].Ho * b[i].Wo * 64);
        part = std::max(part, team_groups(b[i]) << (10 + team_log_kw(b[i].Cin / 16)));
    }
}

}  // namespace

// A workgroup of a team waits for the others, so all of them have to find a place on the chip whatever else runs there. A compute
// unit holds three (registers, LDS); kernels that wait for nobody make room in the end; and with an eighth of the compute units'
// number per launch, 24 launches that wait, more than the hardware runs queues at a time, fit together. A stream may be confined
// to some of the compute units: those count.
size_t dwpw_team_exchange(const DwpwRunBlock *blocks, int n_blocks, int N, bool head, hipStream_t s)
{
    const int T = team_size(blocks, n_blocks);
    if (T > kTeamMax || T < 2 || 8L * N * T > device_cus()) return 0;
    uint32_t mask[32] = {};
    if (hipExtStreamGetCUMask(s, 32, mask) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    int cus = 0;
    for (uint32_t m : mask) cus += __builtin_popcount(m);
    if (8L * N * T > cus) return 0;
    for (int i = 0; i < n_blocks; ++i) {
        const int nCbi = blocks[i].Cin / 16, log_kw = team_log_kw(nCbi), gw = kTeamWaves >> log_kw;
        const int J = (nCbi + (1 << log_kw) - 1) >> log_kw;
        if (J * ((team_groups(blocks[i]) + gw - 1) / gw) > kTeamItems) return 0;
    }
    int plane, part;
    team_lds(blocks, n_blocks, plane, part);
    if (plane + 2 * part > 52 * 1024) return 0;
    return (size_t)N * team_exchange_bytes(blocks, n_blocks, head);
}

hipError_t launch_dwpw_team(const float *in, float *out, const DwpwRunBlock *blocks, int n_blocks, int N, const DwpwRunHead &head,
                            void *exchange, hipStream_t s)
{
    TeamArgs a;
    a.in = in; a.out = out; a.exchange = (char *)exchange;
    a.head = head.filt; a.head_Co = head.Co; a.head_Cob = head.Cob;
    a.n_blocks = n_blocks;
    a.team = team_size(blocks, n_blocks);
    a.by_team = make_fastdiv(a.team);
    a.exchange_bytes = (unsigned)team_exchange_bytes(blocks, n_blocks, head.filt != nullptr);
    team_lds(blocks, n_blocks, a.plane_bytes, a.part_bytes);
    for (int i = 0; i < kDwpwChainMaxBlocks; ++i) {
        const DwpwRunBlock &b = blocks[i < n_blocks ? i : n_blocks - 1];
        TeamBlock &d = a.block[i];
        d.dw = b.dw; d.pw = b.pw; d.dw_relu = b.dw_relu; d.pw_relu = b.pw_relu;
        d.nCbi = b.Cin / 16; d.nCbo = b.Cout / 16;
        d.Hi = b.Hi; d.Wi = b.Wi; d.Ho = b.Ho; d.Wo = b.Wo; d.stride = b.stride; d.pt = b.pt; d.pl = b.pl;
        d.log_kw = team_log_kw(d.nCbi);
        d.by_Wo = make_fastdiv(b.Wo);
    }
    const unsigned quads = (unsigned)((size_t)N * a.exchange_bytes / 16);
    hipLaunchKernelGGL(team_clear, dim3((quads + kTeamThreads - 1) / kTeamThreads), dim3(kTeamThreads), 0, s, (uint4 *)exchange, quads);
    hipLaunchKernelGGL(dwpw_team, dim3((unsigned)(N * a.team)), dim3(kTeamThreads), 64 + (size_t)a.plane_bytes + 2 * (size_t)a.part_bytes, s, a);
    return hipGetLastError();
}

}  // namespace small
