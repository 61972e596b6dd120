// The linear branch's state and gate for short sequences, as device code for a launch of their own and for workgroups that ride in the
// large-tile attention kernel's launch.
//
// A call of a few thousand tokens is a chain of launches that are a few memory latencies each, and most of the chip has nothing to do in any of
// them.  The attention needs state and gate in its epilogues only, so its launch begins with workgroups that compute those while the others
// multiply.  A head has a word in the workspace in which riders count themselves when their results are there, and tiles when they have no
// more use for it.  A tile waits for the word for a bounded time, and then computes the head's state and its sample's gate itself (the same
// bits, to the same place): no workgroup depends on another one being run.
//
// Nothing has to be set in the workspace.  A word counts if it carries the call's tag; whoever finds another one puts the tag there, and
// whoever completes the count sets the word to 0, which is no call's tag, so a captured call, which keeps its tag, finds it unused on
// every replay.  Workgroups run on XCDs whose L2 caches do not see each other: what passes between them is written and read with
// device-scope accesses, which go past those caches, and stores are acknowledged before a workgroup counts itself in.
#pragma once
#include "salad_internal.h"

namespace salad {

// a head's word: riders that are done, tiles that are done with it (two units each), tag
constexpr uint64_t RIDE_TILE = 1ull << 10, RIDE_COUNT = (1ull << RIDE_COUNT_BITS) - 1;

__device__ inline uint64_t ride_load(const uint64_t *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void ride_store(uint64_t *p, uint64_t v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline float ride_loadf(const float *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void ride_storef(float *p, float v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// The arguments of the ride are read from the kernel's own (its first parameter) where they are used: held in scalar registers from the
// start on, they make those of the attention's loop spill.
typedef const __attribute__((address_space(4))) AttnArgs &CallRef;
__device__ inline CallRef call_args()
{
    uint64_t p = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return *(const __attribute__((address_space(4))) AttnArgs *)p;
}

// adds inc to a word of this tag; its value then
__device__ inline uint64_t ride_settle(uint64_t *w, uint64_t tag, uint64_t inc, uint64_t now)      // now: what an addition of inc has left
{
    while ((now & ~RIDE_COUNT) != tag) {
        if (__hip_atomic_compare_exchange_strong(w, &now, tag + inc, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) now = tag + inc;
        else if ((now & ~RIDE_COUNT) == tag) now = __hip_atomic_fetch_add(w, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + inc;
    }
    return now;
}

// every thread's stores are acknowledged, and every thread is here
__device__ inline void ride_published()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt 0
    __syncthreads();
}

__device__ inline uint32_t ride_relu(uint32_t x)          // of two bf16 values: a negative one is a negative integer
{
    typedef short s16x2 __attribute__((ext_vector_type(2)));
    s16x2 v = __builtin_bit_cast(s16x2, x), z = {0, 0};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(v, z));
}

template <int CTRL> __device__ inline float ride_add_dpp(float x)
{
    return x + __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(x), CTRL, 0xf, 0xf, false));
}
// sum over the wave in every lane, in the order of shuffles by 32, 16, 8, 4, 2, 1
__device__ inline float ride_wave_sum(float x)
{
    auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    x = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    x = ride_add_dpp<0x128>(x);      // row_ror 8, 4, 2, 1: the values repeat after 16, 8, 4, 2 lanes by then
    x = ride_add_dpp<0x124>(x);
    x = ride_add_dpp<0x122>(x);
    return ride_add_dpp<0x121>(x);
}

// Sums v0 .. v1 - 1 of a sample, v = part * 4 + wave of gate_part with the same bits: of the sigmoids of tokens v tok + t + i stride, t < tok, in
// ascending order.  A wave takes four tokens of one of its sums at a time, a chunk of 512 channels of each in turn, with the weights in LDS
// and three such steps of loads ahead.  (With a token and a chunk at a time the dot product's chain and the scalar code between are 700
// cycles for 1 KB.)
template <int NT>
__device__ inline __attribute__((always_inline)) void ride_gate(const void *x_t, const float *w_gate, float bias, int N, int D, int tok, int nparts,
                                                                float *sums, int b, int v0, int v1, unsigned char *smem)
{
    constexpr int NW = NT / 64, AHEAD = 4;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nch = (D + 511) >> 9;
    float4 *wlo = reinterpret_cast<float4 *>(smem), *whi = wlo + nch * 64;
    for (int i = tid; i < nch * 64; i += NT) {
        const float *w = w_gate + min(i * 8, D - 8);          // a caller's pointer, aligned to 4 bytes
        const bool in = i * 8 < D;
        wlo[i] = in ? make_float4(w[0], w[1], w[2], w[3]) : make_float4(0.f, 0.f, 0.f, 0.f);
        whi[i] = in ? make_float4(w[4], w[5], w[6], w[7]) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    const int nv = nparts * 4, stride = nv * tok, quad = 4 / tok * stride;
    const bool ragged = (D & 511) != 0;
    int dk[4];                            // a step's four tokens, from its first on
#pragma unroll
    for (int k = 0; k < 4; ++k) dk[k] = (k & (tok - 1)) + k / tok * stride;
    const char *xb = reinterpret_cast<const char *>(x_t) + (size_t)b * N * D * 2;
    sums += (size_t)b * nv;
    for (int v = v0 + tid; v < v1; v += NT)
        if (v * tok >= N) ride_storef(sums + v, 0.f);
    struct At { int v, n, c; };           // sum, first token, chunk
    auto next = [&](At &x) __attribute__((always_inline)) {
        if (++x.c == nch) {
            x.c = 0;
            x.n += quad;
            if (x.n >= N) { x.v += NW; x.n = x.v * tok; }
        }
    };
    auto live = [&](const At &x) __attribute__((always_inline)) { return x.v < v1 && x.n < N; };
    At ld{v0 + wave, (v0 + wave) * tok, 0}, at = ld;
    uint4 buf[AHEAD][4];
    auto load = [&](uint4 (&x)[4]) __attribute__((always_inline)) {          // past the end: rows of the sample that nobody uses
        const unsigned off = (unsigned)min(ld.c * 64 + lane, (D >> 3) - 1) * 16u;
#pragma unroll
        for (int k = 0; k < 4; ++k)
            x[k] = *reinterpret_cast<const uint4 *>(xb + (size_t)min(ld.n + dk[k], N - 1) * D * 2 + off);
        if (live(ld)) next(ld);
    };
    if (live(at)) {
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) load(buf[i]);
        float dot[4] = {}, acc = 0.f;
        bool more = true;
        while (more) {
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) {
                if (more) {
                    const int ci = at.c * 64 + lane;
                    const float4 wa = wlo[ci], wb = whi[ci];
                    const float w[8] = {wa.x, wa.y, wa.z, wa.w, wb.x, wb.y, wb.z, wb.w};
                    const bool end = at.c == nch - 1;
                    if (end && ragged && ci * 8 >= D)
#pragma unroll
                        for (int k = 0; k < 4; ++k) buf[i][k] = make_uint4(0, 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            const uint32_t x = j == 0 ? buf[i][k].x : j == 1 ? buf[i][k].y : j == 2 ? buf[i][k].z : buf[i][k].w;
                            dot[k] = fmaf(__uint_as_float(x << 16), w[2 * j], dot[k]);
                            dot[k] = fmaf(__uint_as_float(x & 0xffff0000u), w[2 * j + 1], dot[k]);
                        }
                    if (end) {
                        float sg[4];
#pragma unroll
                        for (int k = 0; k < 4; ++k) sg[k] = 1.f / (1.f + __expf(-(ride_wave_sum(dot[k]) + bias)));
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            if (at.n + dk[k] < N) acc += sg[k];
                            dot[k] = 0.f;
                        }
                        if (at.n + quad >= N) {
                            if (lane == 0) ride_storef(sums + at.v, acc);
                            acc = 0.f;
                        }
                    }
                    next(at);
                    more = live(at);
                }
                load(buf[i]);
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Short sequences: the state in one launch, without partial states.  A workgroup owns a slice of a head's Hs, 32 rows by 64 columns,
// over all tokens, and its 8 waves take turns at groups of 16 tokens.  16 rows of 32 channels are one load of a wave (1 KB straight into
// LDS), so a wave has a ring of its own, waits for its own loads only and meets the others once, at the end, where the 8 accumulators are
// added in wave order.  Operands come out of LDS transposed (ds_read_b64_tr_b16): the contraction is over tokens, the rows of the
// stored tensors.  Bound by what a compute unit reads, about 30 GB/s whatever is in flight: 192 bytes a token.  Slices of 32 x 32 are twice as
// many workgroups for two thirds of the bytes: 12 heads, N = 1950 28.8 us a call in place of 24.8, 8 heads, N = 5000 37.1 and 26.2, 2 heads the same.
// ------------------------------------------------------------------------------------------------
constexpr int DIRECT_WAVES = 8;
constexpr int SLICE_COLS = 2;             // times 32 columns of a slice
constexpr int slices_per_head(int d) { return d / 32 * (d / 32 / SLICE_COLS); }
constexpr int direct_lds(int d) { return 9 * 64 * d * 2; }           // what the attention kernel has for its tiles
// loads of a wave for 16 tokens, and how many groups of them it keeps in LDS
constexpr int direct_loads(bool rope) { return 1 + SLICE_COLS + (rope ? 1 : 0); }
constexpr int direct_depth(int d, bool rope) { return direct_lds(d) / 1024 / DIRECT_WAVES / direct_loads(rope); }

// Workgroup i of BH heads' slices: those of a head, which read the same rows, on one XCD (workgroups go to the 8 XCDs in turn)
__device__ inline int slice_head(int BH, int slices, int i)
{
    const int whole = BH / 8 * 8, j = i / (8 * slices);
    return j * 8 < whole ? j * 8 + (i & 7) : whole + (i - whole * slices) / slices;
}
__device__ inline int slice_of(int BH, int slices, int i)
{
    const int whole = BH / 8 * 8, j = i / (8 * slices);
    return j * 8 < whole ? (i - j * (8 * slices)) >> 3 : (i - whole * slices) % slices;
}

template <int D, bool ROPE>
__device__ inline __attribute__((always_inline)) void state_slice(const u16 *__restrict__ k, const u16 *__restrict__ v, int N, const uint32_t *__restrict__ rope_tab,
                                                                  u16 *__restrict__ hfrag, float *__restrict__ Z, int bh, int slice,
                                                                  unsigned char *smem, float (*zsum)[32])
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x16 __attribute__((ext_vector_type(16)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    typedef s16x4 __attribute__((address_space(3))) *Tr;
    union Frag { bf16x8 v; uint32_t w[4]; s16x4 h[2]; };
    constexpr int NC = SLICE_COLS, LOADS = direct_loads(ROPE), DEPTH = direct_depth(D, ROPE), GROUP = LOADS * 1024, NS = D / 16;
    static_assert(DEPTH >= 2 && DIRECT_WAVES * NC * 4096 <= direct_lds(D), "LDS");
    const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int CS = D / 32 / NC;                            // slices side by side
    const int at = slice / CS, ct = slice % CS * NC;           // tile of 32 rows, first tile of 32 columns
    const u16 *kb = k + (size_t)bh * N * D + at * 32, *vb = v + (size_t)bh * N * D + ct * 32;
    const char *rb = reinterpret_cast<const char *>(rope_tab) + at * 64;       // 16 pairs' words: as many bytes as 32 channels of K
    unsigned char *ring = smem + wave * (DEPTH * GROUP);
    const unsigned ring_lds = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) void *)ring);
    const int groups = (N + 15) >> 4, mine = (groups - wave + DIRECT_WAVES - 1) / DIRECT_WAVES;      // this wave's: wave, wave + 8, ...
    auto load = [](const void *base, unsigned off, unsigned lds) __attribute__((always_inline)) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds), "v"(off), "s"(base) : "memory", "m0");
    };
    auto fetch = [&](int i, int slot) __attribute__((always_inline)) {
        const int row = min((wave + i * DIRECT_WAVES) * 16 + (lane >> 2), N - 1);
        const unsigned off = (unsigned)row * (unsigned)(D * 2) + (unsigned)(lane & 3) * 16u, dst = ring_lds + (unsigned)(slot * GROUP);
        load(kb, off, dst);
#pragma unroll
        for (int c = 0; c < NC; ++c) load(vb + c * 32, off, dst + 1024u * (1 + c));
        if (ROPE) load(rb, off, dst + 1024u * (1 + NC));
    };
    // lane (l32, hh): tokens 8 hh .. + 7 of channel l32
    const unsigned toff = (unsigned)((8 * hh + ((l32 >> 2) & 3)) * 64 + (2 * (l32 >> 4) + ((l32 & 3) >> 1)) * 16 + 8 * (l32 & 1));
    auto read = [&](Frag &f, int slot, int piece) __attribute__((always_inline)) {
        unsigned char *p = ring + slot * GROUP + piece * 1024 + toff;
        f.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Tr)(__attribute__((address_space(3))) void *)p);
        f.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((Tr)(__attribute__((address_space(3))) void *)(p + 256));
    };
    auto other = [](uint32_t x) __attribute__((always_inline)) -> uint32_t {           // the neighbouring channel's word
        return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xb1, 0xf, 0xf, false);
    };
    f32x16 acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[c][i] = 0.f;
    float z = 0.f;
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (i < mine) fetch(i, i);
    int slot = 0;
    for (int i = 0; i < mine; ++i) {
        constexpr int AHEAD = (DEPTH - 1) * LOADS;
        if (i + DEPTH <= mine) __builtin_amdgcn_s_waitcnt(0x0F70 | (AHEAD & 15) | (AHEAD >> 4) << 14);      // vmcnt: the groups behind this one
        else __builtin_amdgcn_s_waitcnt(0x0F70);
        asm volatile("" ::: "memory");
        Frag fk, fv[NC], fr;
        read(fk, slot, 0);
#pragma unroll
        for (int c = 0; c < NC; ++c) read(fv[c], slot, 1 + c);
        if (ROPE) read(fr, slot, 1 + NC);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // read: the slot is free
        if (i + DEPTH < mine) fetch(i + DEPTH, slot);
        const int left = N - (wave + i * DIRECT_WAVES) * 16 - 8 * hh;
        if (__builtin_expect((wave + i * DIRECT_WAVES) * 16 + 16 > N, 0)) {      // tokens past the end count as zeros
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t m = 2 * j + 1 < left ? 0xffffffffu : 2 * j < left ? 0xffffu : 0u;
                fk.w[j] &= m;
#pragma unroll
                for (int c = 0; c < NC; ++c) fv[c].w[j] &= m;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) fk.w[j] = ride_relu(fk.w[j]);
        if (ct == 0)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                z += __uint_as_float(fk.w[j] << 16);
                z += __uint_as_float(fk.w[j] & 0xffff0000u);
            }
        if (ROPE) {
            // channel 2p: x c - y s, channel 2p + 1: y c + x s; the even lane holds x and the cosines, the odd one y and the sines
            const bool odd = lane & 1;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t pk = other(fk.w[j]), pr = other(fr.w[j]), cw = odd ? pr : fr.w[j], sw = odd ? fr.w[j] : pr;
                const f16x2 cc = __builtin_bit_cast(f16x2, cw), ss = __builtin_bit_cast(f16x2, sw);
                const float m0 = __uint_as_float(fk.w[j] << 16), m1 = __uint_as_float(fk.w[j] & 0xffff0000u);
                const float o0 = __uint_as_float(pk << 16), o1 = __uint_as_float(pk & 0xffff0000u);
                const float s0 = odd ? (float)ss[0] : -(float)ss[0], s1 = odd ? (float)ss[1] : -(float)ss[1];
                f32x2 r = {m0 * (float)cc[0] + o0 * s0, m1 * (float)cc[1] + o1 * s1};
                fk.w[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fk.v, fv[c].v, acc[c], 0, 0, 0);
        slot = slot + 1 == DEPTH ? 0 : slot + 1;
    }
    // register 4 g + t of lane (l32, hh): row 8 g + 4 hh + t, column l32.  [wave][c][g][lane] of four floats
    __syncthreads();
    float4 *sums = reinterpret_cast<float4 *>(smem);
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            sums[((wave * NC + c) * 4 + g) * 64 + lane] = make_float4(acc[c][4 * g], acc[c][4 * g + 1], acc[c][4 * g + 2], acc[c][4 * g + 3]);
    z += __shfl_xor(z, 32);
    if (lane < 32) zsum[wave][lane] = z;
    __syncthreads();
    for (int e = tid; e < NC * 256; e += DIRECT_WAVES * 64) {
        float4 t = sums[e];
#pragma unroll
        for (int w = 1; w < DIRECT_WAVES; ++w) {
            const float4 x = sums[w * (NC * 256) + e];
            t.x += x.x; t.y += x.y; t.z += x.z; t.w += x.w;
        }
        const int c = e >> 8, g = (e >> 6) & 3, l = e & 63;
        f32x2 lo = {t.x, t.y}, hi = {t.z, t.w};
        uint2 o;
        o.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2));
        o.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2));
        ride_store(reinterpret_cast<uint64_t *>(hfrag + (size_t)bh * D * D + (((ct + c) * NS + 2 * at + (g >> 1)) * 64 + (g & 1) * 32 + (l & 31)) * 8 + 4 * (l >> 5)),
                   (uint64_t)o.x | (uint64_t)o.y << 32);
    }
    if (ct == 0 && tid < 32) {
        float t = zsum[0][tid];
#pragma unroll
        for (int w = 1; w < DIRECT_WAVES; ++w) t += zsum[w][tid];
        ride_storef(Z + (size_t)bh * D + at * 32 + tid, t);
    }
}

// A word of a head, or (from B H on) of a sample, whose gate tasks count in it; each has a cache line, since additions to one line come one after
// the other: 12 words of 32 gate tasks each in a line held up a call of N = 1024 by 7 of 23 us.
__device__ inline uint64_t *ride_word(CallRef a, int i) { return a.ride.words + i * RIDE_STRIDE; }
// one more rider or tile counted in a word; at `full` nobody needs it any more
__device__ inline uint64_t ride_count(CallRef a, int i, uint64_t inc, uint64_t full)
{
    uint64_t *w = ride_word(a, i);
    const uint64_t tag = a.ride.tag;
    const uint64_t now = ride_settle(w, tag, inc, __hip_atomic_fetch_add(w, inc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + inc);
    if ((now & RIDE_COUNT) == full) ride_store(w, 0);
    return now & RIDE_COUNT;
}

// Rider i: a slice of a head's state, or a share of a sample's partial sums.  smem: direct_lds(D); small: [DIRECT_WAVES][32] floats
template <int D, bool ROPE>
__device__ inline __attribute__((always_inline)) void ride(int i, unsigned char *smem, float (*small)[32])
{
    CallRef a = call_args();
    constexpr int SLICES = slices_per_head(D);
    const int H = a.H, BH = a.B * H, tid = threadIdx.x;
    if (a.ride.polls < 0) return;
    if (i < BH * SLICES) {
        const int bh = slice_head(BH, SLICES, i), slice = slice_of(BH, SLICES, i);
        state_slice<D, ROPE>(reinterpret_cast<const u16 *>(a.k), reinterpret_cast<const u16 *>(a.v), a.N, a.rope_tab, a.ride.hfrag, a.ride.Z, bh, slice, smem, small);
        ride_published();
        if (tid == 0) ride_count(call_args(), bh, 1, call_args().ride.full);
    } else {
        const int x = i - BH * SLICES, b = x / a.ride.gate_tasks, part = x - b * a.ride.gate_tasks;
        const int nv = a.ride.nparts * 4, per = (nv + a.ride.gate_tasks - 1) / a.ride.gate_tasks;
        ride_gate<512>(a.ride.x_t, a.ride.w_gate, a.ride.b_gate, a.N, H * D, a.ride.gate_tok, a.ride.nparts, a.ride.gate_sums, b, min(nv, part * per),
                       min(nv, (part + 1) * per), smem);
        ride_published();
        int *last = reinterpret_cast<int *>(&small[0][0]);
        if (tid == 0) {
            const uint64_t all = call_args().ride.gate_tasks;
            *last = ride_count(call_args(), BH + b, 1, all) == all;
        }
        __syncthreads();
        if (*last && tid < H) ride_count(call_args(), b * H + tid, 1, call_args().ride.full);
    }
}

// What a tile does whose head's word does not say in time that riders have: all of it, for its head and sample.
template <int D, bool ROPE>
__device__ inline __attribute__((always_inline)) void ride_alone(int bh, unsigned char *smem, float (*small)[32])
{
    CallRef a = call_args();
    for (int i = 0; i < slices_per_head(D); ++i) {
        state_slice<D, ROPE>(reinterpret_cast<const u16 *>(a.k), reinterpret_cast<const u16 *>(a.v), a.N, a.rope_tab, a.ride.hfrag, a.ride.Z, bh, i, smem, small);
        __syncthreads();
    }
    if (a.ride.nparts > 0)
        ride_gate<512>(a.ride.x_t, a.ride.w_gate, a.ride.b_gate, a.N, a.H * D, a.ride.gate_tok, a.ride.nparts, a.ride.gate_sums, bh / a.H, 0, a.ride.nparts * 4, smem);
    ride_published();
}

}  // namespace salad
