// Top-K dynamic block mask (Sec. 3 "Top-K attention", App. A.1.2), d = 128, bf16.
//   step 1  kblock_mean_kernel      mean key of every run of key_block consecutive tokens of the head's own order
//   step 2  topk_select_kernel      per query token: the topk key blocks with the largest q . mean, as a 64-bit mask
//           topk_tile_lists_kernel  per tile of 256 queries: the 64-token blocks the attention kernel has to visit
//   step 3  the large-tile attention kernel in its token-mask mode
// The selection is an integer decided by floating point, so its arithmetic is fixed: fp32 throughout, a block's sum
// taken token by token in ascending order and divided by the token count, a score accumulated over the channels in
// ascending order with a fused multiply-add, a block replaces a kept one only on a strictly larger score (ties go
// to the lower index).  No fast-math: the division and the fused multiply-adds are the IEEE ones.  (Scores from the matrix cores decide where they
// differ by more than they can be off; see topk_select_kernel.)
#include "salad_internal.h"

namespace salad {

namespace {
constexpr int D = 128;
}  // namespace

// grid (nbk, BH), 64 threads: thread c sums channels 2 c and 2 c + 1 of the block's keys in the order of the head's positions
// (App. A.1.1: position p of a temporal head is stored row (p mod T) HW + p div T; a spatial head's is row p).
// A read of K by 480 single waves: what counts is the bytes in flight, 64 rows or 16 KB each, and few instructions per row, so a row
// number is one lane's and is read from it (stepping the position row by row took 37.6 us).  At N = 32760, 12 heads, 40 key blocks
// 21.3 us for either order = 4.7 TB/s; with 16 rows of 2-byte loads in flight 29.2 us spatial and 52.7 temporal.
__global__ __launch_bounds__(64) void kblock_mean_kernel(const u16 *__restrict__ k, int N, int key_block, int nbk,
                                                         float *__restrict__ means, unsigned long long kind_mask, int H,
                                                         int T, int HW)
{
    const int J = blockIdx.x, bh = blockIdx.y, c = threadIdx.x;
    const int t0 = J * key_block, t1 = min(N, t0 + key_block);
    const bool temporal = T > 1 && ((kind_mask >> (bh % H)) & 1ull);
    // position p = loc T + f (location loc, frame f) is stored row f HW + loc (spatial: one frame): lane c holds it for position t + c
    const int frames = temporal ? T : 1, step = temporal ? HW : 0, df = 64 % frames, dloc = 64 / frames;
    int loc = (t0 + c) / frames, f = t0 + c - loc * frames;
    const uint32_t *base = reinterpret_cast<const uint32_t *>(k + (size_t)bh * N * D);
    float s0 = 0.f, s1 = 0.f;
    auto add_rows = [&](auto count, int row, int first) __attribute__((always_inline)) {
        constexpr int U = decltype(count)::value;
        uint32_t x[U];
#pragma unroll
        for (int i = 0; i < U; ++i) x[i] = (base + (size_t)__builtin_amdgcn_readlane(row, first + i) * (D / 2))[c];
#pragma unroll
        for (int i = 0; i < U; ++i) {
            s0 = __fadd_rn(s0, __uint_as_float(x[i] << 16));
            s1 = __fadd_rn(s1, __uint_as_float(x[i] & 0xffff0000u));
        }
    };
    int t = t0;
    for (; t + 64 <= t1; t += 64) {
        add_rows(std::integral_constant<int, 64>{}, f * step + loc, 0);
        f += df;
        loc += dloc;
        if (f >= frames) { f -= frames; ++loc; }
    }
    const int row = f * step + loc;
    int i = 0;
    for (; t + i + 8 <= t1; i += 8) add_rows(std::integral_constant<int, 8>{}, row, i);
    for (; t + i < t1; ++i) add_rows(std::integral_constant<int, 1>{}, row, i);
    float2 *out = reinterpret_cast<float2 *>(means + ((size_t)bh * nbk + J) * D);
    out[c] = make_float2(__fdiv_rn(s0, (float)(t1 - t0)), __fdiv_rn(s1, (float)(t1 - t0)));
}

hipError_t launch_kblock_mean(const u16 *k, int BH, int N, int key_block, int nbk, float *means, unsigned long long kind_mask,
                              int H, int T, int HW, hipStream_t st)
{
    launch_kernel(kblock_mean_kernel, dim3(nbk, BH), dim3(64), 0, st, k, N, key_block, nbk, means, kind_mask, H, T, HW);
    return take_launch_status();
}

// Selection for more than topk key blocks.  The definition's scores, 128-step chains of fp32 multiply-adds, are 5120 vector instructions a wave at 40
// blocks (91 us at N = 32760, 12 heads); here scores come off the matrix cores first: a mean is the sum of three bf16 values (24 bits; the last
// part is below 2^-26 of it), a query is bf16 as it is, products are exact and sums fp32.  Such a score is off the definition's by no more than
//   (SELECT_MATRIX + SELECT_CHAIN) |q| |m| + 2^-17 of itself:  8 products of 16 channels, 17 additions each that may cut at 2^-23 of sums up to
//   |q| |m|, the two small parts, which go first, at 2^-9 of that, and what the three parts leave; the chain's 128 roundings of 2^-24 of sums up to
//   |q| |m| (both reached only where the first channels have all of it); the block's number in the six low bits
// so where the topk-th and the next score are further apart than twice that, the selection is the definition's.  Where they are not (ties and
// values that are not finite among them), the scores that are open, within that of both, are computed as defined, a lane each, and selected
// with the definition's rules; a workgroup with a wave that has many of them does all of its queries the definition's way.
constexpr float SELECT_MATRIX = (8 * 17 + 2) * 0x1p-23f, SELECT_CHAIN = (128 + 1) * 0x1p-24f;
typedef __bf16 sel_bf16x8 __attribute__((ext_vector_type(8)));
typedef float sel_f32x16 __attribute__((ext_vector_type(16)));
// Open scores that a wave computes, for each tile of 32 key blocks: what fits the products' LDS with the means, and about where all scores of the
// workgroup's queries the definition's way are no more work
constexpr int SELECT_PAIRS = 320;

// the best SLOTS of scores offered in ascending order of blocks: a strict comparison keeps earlier blocks ahead on ties; an empty slot (index
// -1) always gives way; once placed, the displaced pairs all move down one slot
template <int SLOTS> struct BestBlocks {
    float best[SLOTS];
    int bidx[SLOTS];
    __device__ inline void clear()
    {
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) { best[i] = -INFINITY; bidx[i] = -1; }
    }
    __device__ inline void offer(float v, int id)
    {
        bool carry = false;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i) {
            const bool take = (id >= 0) && (carry || bidx[i] < 0 || v > best[i]);
            carry = carry || take;
            const float tv = best[i];
            const int ti = bidx[i];
            best[i] = take ? v : tv;
            bidx[i] = take ? id : ti;
            v = take ? tv : v;
            id = take ? ti : id;
        }
    }
    __device__ inline unsigned long long mask(int topk) const
    {
        unsigned long long m = 0ull;
#pragma unroll
        for (int i = 0; i < SLOTS; ++i)
            if (i < topk && bidx[i] >= 0) m |= 1ull << bidx[i];
        return m;
    }
};

// a score as defined; chunk c of the mean at c ^ swap
__device__ inline __attribute__((always_inline)) float defined_score(const u16 *row, const float4 *m, int swap = 0)
{
    float x = 0.f;
#pragma unroll 4
    for (int c = 0; c < D / 8; ++c) {
        const uint4 v = *reinterpret_cast<const uint4 *>(row + c * 8);
        const float4 m0 = m[(2 * c) ^ swap], m1 = m[(2 * c + 1) ^ swap];
        x = __fmaf_rn(__uint_as_float(v.x << 16), m0.x, x); x = __fmaf_rn(__uint_as_float(v.x & 0xffff0000u), m0.y, x);
        x = __fmaf_rn(__uint_as_float(v.y << 16), m0.z, x); x = __fmaf_rn(__uint_as_float(v.y & 0xffff0000u), m0.w, x);
        x = __fmaf_rn(__uint_as_float(v.z << 16), m1.x, x); x = __fmaf_rn(__uint_as_float(v.z & 0xffff0000u), m1.y, x);
        x = __fmaf_rn(__uint_as_float(v.w << 16), m1.z, x); x = __fmaf_rn(__uint_as_float(v.w & 0xffff0000u), m1.w, x);
    }
    return x;
}

// grid (ceil(N / 256), BH), 256 threads: a wave owns 64 queries, two column sets of the products; JT tiles of 32 key blocks.  N = 32760, 12 heads (us, all
// mask steps; before: the definition alone): 4 of 40 blocks 147 -> 110, 8 of 64 251 -> 141; 5 heads, N = 7800, 1 of 61 97 -> 43.  Two to four turns
// of 256 queries a workgroup, for which the means are taken apart once, gave 135 where one gave 122.
// What all keys have in common widens the bound and leaves the scores' differences as they are.  4 of 40 blocks of normal keys with as much as 1, 3, 10, 30
// of it in every channel: 113, 116, 123, 145 (before 141; where a wave took all scores of
// its doubtful queries one query at a time, up to 6 of them, 201, 208, 208, -).  All keys equal, so that
// every score is open: 212 (144).  Less the average of 8 means it was 131, and 133, 135, 142, 180 there, with fewer waves for its registers.
template <int JT, int SLOTS>
__global__ __launch_bounds__(256, 2) void topk_select_kernel(const u16 *__restrict__ q, const float *__restrict__ means, int N, int nbk, int topk,
                                                             unsigned long long *__restrict__ mask)
{
    constexpr int NS = D / 16, PAIRS = JT * SELECT_PAIRS;
    __shared__ __attribute__((aligned(16))) uint4 frag[3][JT][NS][64];          // operand order: lane (row l32, channels 8 hh ..)
    __shared__ float norm[JT * 32];
    __shared__ int many;                           // a wave has more open scores than lanes (1), than it computes (2)
    const int bh = blockIdx.y, tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hh = lane >> 5;
    const float *mb = means + (size_t)bh * nbk * D;
    const float4 *mf = reinterpret_cast<const float4 *>(mb);
    if (nbk <= topk) {                      // every block
        const int n = blockIdx.x * 256 + tid;
        if (n < N) mask[(size_t)bh * N + n] = ~0ull >> (64 - nbk);
        return;
    }
    if (tid < JT * 32) norm[tid] = 0.f;
    if (tid == 0) many = 0;
    __syncthreads();
    // the three parts of the means, largest last
    for (int x = tid; x < JT * NS * 64; x += 256) {
        const int jt = x / (NS * 64), st = x / 64 % NS, J = jt * 32 + (x & 31), c = st * 16 + ((x >> 5) & 1) * 8;
        uint32_t w[3][4];
        float v[8], t = 0.f;
        const float4 *m = reinterpret_cast<const float4 *>(mb + min(J, nbk - 1) * D + c);
        *reinterpret_cast<float4 *>(v) = m[0];
        *reinterpret_cast<float4 *>(v + 4) = m[1];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            float a = J < nbk ? v[2 * e] : 0.f, b = J < nbk ? v[2 * e + 1] : 0.f;
            t = fmaf(a, a, fmaf(b, b, t));
#pragma unroll
            for (int s = 2; s >= 0; --s) {
                const uint32_t ha = f32_to_bf16_rne(a), hb = f32_to_bf16_rne(b);
                w[s][e] = ha | hb << 16;
                a -= __uint_as_float(ha << 16);
                b -= __uint_as_float(hb << 16);
            }
        }
#pragma unroll
        for (int s = 0; s < 3; ++s) frag[s][jt][st][x & 63] = make_uint4(w[s][0], w[s][1], w[s][2], w[s][3]);
        atomicAdd(&norm[J], t);            // for a bound: the order does not matter
    }
    __syncthreads();
    float mm = norm[lane & (JT * 32 - 1)];                       // largest |m|^2; a NaN in it is one in the scores, too
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) mm = fmaxf(mm, __shfl_xor(mm, o));
    const int n0 = blockIdx.x * 256 + (tid >> 6) * 64;
    uint4 qf[2][NS];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const uint4 *src = reinterpret_cast<const uint4 *>(q + ((size_t)bh * N + min(n0 + u * 32 + l32, N - 1)) * D) + hh;
#pragma unroll
        for (int st = 0; st < NS; ++st) qf[u][st] = src[st * 2];
    }
    sel_f32x16 acc[2][JT];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[u][jt][r] = 0.f;
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int st = 0; st < NS; ++st)
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) {
                const sel_bf16x8 a = __builtin_bit_cast(sel_bf16x8, frag[s][jt][st][lane]);
#pragma unroll
                for (int u = 0; u < 2; ++u)
                    acc[u][jt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, __builtin_bit_cast(sel_bf16x8, qf[u][st]), acc[u][jt], 0, 0, 0);
            }
    const unsigned long long every = ~0ull >> (64 - nbk);
    unsigned long long doubtful = 0ull;                            // bit i: query n0 + i
    float above[2], below[2];
    bool whole[2];                                                 // nothing is known
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        float qq = 0.f;
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            const uint32_t w[4] = {qf[u][st].x, qf[u][st].y, qf[u][st].z, qf[u][st].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float x = __uint_as_float(w[e] << 16), y = __uint_as_float(w[e] & 0xffff0000u);
                qq = fmaf(x, x, fmaf(y, y, qq));
            }
        }
        qq += __shfl_xor(qq, 32);
        // the lane's half of its query's scores (rows 8 g + 4 hh + t of a tile), each with its block's number; the SLOTS + 1 largest, descending
        float b[SLOTS + 1];
#pragma unroll
        for (int i = 0; i <= SLOTS; ++i) b[i] = -INFINITY;
        bool finite = true;
        auto put = [&](float v) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i <= SLOTS; ++i) {
                const float hi = fmaxf(b[i], v);
                v = fminf(b[i], v);
                b[i] = hi;
            }
        };
#pragma unroll
        for (int jt = 0; jt < JT; ++jt)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int J = jt * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
                const float v = acc[u][jt][r];
                finite = finite && (fabsf(v) < INFINITY || J >= nbk);
                put(J < nbk ? __uint_as_float((__float_as_uint(v) & ~63u) | (uint32_t)J) : -INFINITY);
            }
        float other[SLOTS + 1];
#pragma unroll
        for (int i = 0; i <= SLOTS; ++i) other[i] = __shfl_xor(b[i], 32);
#pragma unroll
        for (int i = 0; i <= SLOTS; ++i) put(other[i]);
        unsigned long long m = 0ull;
        float last = b[0], next = b[0];
#pragma unroll
        for (int i = 0; i <= SLOTS; ++i) {
            if (i < topk) {
                m |= 1ull << (__float_as_uint(b[i]) & 63u);
                last = b[i];
            }
            if (i == topk) next = b[i];
        }
        // tiny norms: the parts of the means, or the queries, may be below what a product takes.  From 1e-13 on all that is lost below 2^-126 is
        // less than 2e-5 of the bound.  The product of the two squares may be below 2^-149 then, that of the norms is not.
        const unsigned long long bad = __ballot(!(finite && qq > 1e-26f && mm > 1e-26f));
        const bool bounded = !(((uint32_t)bad | (uint32_t)(bad >> 32)) >> l32 & 1u);
        const float margin = 2 * (SELECT_MATRIX + SELECT_CHAIN) * (sqrtf(qq) * sqrtf(mm)) + 1.6e-5f * fmaxf(fabsf(last), fabsf(next));
        const bool sure = bounded && last - next > margin;
        const unsigned long long no = __ballot(!sure);
        doubtful |= (no & 0xffffffffull) << (u * 32);
        const int n = n0 + u * 32 + l32;
        if (hh == 0 && sure && n < N) mask[(size_t)bh * N + n] = m;
        above[u] = next + margin;
        below[u] = last - margin;
        whole[u] = !bounded;
    }
    if (N - n0 < 64) doubtful &= N > n0 ? (1ull << (N - n0)) - 1ull : 0ull;
    // one query in 64, which is usual where there is any: its scores as defined, a lane a block (16 heads, N = 270 10.1 -> 9.0 us against the list below)
    if (__popcll(doubtful) == 1) {
        const int i = __builtin_ctzll(doubtful);
        const u16 *row = q + ((size_t)bh * N + n0 + i) * D;
        const float x = defined_score(row, mf + min(lane, nbk - 1) * (D / 4));
        unsigned long long m;
        if (__all(fabsf(x) < INFINITY)) {              // a block is chosen if fewer than topk are ahead of it
            int ahead = 0;
            for (int J = 0; J < nbk; ++J) {
                const float y = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), J));
                ahead += y > x || (y == x && J < lane);
            }
            m = __ballot(lane < nbk && ahead < topk);
        } else {
            BestBlocks<SLOTS> best;
            best.clear();
            for (int J = 0; J < nbk; ++J) best.offer(__uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(x), J)), J);
            m = best.mask(topk);
        }
        if (lane == 0) mask[(size_t)bh * N + n0 + i] = m;
        doubtful = 0ull;
    }
    // of query n0 + lane, if it is doubtful: blocks ahead of the first left out by more than the margin are chosen, those behind the last chosen by more
    // are not; the others are open
    unsigned long long chosen = 0ull, open = 0ull;
    int first = 0, pairs = 0;               // this lane's in the wave's list; all of them
    const bool mine = doubtful >> lane & 1ull;
    if (doubtful) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            uint32_t yes[2] = {}, may[2] = {};
#pragma unroll
            for (int jt = 0; jt < JT; ++jt) {
#pragma unroll
                for (int r = 15; r >= 0; --r) {
                    const float v = acc[u][jt][r];
                    yes[jt] += yes[jt] + (v > above[u]);
                    may[jt] += may[jt] + !(v < below[u]);
                }
                may[jt] &= ~yes[jt];
            }
            // bit r of these two halves -> bit of the block
            auto of_blocks = [&](const uint32_t (&x)[2]) __attribute__((always_inline)) -> unsigned long long {
                uint32_t w[2];
#pragma unroll
                for (int jt = 0; jt < 2; ++jt) {
                    uint32_t t = (x[jt] | x[jt] << 8) & 0x00ff00ffu;
                    t = ((t | t << 4) & 0x0f0f0f0fu) << 4 * hh;
                    auto both = __builtin_amdgcn_permlane32_swap(t, t, false, false);
                    w[jt] = both[0] | both[1];
                }
                return (unsigned long long)w[1] << 32 | w[0];
            };
            const unsigned long long ahead = of_blocks(yes), among = of_blocks(may);
            if (hh == u && mine) {
                chosen = whole[u] ? 0ull : ahead & every;
                open = whole[u] ? every : among & every;
            }
        }
#pragma unroll
        for (int i = 0; i < 7; ++i) {
            const unsigned long long x = __ballot(__popcll(open) >> i & 1);
            first += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(x >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)x, 0)) << i;
            pairs += __popcll(x) << i;
        }
        if (lane == 0 && pairs > 64) atomicOr(&many, pairs > PAIRS ? 3 : 1);
    }
    __syncthreads();
    const int how = many;
    if (__builtin_expect(how & 2, 0)) {
        // the definition, a thread a query, the means as broadcast words in LDS, GROUP blocks' chains at a time
        constexpr int GROUP = 20;
        float *sm = reinterpret_cast<float *>(frag);
        for (int i = tid; i < nbk * D; i += 256) sm[i] = mb[i];
        __syncthreads();
        const int n = blockIdx.x * 256 + tid;
        const uint4 *row = reinterpret_cast<const uint4 *>(q + ((size_t)bh * N + min(n, N - 1)) * D);
        BestBlocks<SLOTS> best;
        best.clear();
#pragma unroll 1
        for (int J = 0; J < nbk; J += GROUP) {
            float x[GROUP] = {};
            const float *m[GROUP];
#pragma unroll
            for (int i = 0; i < GROUP; ++i) m[i] = sm + min(J + i, nbk - 1) * D;
            uint4 v = row[0];
#pragma unroll 1
            for (int c = 0; c < D / 8; ++c) {
                const uint32_t w[4] = {v.x, v.y, v.z, v.w};
                v = row[min(c + 1, D / 8 - 1)];
                float qv[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) qv[e] = (e & 1) ? __uint_as_float(w[e >> 1] & 0xffff0000u) : __uint_as_float(w[e >> 1] << 16);
#pragma unroll
                for (int i = 0; i < GROUP; ++i) {
                    const float4 m0 = *reinterpret_cast<const float4 *>(m[i] + c * 8), m1 = *reinterpret_cast<const float4 *>(m[i] + c * 8 + 4);
                    x[i] = __fmaf_rn(qv[0], m0.x, x[i]); x[i] = __fmaf_rn(qv[1], m0.y, x[i]);
                    x[i] = __fmaf_rn(qv[2], m0.z, x[i]); x[i] = __fmaf_rn(qv[3], m0.w, x[i]);
                    x[i] = __fmaf_rn(qv[4], m1.x, x[i]); x[i] = __fmaf_rn(qv[5], m1.y, x[i]);
                    x[i] = __fmaf_rn(qv[6], m1.z, x[i]); x[i] = __fmaf_rn(qv[7], m1.w, x[i]);
                }
            }
#pragma unroll
            for (int i = 0; i < GROUP; ++i)
                if (J + i < nbk) best.offer(x[i], J + i);
        }
        if (n < N) mask[(size_t)bh * N + n] = best.mask(topk);
        return;
    }
    // the open scores as defined, a lane a (query, block) pair; where a wave has many, which read many rows of means at once, from LDS, chunk c of
    // row J at c ^ (J % 16)
    float4 *lm = reinterpret_cast<float4 *>(frag);
    if (how) {
        for (int i = tid; i < nbk * (D / 4); i += 256) lm[i ^ (i / (D / 4) & 15)] = mf[i];
        __syncthreads();
    }
    if (!doubtful) return;                  // (by the numbers of the blocks in the scores a query can be doubtful and no score be open)
    u16 *list = reinterpret_cast<u16 *>(lm + JT * 32 * (D / 4)) + (tid >> 6) * (PAIRS * 3);
    float *score = reinterpret_cast<float *>(list + PAIRS);
    static_assert(sizeof(frag) >= JT * 32 * D * 4 + 4 * PAIRS * 6, "LDS");
    {
        int i = first;
        for (unsigned long long o = open; o; o &= o - 1ull) list[i++] = (u16)(lane << 6 | __builtin_ctzll(o));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int i = lane; i < pairs; i += 64) {
        const int J = list[i] & 63;
        const u16 *row = q + ((size_t)bh * N + n0 + (list[i] >> 6)) * D;
        if (how) score[i] = defined_score(row, lm + J * (D / 4), J & 15);
        else score[i] = defined_score(row, mf + J * (D / 4));
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (mine) {
        BestBlocks<SLOTS> best;
        best.clear();
        int i = first;
        for (unsigned long long o = open; o; o &= o - 1ull) best.offer(score[i++], __builtin_ctzll(o));
        mask[(size_t)bh * N + n0 + lane] = chosen | best.mask(topk - __popcll(chosen));
    }
}

hipError_t launch_topk_select(const u16 *q, const float *means, int BH, int N, int nbk, int topk,
                              unsigned long long *mask, hipStream_t st)
{
    const dim3 grid((N + 255) / 256, BH), block(256);
    auto go = [&](auto kern) { launch_kernel(kern, grid, block, 0, st, q, means, N, nbk, topk, mask); };
    if (nbk <= 32) topk <= 4 ? go(topk_select_kernel<1, 4>) : go(topk_select_kernel<1, 8>);
    else topk <= 4 ? go(topk_select_kernel<2, 4>) : go(topk_select_kernel<2, 8>);
    return take_launch_status();
}

// grid (ntiles, BH), 256 threads: thread t holds the mask of query 256 tile + t; attention wave w of the tile owns
// queries 32 w .. 32 w + 31.  Entry = block | J << 16 | wave bits << 24, key blocks ascending, their 64-token
// blocks ascending.
__global__ __launch_bounds__(256) void topk_tile_lists_kernel(const unsigned long long *__restrict__ mask, int N, int nb,
                                                              int bpb, int nbk, int ntiles, int cap,
                                                              uint32_t *__restrict__ lists, int32_t *__restrict__ counts)
{
    __shared__ unsigned long long wmask[8];
    __shared__ int offs[65];
    const int tile = blockIdx.x, bh = blockIdx.y, t = threadIdx.x, lane = t & 63;
    const int n = tile * 256 + t;
    unsigned long long m = n < N ? mask[(size_t)bh * N + n] : 0ull;
    // OR over each run of 32 lanes
#pragma unroll
    for (int o = 1; o < 32; o <<= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)m, o), hi = __shfl_xor((uint32_t)(m >> 32), o);
        m |= ((unsigned long long)hi << 32) | lo;
    }
    if ((lane & 31) == 0) wmask[t >> 5] = m;
    __syncthreads();
    if (t < 64) {
        unsigned long long u = 0ull;
#pragma unroll
        for (int w = 0; w < 8; ++w) u |= wmask[w];
        const int J = t;
        int cnt = 0;
        if (J < nbk && ((u >> J) & 1ull)) cnt = min(nb, (J + 1) * bpb) - J * bpb;
        // exclusive prefix sum over the 64 lanes
        int incl = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int x = __shfl_up(incl, o);
            if (lane >= o) incl += x;
        }
        offs[J] = incl - cnt;
        if (J == 63) offs[64] = incl;
    }
    __syncthreads();
    uint32_t *out = lists + ((size_t)bh * ntiles + tile) * cap;
    for (int J = 0; J < nbk; ++J) {
        const int o0 = offs[J], c = offs[J + 1] - o0;
        if (c == 0) continue;
        uint32_t bits = 0u;
#pragma unroll
        for (int w = 0; w < 8; ++w) bits |= (uint32_t)((wmask[w] >> J) & 1ull) << (24 + w);
        for (int i = t; i < c; i += 256) out[o0 + i] = (uint32_t)(J * bpb + i) | ((uint32_t)J << 16) | bits;
    }
    if (t == 0) counts[bh * ntiles + tile] = offs[64];
}

hipError_t launch_topk_tile_lists(const unsigned long long *mask, int BH, int N, int nb, int key_block, int nbk,
                                  uint32_t *lists, int32_t *counts, hipStream_t st)
{
    const int ntiles = (nb + 3) / 4;
    launch_kernel(topk_tile_lists_kernel, dim3(ntiles, BH), dim3(256), 0, st, mask, N, nb, key_block / 64, nbk,
                       ntiles, tile_list_cap(nb), lists, counts);
    return take_launch_status();
}

// ---- regrouping by key block -----------------------------------------------------------------------------------
// The queries that keep key block J are gathered into runs of 256 ("query tiles" of the attention kernel), so that
// the work is the kept (query, key block) pairs whatever the selection looks like; every pair gets a slot in
// [0, N * kk) of its (sample, head), key blocks ascending, queries ascending inside a key block.

// Chunks of 1024 queries.  Wave w of a chunk publishes, for every key block J, the ballot of its 64 queries' bit J.
__device__ inline void chunk_ballots(unsigned long long m, int nbk, unsigned long long (*wb)[64], int wv, int lane)
{
    for (int J = 0; J < nbk; ++J) {
        const unsigned long long bal = __ballot((m >> J) & 1ull);
        if (lane == 0) wb[wv][J] = bal;
    }
}

// grid (nch, BH), 1024 threads: ccnt[(bh * nch + chunk) * 64 + J] = queries of the chunk keeping block J
__global__ __launch_bounds__(1024) void topk_count_kernel(const unsigned long long *__restrict__ mask, int N, int nbk,
                                                          int nch, int32_t *__restrict__ ccnt)
{
    __shared__ unsigned long long wb[16][64];
    const int chunk = blockIdx.x, bh = blockIdx.y, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int n = chunk * 1024 + t;
    const unsigned long long m = n < N ? mask[(size_t)bh * N + n] : 0ull;
    chunk_ballots(m, nbk, wb, wv, lane);
    __syncthreads();
    if (t < 64) {
        int c = 0;
        if (t < nbk)
#pragma unroll
            for (int w = 0; w < 16; ++w) c += __popcll(wb[w][t]);
        ccnt[((size_t)bh * nch + chunk) * 64 + t] = c;
    }
}

// grid (BH), 64 threads (lane J = key block J).  cbase[(bh * nch + chunk) * 64 + J] = first slot (within the
// sample-head) of the chunk's queries keeping J = slots of key blocks < J + those of earlier chunks.  Tile descriptors
// (bh, J, first slot, queries) for every run of up to 256 queries, key blocks in order, at desc[bh * mt ...]; the
// unused descriptors of the sample-head's mt are written with zero queries (their workgroups return at once).
__global__ __launch_bounds__(64) void topk_plan_kernel(const int32_t *__restrict__ ccnt, int nbk, int nch,
                                                       int32_t *__restrict__ cbase, uint4 *__restrict__ desc, int mt)
{
    const int bh = blockIdx.x, J = threadIdx.x;
    // the per-chunk counts of this key block, 32 chunks' loads in flight at a time (the loop is latency-bound)
    const int32_t *cc = ccnt + (size_t)bh * nch * 64 + J;
    int c = 0;
    if (J < nbk)
        for (int ch0 = 0; ch0 < nch; ch0 += 32) {
            int x[32];
#pragma unroll
            for (int i = 0; i < 32; ++i) x[i] = ch0 + i < nch ? cc[(size_t)(ch0 + i) * 64] : 0;
#pragma unroll
            for (int i = 0; i < 32; ++i) c += x[i];
        }
    // exclusive prefix sums over the key blocks: slots and tiles
    const int tl = (c + 255) >> 8;
    int s_incl = c, t_incl = tl;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int xs = __shfl_up(s_incl, o), xt = __shfl_up(t_incl, o);
        if (J >= o) { s_incl += xs; t_incl += xt; }
    }
    const int s0 = s_incl - c, t0 = t_incl - tl;
    const int used = __shfl(t_incl, 63);
    if (J < nbk) {
        int run = s0;
        int32_t *cb = cbase + (size_t)bh * nch * 64 + J;
        for (int ch0 = 0; ch0 < nch; ch0 += 32) {
            int x[32];
#pragma unroll
            for (int i = 0; i < 32; ++i) x[i] = ch0 + i < nch ? cc[(size_t)(ch0 + i) * 64] : 0;
#pragma unroll
            for (int i = 0; i < 32; ++i) {
                if (ch0 + i < nch) cb[(size_t)(ch0 + i) * 64] = run;
                run += x[i];
            }
        }
        for (int i = 0; i < tl; ++i)
            if (t0 + i < mt)
                desc[(size_t)bh * mt + t0 + i] = make_uint4((uint32_t)bh, (uint32_t)J, (uint32_t)(s0 + i * 256), (uint32_t)min(256, c - i * 256));
    }
    for (int i = used + J; i < mt; i += 64) desc[(size_t)bh * mt + i] = make_uint4((uint32_t)bh, 0u, 0u, 0u);
}

// grid (nch, BH), 1024 threads: gidx[bh * slots + slot] = n and slot_of[(bh * N + n) * kk + r] = slot for every kept
// pair of the chunk; inside a key block the queries stay in ascending order (slot = chunk base + queries of lower
// waves + lower lanes keeping the block), r = rank of the block among the query's kept blocks.
__global__ __launch_bounds__(1024) void topk_group_kernel(const unsigned long long *__restrict__ mask, int N, int nbk, int kk,
                                                          int nch, const int32_t *__restrict__ cbase,
                                                          int32_t *__restrict__ gidx, int32_t *__restrict__ slot_of)
{
    __shared__ unsigned long long wb[16][64];
    __shared__ int wpre[16][64];
    const int chunk = blockIdx.x, bh = blockIdx.y, t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int n = chunk * 1024 + t;
    const size_t slots = (size_t)N * kk;
    unsigned long long m = n < N ? mask[(size_t)bh * N + n] : 0ull;
    chunk_ballots(m, nbk, wb, wv, lane);
    __syncthreads();
    {
        const int J = lane;                             // thread (wv, J): queries of lower waves keeping J
        int c = 0;
        if (J < nbk)
            for (int w = 0; w < wv; ++w) c += __popcll(wb[w][J]);
        wpre[wv][J] = c + (J < nbk ? cbase[((size_t)bh * nch + chunk) * 64 + J] : 0);
    }
    __syncthreads();
    int r = 0;
    while (m != 0ull && r < kk) {
        const int J = __ffsll((long long)m) - 1;
        m &= m - 1ull;
        if (J < nbk) {
            const int slot = wpre[wv][J] + __popcll(wb[wv][J] & ((1ull << lane) - 1ull));
            if (slot >= 0 && (size_t)slot < slots) {
                gidx[(size_t)bh * slots + slot] = n;
                slot_of[((size_t)bh * N + n) * kk + r] = slot;
            }
        }
        ++r;
    }
}

// out[bh, n, :] = sum_r w_r O_r / sum_r w_r over the query's kk partial results (normalised per key block, bf16, with
// log2-domain log-sum-exp lse_r), w_r = 2^(lse_r - max lse): Eq. (2) over the union of the kept blocks.
// 16 lanes per query (8 channels each) and two queries per thread, so that enough independent gathers are in flight
// (the chain mask -> slot -> partial row is three dependent loads); grid ceil(BH * N / 32), 256 threads.
__global__ __launch_bounds__(256) void topk_merge_kernel(const u16 *__restrict__ po, const float *__restrict__ lse,
                                                         const int32_t *__restrict__ slot_of,
                                                         const unsigned long long *__restrict__ mask, int BH, int N, int kk,
                                                         u16 *__restrict__ out, float *__restrict__ o_dbg)
{
    const size_t nq = (size_t)BH * N;
    const size_t q0 = (size_t)blockIdx.x * 32 + (threadIdx.x >> 4);
    const int c8 = (threadIdx.x & 15) * 8;
    const size_t slots = (size_t)N * kk;
    size_t qi[2];
    int cnt[2], sl[2][8];
    float l[2][8], mx[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        qi[u] = q0 + 16 * u;
        cnt[u] = qi[u] < nq ? min(kk, (int)__popcll(mask[qi[u]])) : 0;     // only the ranks the regrouping pass filled in
    }
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 8; ++r) sl[u][r] = r < cnt[u] ? slot_of[qi[u] * kk + r] : 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const size_t bh = qi[u] < nq ? qi[u] / N : 0;
        mx[u] = -INFINITY;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            l[u][r] = r < cnt[u] ? lse[bh * slots + sl[u][r]] : -INFINITY;
            mx[u] = fmaxf(mx[u], l[u][r]);
        }
    }
    uint4 x[2][8];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const size_t bh = qi[u] < nq ? qi[u] / N : 0;
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (r < cnt[u]) x[u][r] = *reinterpret_cast<const uint4 *>(po + (bh * slots + sl[u][r]) * D + c8);
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        if (qi[u] >= nq) continue;
        float acc[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] = 0.f;
        float den = 0.f;
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (r < cnt[u]) {
                const float wgt = __builtin_amdgcn_exp2f(l[u][r] - mx[u]);
                const uint32_t w4[4] = {x[u][r].x, x[u][r].y, x[u][r].z, x[u][r].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    acc[2 * j] = fmaf(wgt, __uint_as_float(w4[j] << 16), acc[2 * j]);
                    acc[2 * j + 1] = fmaf(wgt, __uint_as_float(w4[j] & 0xffff0000u), acc[2 * j + 1]);
                }
                den += wgt;
            }
        }
        const float inv = den > 0.f ? 1.f / den : 0.f;
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[j] *= inv;
        typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
        typedef float f32x2_t __attribute__((ext_vector_type(2)));
        uint4 pk;
        pk.x = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){acc[0], acc[1]}, bf16x2_t));
        pk.y = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){acc[2], acc[3]}, bf16x2_t));
        pk.z = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){acc[4], acc[5]}, bf16x2_t));
        pk.w = __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){acc[6], acc[7]}, bf16x2_t));
        *reinterpret_cast<uint4 *>(out + qi[u] * D + c8) = pk;
        if (o_dbg) {
            *reinterpret_cast<float4 *>(o_dbg + qi[u] * D + c8) = make_float4(acc[0], acc[1], acc[2], acc[3]);
            *reinterpret_cast<float4 *>(o_dbg + qi[u] * D + c8 + 4) = make_float4(acc[4], acc[5], acc[6], acc[7]);
        }
    }
}

// query tiles per sample-head: every key block can leave one partly filled tile
int topk_tiles_per_head(int N, int kk, int nbk) { return (int)(((long long)N * kk + 255) / 256) + nbk; }
int topk_max_tiles(int BH, int N, int kk, int nbk) { return BH * topk_tiles_per_head(N, kk, nbk); }

hipError_t launch_topk_group(const unsigned long long *mask, int BH, int N, int nbk, int kk, int32_t *ccnt,
                             int32_t *cbase, uint4 *desc, int32_t *gidx, int32_t *slot_of, hipStream_t st)
{
    const int nch = (N + 1023) / 1024;
    launch_kernel(topk_count_kernel, dim3(nch, BH), dim3(1024), 0, st, mask, N, nbk, nch, ccnt);
    launch_kernel(topk_plan_kernel, dim3(BH), dim3(64), 0, st, ccnt, nbk, nch, cbase, desc, topk_tiles_per_head(N, kk, nbk));
    launch_kernel(topk_group_kernel, dim3(nch, BH), dim3(1024), 0, st, mask, N, nbk, kk, nch, cbase, gidx, slot_of);
    return take_launch_status();
}

hipError_t launch_topk_merge(const u16 *po, const float *lse, const int32_t *slot_of, const unsigned long long *mask,
                             int BH, int N, int kk, u16 *out, float *o_dbg, hipStream_t st)
{
    const size_t nq = (size_t)BH * N;
    launch_kernel(topk_merge_kernel, dim3((unsigned)((nq + 31) / 32)), dim3(256), 0, st, po, lse, slot_of, mask, BH, N, kk, out, o_dbg);
    return take_launch_status();
}

}  // namespace salad
