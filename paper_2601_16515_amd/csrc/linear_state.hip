// Linear-attention state, Eq. (3):  Hs = sum_j relu(K_j)^T V_j  (d x d),  Z = sum_j relu(K_j).
//
// bf16 kernel.  HBM-bound: K and V are each read once (4*N*d bytes per head) for 2*N*d*d flops,
// 64 flop/byte at d = 128 - below the MFMA ridge but above what plain FMAs sustain, so the outer
// products run on bf16 MFMA with fp32 accumulators.  The contraction runs over tokens, which is
// the row index of the stored [N, d] tensors, so both operands must be transposed on the way:
// each thread loads a (TPT tokens x 8 features) patch with 16-byte loads, transposes it in
// registers with byte permutes and writes token-contiguous vectors to LDS; MFMA operands are then
// single 16-byte LDS reads.  The LDS tile is [feature][64 tokens + 8 pad] with the 8-token group
// index XOR-ed by (feature / 16) so that both the 8-byte transposed writes and the 16-byte operand
// reads spread over all banks.
//
// One workgroup (4 waves) owns one d x d accumulator: wave w holds the (w/2, w%2) quadrant.
// The token range of a head is cut into chunks, one workgroup each; the fp32 partial states go to
// the workspace and are added in chunk order by the finalize kernel (no float atomics, so results
// are reproducible run to run).
#include "gate_part.h"
#include "linear_ride.h"

#include <cmath>

namespace salad {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

int state_tiles_per_chunk(int BH, int N, int D, int target_wgs)
{
    int tiles = (N + 63) / 64;
    int want = target_wgs / (BH > 0 ? BH : 1);
    if (want < 1) want = 1;
    if (want > tiles) want = tiles;
    const int spread = (tiles + want - 1) / want;
    if (target_wgs != STATE_WGS) return spread;
    // A chunk's partial state, written and read again, is as many bytes as four tiles of K and V (d = 64: two), all of a head's are added
    // up in the next launch, and the gate's workgroups ride in this one, so short chunks cost more than they save: with t us per tile
    // and r per partial state the time tiles t + BH chunks r is least at sqrt(BH tiles r / t) tiles per chunk.  r / t = 1/32, d = 64 1/48, by
    // layer calls of 98 shapes each (640 to 32760 tokens, 2 to 80 heads, 2 kept blocks): 0.967 and 0.983 of the time with the spread
    // alone in the mean, slower than it by up to 4 and 2.5 %; 1/32 at d = 64 0.983, slower by up to 4 %, 1/80 at d = 128 0.977.  From BH tiles =
    // 2048 (1365) on the spread decides.  State and reduce alone, without the gate, like chunks to be shorter: 1/80 for both.
    // N = 1280, 12 heads 27.0 -> 24.1 us, N = 1950, 16 heads 29.9 -> 26.4, N = 6000, 5 heads 29.8 -> 26.0; d = 64: 18.8 -> 16.6, 20.9 -> 18.8.
    const int least = (int)std::ceil(std::sqrt((double)BH * tiles / (D == 128 ? 32 : 48)));
    return spread > least ? spread : least < tiles ? least : tiles;
}

int state_num_chunks(int BH, int N, int D, int target_wgs)
{
    int tiles = (N + 63) / 64;
    int tpc = state_tiles_per_chunk(BH, N, D, target_wgs);
    return (tiles + tpc - 1) / tpc;
}

constexpr int XT_PITCH = 72;   // 64 tokens + 8 pad, in bf16 elements (144 bytes)

// element offset of (row = feature, tok) in a transposed tile
__device__ inline int xt_off(int row, int tok)
{
    return row * XT_PITCH + ((((tok >> 3) ^ (row >> 4)) & 7) << 3) + (tok & 7);
}

__device__ inline uint32_t relu_bf16x2(uint32_t x)
{
    s16x2 v = __builtin_bit_cast(s16x2, x);
    s16x2 z = {0, 0};
    v = __builtin_elementwise_max(v, z);   // negative bf16 (sign bit set) is a negative int16
    return __builtin_bit_cast(uint32_t, v);
}

// ROPE: the rotary linear branch (Sec. 4.1): after the ReLU and the Z sums (which stay unrotated), channel pair
// (2p, 2p+1) of token n is rotated by the angle whose cosine and sine sit, as two fp16 values in one word, at
// rope_tab[n * D/2 + p], before it enters the outer products, so the state is sum_j (R_j relu(K_j))^T V_j.
template <int D, bool ROPE>
__device__ inline __attribute__((always_inline)) void state_chunk(const u16 *__restrict__ k, const u16 *__restrict__ v, int N, int tiles_per_chunk,
                                                                  int P, float *__restrict__ partial, const uint32_t *__restrict__ rope_tab,
                                                                  int bh, int chunk)
{
    constexpr int CH = D / 8;          // 16-byte chunks per row
    constexpr int TPT = D / 32;        // tokens per thread per tile (4 for d=128, 2 for d=64)
    constexpr int QT = D / 64;         // 32x32 tiles per side of a wave's quadrant
    __shared__ __attribute__((aligned(16))) u16 KT[D * XT_PITCH];
    __shared__ __attribute__((aligned(16))) u16 VT[D * XT_PITCH];
    __shared__ float zred[4][D];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, hh = lane >> 5;
    const int fg = tid % CH, tq = tid / CH;   // feature group (8 features), token group (TPT tokens)
    const u16 *kb = k + (size_t)bh * N * D;
    const u16 *vb = v + (size_t)bh * N * D;
    const int tile0 = chunk * tiles_per_chunk;
    int tile1 = tile0 + tiles_per_chunk;
    const int tiles = (N + 63) / 64;
    if (tile1 > tiles) tile1 = tiles;

    f32x16 acc[QT][QT];
#pragma unroll
    for (int i = 0; i < QT; ++i)
#pragma unroll
        for (int j = 0; j < QT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    float zacc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) zacc[e] = 0.f;

    // two tiles of global loads are kept in flight per thread (register buffers 0 and 1)
    uint4 kreg[2][TPT], vreg[2][TPT];
    uint4 creg[2][ROPE ? TPT : 1];     // (cos, sin) of the patch's 4 channel pairs
    auto gload = [&](uint4 (&kr)[TPT], uint4 (&vr)[TPT], uint4 *cr, int tile) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < TPT; ++i) {
            int n = tile * 64 + tq * TPT + i;
            if (n < N) {
                kr[i] = *reinterpret_cast<const uint4 *>(kb + (size_t)n * D + fg * 8);
                vr[i] = *reinterpret_cast<const uint4 *>(vb + (size_t)n * D + fg * 8);
                if (ROPE) cr[i] = *reinterpret_cast<const uint4 *>(rope_tab + (size_t)n * (D / 2) + fg * 4);
            } else {
                kr[i] = make_uint4(0, 0, 0, 0);
                vr[i] = make_uint4(0, 0, 0, 0);
                if (ROPE) cr[i] = make_uint4(0x3c00u, 0x3c00u, 0x3c00u, 0x3c00u);   // cos = 1, sin = 0
            }
        }
    };
    // transposed store of a (TPT x 8) patch: for feature f, TPT consecutive tokens
    auto tstore = [&](u16 *dst, const uint4 (&r)[TPT]) __attribute__((always_inline)) {
        uint32_t w[TPT][4];
#pragma unroll
        for (int i = 0; i < TPT; ++i) { w[i][0] = r[i].x; w[i][1] = r[i].y; w[i][2] = r[i].z; w[i][3] = r[i].w; }
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            const uint32_t sel = (f & 1) ? 0x07060302u : 0x05040100u;
            int off = xt_off(fg * 8 + f, tq * TPT);
            if (TPT == 4) {
                uint2 o;
                o.x = __builtin_amdgcn_perm(w[1][f >> 1], w[0][f >> 1], sel);
                o.y = __builtin_amdgcn_perm(w[3][f >> 1], w[2][f >> 1], sel);
                *reinterpret_cast<uint2 *>(dst + off) = o;
            } else {
                uint32_t o = __builtin_amdgcn_perm(w[1][f >> 1], w[0][f >> 1], sel);
                *reinterpret_cast<uint32_t *>(dst + off) = o;
            }
        }
    };

    const int wa = wave >> 1, wc = wave & 1;
    auto step = [&](uint4 (&kr)[TPT], uint4 (&vr)[TPT], uint4 *cr, int tile) __attribute__((always_inline)) {
        // ReLU on K, running sums for Z
#pragma unroll
        for (int i = 0; i < TPT; ++i) {
            kr[i].x = relu_bf16x2(kr[i].x); kr[i].y = relu_bf16x2(kr[i].y);
            kr[i].z = relu_bf16x2(kr[i].z); kr[i].w = relu_bf16x2(kr[i].w);
            uint32_t w4[4] = {kr[i].x, kr[i].y, kr[i].z, kr[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                zacc[2 * j] += __uint_as_float(w4[j] << 16);
                zacc[2 * j + 1] += __uint_as_float(w4[j] & 0xffff0000u);
            }
            if (ROPE) {
                const uint32_t cw[4] = {cr[i].x, cr[i].y, cr[i].z, cr[i].w};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float x = __uint_as_float(w4[j] << 16), y = __uint_as_float(w4[j] & 0xffff0000u);
                    const f16x2 hcs = __builtin_bit_cast(f16x2, cw[j]);
                    const float cc = (float)hcs[0], ss = (float)hcs[1];
                    f32x2 r = {x * cc - y * ss, x * ss + y * cc};
                    w4[j] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2));
                }
                kr[i] = make_uint4(w4[0], w4[1], w4[2], w4[3]);
            }
        }
        tstore(KT, kr);
        tstore(VT, vr);
        __syncthreads();
        if (tile + 2 < tile1) gload(kr, vr, cr, tile + 2);
#pragma unroll
        for (int s = 0; s < 4; ++s) {   // 16 tokens per MFMA
            bf16x8 af[QT], bfr[QT];
#pragma unroll
            for (int i = 0; i < QT; ++i) {
                int ra = (wa * QT + i) * 32 + l32;
                int rc = (wc * QT + i) * 32 + l32;
                af[i] = *reinterpret_cast<const bf16x8 *>(KT + xt_off(ra, s * 16 + hh * 8));
                bfr[i] = *reinterpret_cast<const bf16x8 *>(VT + xt_off(rc, s * 16 + hh * 8));
            }
#pragma unroll
            for (int i = 0; i < QT; ++i)
#pragma unroll
                for (int j = 0; j < QT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[i], bfr[j], acc[i][j], 0, 0, 0);
        }
        __syncthreads();
    };
    if (tile0 < tile1) gload(kreg[0], vreg[0], creg[0], tile0);
    if (tile0 + 1 < tile1) gload(kreg[1], vreg[1], creg[1], tile0 + 1);
    for (int tile = tile0; tile < tile1; tile += 2) {
        step(kreg[0], vreg[0], creg[0], tile);
        if (tile + 1 < tile1) step(kreg[1], vreg[1], creg[1], tile + 1);
    }

    // partial Hs: accumulator register r of lane (l32, hh) is row a = 8*(r/4) + 4*hh + r%4, col c = l32
    const int per = D * D + D;
    float *out = partial + ((size_t)bh * P + chunk) * per;
#pragma unroll
    for (int i = 0; i < QT; ++i)
#pragma unroll
        for (int j = 0; j < QT; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                int a = (wa * QT + i) * 32 + 8 * (r >> 2) + 4 * hh + (r & 3);
                int c = (wc * QT + j) * 32 + l32;
                out[a * D + c] = acc[i][j][r];
            }
    // partial Z: threads with the same fg hold sums over different tokens.  Within a wave the lanes
    // with equal fg are CH apart; across waves go through LDS in wave order.
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        float zz = zacc[e];
        for (int o = CH; o < 64; o <<= 1) zz += __shfl_xor(zz, o);
        zacc[e] = zz;
    }
    if (lane < CH) {
#pragma unroll
        for (int e = 0; e < 8; ++e) zred[wave][lane * 8 + e] = zacc[e];
    }
    __syncthreads();
    if (tid < D) out[D * D + tid] = (zred[0][tid] + zred[1][tid]) + (zred[2][tid] + zred[3][tid]);
}

template <int D, bool ROPE = false>
__global__ __launch_bounds__(256, 2) void state_partial_kernel(const u16 *__restrict__ k,
                                                               const u16 *__restrict__ v, int N,
                                                               int tiles_per_chunk, int P,
                                                               float *__restrict__ partial,
                                                               const int32_t *__restrict__ drop, int H,
                                                               const uint32_t *__restrict__ rope_tab = nullptr)
{
    // ROPE: the sample-head index runs fastest over the grid, so that the workgroups that read the same rows of the
    // angle tables (same token chunk, different heads) run at the same time and the tables come from HBM once
    const int bh = ROPE ? blockIdx.x : blockIdx.y, chunk = ROPE ? blockIdx.y : blockIdx.x;
    if (drop && drop[bh / H]) return;                  // pruned sample (Sec. 4.3): K, V are not read
    state_chunk<D, ROPE>(k, v, N, tiles_per_chunk, P, partial, rope_tab, bh, chunk);
}

// State chunks and gate partial sums in one launch: both are passes over inputs that nothing before them writes, and alone each
// has a start and an end in which the memory system idles (the state leaves half a CU's wave slots empty, too).  The gate's
// workgroups come last in the grid and fill in behind the state's.  Layer call, two launches -> one: N = 1950, H = 12 42.0 -> 37.5 us;
// N = 12480 292.1 -> 285.9; N = 32760 708.7 -> 703.6 (rotary 735.8 -> 729.3); N = 75600, H = 40 11438 -> 11396; no size where it
// lost.  The same bits as the two launches.
template <int D, int NCH, int TOK, bool ROPE>
__global__ __launch_bounds__(256, 2) void state_gate_kernel(const u16 *__restrict__ k, const u16 *__restrict__ v, int N, int tiles_per_chunk, int P,
                                                            float *__restrict__ partial, int BH, GateArgs g,
                                                            const uint32_t *__restrict__ rope_tab)
{
    __shared__ float wave_sum[4];
    const int i = blockIdx.x, state_blocks = BH * P;
    // ROPE: heads fastest, see state_partial_kernel
    if (i < state_blocks) state_chunk<D, ROPE>(k, v, N, tiles_per_chunk, P, partial, rope_tab, ROPE ? i % BH : i / P, ROPE ? i / BH : i % P);
    else gate_part<true, NCH, TOK>(g.x_t, g.w, g.bias, N, g.D, g.partial, g.nparts, (i - state_blocks) / g.nparts, (i - state_blocks) % g.nparts,
                                   threadIdx.x >> 6, wave_sum);
}

// wider rows keep the gate weights in LDS (gate_partial_wide_kernel) and stay a launch of their own
bool state_gate_fits(const GateArgs &g, int B, int BH, int P)
{
    return g.D <= 512 * GATE_MAX_CHUNKS && grid_dim_fits((long long)BH * P + (long long)g.nparts * B, 256);
}

hipError_t launch_state_gate_bf16(const u16 *k, const u16 *v, int BH, int N, int D, float *partial, int target_wgs, const GateArgs &g, int B,
                                  hipStream_t st, const uint32_t *rope_tab)
{
    if (rope_tab && D != 128) return hipErrorInvalidValue;
    const int tpc = state_tiles_per_chunk(BH, N, D, target_wgs), P = state_num_chunks(BH, N, D, target_wgs);
    const int nch = (g.D / 8 + 63) / 64;
    const dim3 grid(BH * P + g.nparts * B), block(256);
    auto go = [&](auto kern) { launch_kernel(kern, grid, block, 0, st, k, v, N, tpc, P, partial, BH, g, rope_tab); };
    auto by_width = [&](auto dc, auto rc) {
        constexpr int DD = decltype(dc)::value;
        constexpr bool R = decltype(rc)::value;
        if (nch <= 1) go(state_gate_kernel<DD, 1, 4, R>);
        else if (nch <= 2) go(state_gate_kernel<DD, 2, 4, R>);
        else if (nch <= 3) go(state_gate_kernel<DD, 3, 2, R>);
        else if (nch <= 5) go(state_gate_kernel<DD, 5, 2, R>);
        else go(state_gate_kernel<DD, GATE_MAX_CHUNKS, 1, R>);
    };
    if (rope_tab) by_width(std::integral_constant<int, 128>{}, std::true_type{});
    else if (D == 128) by_width(std::integral_constant<int, 128>{}, std::false_type{});
    else by_width(std::integral_constant<int, 64>{}, std::false_type{});
    return take_launch_status();
}

hipError_t launch_state_partial_bf16(const u16 *k, const u16 *v, int BH, int N, int D,
                                     float *partial, const int32_t *drop, int H, int target_wgs, hipStream_t st,
                                     const uint32_t *rope_tab)
{
    int tpc = state_tiles_per_chunk(BH, N, D, target_wgs);
    int P = state_num_chunks(BH, N, D, target_wgs);
    dim3 grid(P, BH), block(256);
    if (rope_tab) {
        if (D != 128) return hipErrorInvalidValue;
        launch_kernel((state_partial_kernel<128, true>), dim3(BH, P), block, 0, st, k, v, N, tpc, P, partial, drop, H, rope_tab);
        return take_launch_status();
    }
    if (D == 128)
        launch_kernel((state_partial_kernel<128, false>), grid, block, 0, st, k, v, N, tpc, P, partial, drop, H, nullptr);
    else
        launch_kernel((state_partial_kernel<64, false>), grid, block, 0, st, k, v, N, tpc, P, partial, drop, H, nullptr);
    return take_launch_status();
}

// Short sequences (linear_ride.h), where the slices do not ride with the attention because each stage is being timed.
template <int D, bool ROPE>
__global__ __launch_bounds__(512) void state_direct_kernel(const u16 *__restrict__ k, const u16 *__restrict__ v, int N, int BH, int H, const int32_t *__restrict__ drop,
                                                           const uint32_t *__restrict__ rope_tab, u16 *__restrict__ hfrag, float *__restrict__ Z)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    __shared__ float small[DIRECT_WAVES][32];
    const int bh = slice_head(BH, slices_per_head(D), blockIdx.x), slice = slice_of(BH, slices_per_head(D), blockIdx.x);
    if (drop && drop[bh / H]) return;                  // pruned sample (Sec. 4.3): K, V are not read
    state_slice<D, ROPE>(k, v, N, rope_tab, hfrag, Z, bh, slice, smem, small);
}

hipError_t launch_state_direct(const u16 *k, const u16 *v, int B, int H, int N, int D, const int32_t *drop, const uint32_t *rope_tab, u16 *hfrag, float *Z,
                               hipStream_t st)
{
    auto go = [&](auto dc, auto rc) -> hipError_t {
        constexpr int DD = decltype(dc)::value;
        auto kern = state_direct_kernel<DD, decltype(rc)::value>;
        static bool attr_done[16] = {};
        if (hipError_t e = dyn_lds_attr_once(reinterpret_cast<const void *>(kern), direct_lds(DD), attr_done); e != hipSuccess) return e;
        launch_kernel(kern, dim3(B * H * slices_per_head(DD)), dim3(512), (size_t)direct_lds(DD), st, k, v, N, B * H, H, drop, rope_tab, hfrag, Z);
        return take_launch_status();
    };
    if (D == 64) return rope_tab ? hipErrorInvalidValue : go(std::integral_constant<int, 64>{}, std::false_type{});
    return rope_tab ? go(std::integral_constant<int, 128>{}, std::true_type{}) : go(std::integral_constant<int, 128>{}, std::false_type{});
}

// (cos, sin) tables of the rotary linear branch, fp32 [n] each -> one word per angle: fp16 cos | fp16 sin << 16
__global__ __launch_bounds__(256) void rope_pack_kernel(const float *__restrict__ c, const float *__restrict__ s_, size_t n,
                                                        uint32_t *__restrict__ out)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    f16x2 h = {(_Float16)c[i], (_Float16)s_[i]};
    out[i] = __builtin_bit_cast(uint32_t, h);
}

hipError_t launch_rope_pack(const float *rope_cos, const float *rope_sin, size_t n, uint32_t *tab, hipStream_t st)
{
    launch_kernel(rope_pack_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, rope_cos, rope_sin, n, tab);
    return take_launch_status();
}

// ------------------------------------------------------------------------------------------------
// fp32 state for small shapes, on v_mfma_f32_16x16x4_f32 (fp32 operands and accumulation).  A workgroup owns one 16 x 16
// tile of Hs of one head, so that even one head fills 16 (d = 64) or 64 (d = 128) workgroups, and deals the tokens to its 16
// waves in groups of 4 (group j to wave j mod 16): row i of the A operand is channel a0 + i of a token's relu(K), column i
// of B channel c0 + i of its V, the 4 tokens are the contraction.  8 groups of loads are in flight per wave.  The 16
// accumulators are added in wave order through LDS: the same result whatever the launch looks like.  The workgroups of
// the first column also add up Z.
// Bound by the latency of the loads: B = 1, H = 4, N = 2080, d = 64: 8.2 us against 18.5 us with one thread per element
// and token group; H = 2, N = 1024: 5.3 against 7.2 us.
// ------------------------------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ inline __attribute__((always_inline)) void state_f32_tile(const float *__restrict__ k, const float *__restrict__ v, int N, int D,
                                                                     float *__restrict__ Hs, float *__restrict__ Z, int bh, int tile)
{
    __shared__ float part[16][256], zpart[16][16];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
    const int nt = D / 16, a0 = (tile / nt) * 16, c0 = (tile % nt) * 16;
    const float *kb = k + (size_t)bh * N * D + a0 + i;
    const float *vb = v + (size_t)bh * N * D + c0 + i;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    float z = 0.f;
    for (int n0 = w * 4; n0 < N; n0 += 8 * 64) {
        float kk[8], vv[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {                  // tokens past the end: any existing row, weight 0
            const int n = n0 + u * 64 + g;
            const size_t off = (size_t)(n < N ? n : N - 1) * D;
            kk[u] = kb[off];
            vv[u] = vb[off];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const bool live = n0 + u * 64 + g < N;
            kk[u] = live ? fmaxf(kk[u], 0.f) : 0.f;
            z += kk[u];
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(kk[u], live ? vv[u] : 0.f, acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) part[w][(4 * g + r) * 16 + i] = acc[r];   // register r of lane (i, g): row 4 g + r, column i
    z += __shfl_xor(z, 16);
    z += __shfl_xor(z, 32);
    if (g == 0) zpart[w][i] = z;
    __syncthreads();
    const int e = threadIdx.x;
    if (e < 256) {
        float t = part[0][e];
#pragma unroll
        for (int x = 1; x < 16; ++x) t += part[x][e];
        Hs[(size_t)bh * D * D + (size_t)(a0 + e / 16) * D + c0 + e % 16] = t;
    } else if (e < 272 && c0 == 0) {
        float t = zpart[0][e - 256];
#pragma unroll
        for (int x = 1; x < 16; ++x) t += zpart[x][e - 256];
        Z[(size_t)bh * D + a0 + e - 256] = t;
    }
}

__global__ __launch_bounds__(1024) void state_f32_kernel(const float *__restrict__ k, const float *__restrict__ v,
                                                         int N, int D, float *__restrict__ Hs, float *__restrict__ Z,
                                                         const int32_t *__restrict__ drop, int H)
{
    if (drop && drop[blockIdx.y / H]) return;          // pruned sample (Sec. 4.3)
    state_f32_tile(k, v, N, D, Hs, Z, blockIdx.y, blockIdx.x);
}

// fp32 state and gate in one launch: state tiles first, then workgroups of four gate partial sums each.  Layer call at H = 2,
// N = 1024, d = 64: 19.0 -> 16.9 us.  Rows up to 1024 channels: the gate weights of wider ones do not fit the 128 registers
// of a 1024-thread workgroup.
__global__ __launch_bounds__(1024) void state_gate_f32_kernel(const float *__restrict__ k, const float *__restrict__ v, int N, int D,
                                                              float *__restrict__ Hs, float *__restrict__ Z, int BH, GateArgs g)
{
    __shared__ float wave_sum[4][4];
    const int tiles = (D / 16) * (D / 16), i = blockIdx.x;
    if (i < tiles * BH) {
        state_f32_tile(k, v, N, D, Hs, Z, i / tiles, i % tiles);
        return;
    }
    const int per_b = (g.nparts + 3) / 4, x = i - tiles * BH, w = threadIdx.x >> 6;
    gate_part<false, 2, 1>(g.x_t, g.w, g.bias, N, g.D, g.partial, g.nparts, x / per_b, (x % per_b) * 4 + (w >> 2), w & 3, wave_sum[w >> 2]);
}

static long long state_gate_f32_blocks(const GateArgs &g, int B, int BH, int D)
{
    return (long long)(D / 16) * (D / 16) * BH + (g.nparts + 3) / 4 * (long long)B;
}

bool state_gate_f32_fits(const GateArgs &g, int B, int BH, int D)
{
    return g.D <= 1024 && grid_dim_fits(state_gate_f32_blocks(g, B, BH, D), 1024);
}

hipError_t launch_state_gate_f32(const float *k, const float *v, int BH, int N, int D, float *Hs, float *Z, const GateArgs &g, int B,
                                 hipStream_t st)
{
    launch_kernel(state_gate_f32_kernel, dim3((unsigned)state_gate_f32_blocks(g, B, BH, D)), dim3(1024), 0, st, k, v, N, D, Hs, Z, BH, g);
    return take_launch_status();
}

hipError_t launch_state_f32(const float *k, const float *v, int BH, int N, int D, float *Hs, float *Z,
                            const int32_t *drop, int H, hipStream_t st)
{
    dim3 grid((D / 16) * (D / 16), BH), block(1024);
    launch_kernel(state_f32_kernel, grid, block, 0, st, k, v, N, D, Hs, Z, drop, H);
    return take_launch_status();
}

}  // namespace salad
