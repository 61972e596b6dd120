// Block-sparse softmax attention (Eq. (2)) with the fused linear apply / scale / sum epilogue, fp32.  gfx950 only.
//
// fp32 calls are small (reference and debugging runs), so the grid is what has to be found: one workgroup = 4 waves =
// 16 query positions of one (batch, head), and the row's kept keys are dealt to the 4 waves in units of 32 keys.
// Every wave runs its own online softmax over its units; the four partial results meet in LDS at the end.
//
// Both products run on v_mfma_f32_16x16x4_f32 (fp32 operands, fp32 accumulation), transposed so that lane i + 16 g
// belongs to query i:
//   S^T = K Q^T    A = K: row = key i of a 16-key tile, k = g; B = Q^T: column = query i, k = g.  The order of a
//                  contraction is free, so step 4 x + y takes channels 16 x + 4 g + y and operands are 16-byte pieces of a
//                  row.  K rows pass through a wave-private LDS tile: read straight into operand order, neighbouring
//                  lanes would sit in 16 different rows and every load would cost 64 line lookups instead of 8.
//   O^T += V^T P^T the accumulators of S^T hold keys 4 g + r of the tile, r = 0..3; step r takes exactly those keys,
//                  so they are the B operand as they stand.  A row i of tile dt is channel i d/16 + dt: a lane's
//                  operands for all tiles are d/16 consecutive floats of one V row, straight from memory.
// Bound by the latency of a unit's loads and softmax on the smallest grids, by the fp32 matrix rate (64 steps of 32 cycles per
// wave and unit at d = 64) with two or three waves per SIMD beyond that.  One wave per query with the dot products on the
// vector unit took 48.0 us at B = 1, H = 2, N = 1024, d = 64, 4 of 16 blocks kept and 481 us at H = 4, N = 2080, 16 of 33 kept;
// this takes 8.5 and 44.9 us (50.3 us with K read straight into operand order).
#include <algorithm>

#include "salad_internal.h"

namespace salad {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// DIV: N * T does not fit 32 bits and p / T is a real division instead of a multiply-high with a.t_magic
template <int D, bool DIV>
__global__ __launch_bounds__(256, 2) void sparse_attn_f32_kernel(AttnArgs a, int ntiles, int total, int per_xcd)
{
    constexpr int NX = D / 16;              // 16-byte pieces of a lane's K or Q channels; channel tiles of O^T
    constexpr int KT = 2;                   // 16-key tiles per unit
    constexpr int PITCH = D + 4;            // 4 banks between rows: 16 rows x 64 bytes of an operand read spread over all banks
    constexpr int LPR = D / 4, RPI = 64 / LPR, NK = 32 / RPI;   // lanes per K row, rows per load, loads per unit
    // wave-private: the unit's K rows; after the last unit rows 0..15 take the wave's partial result
    __shared__ __attribute__((aligned(16))) float stage[4][32][PITCH];
    __shared__ float msh[4][16], lsh[4][16];
    // consecutive workgroups go to the 8 XCDs in turn: give each XCD a contiguous range of a slice's (head, tile)
    const long long l64 = (long long)blockIdx.y * (8ll * per_xcd) + (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (l64 >= total) return;
    const int L = (int)l64;
    const int bh = L / ntiles, tile = L - bh * ntiles, h = bh % a.H;
    const int N = a.N, T = a.T, HW = a.HW;
    const int kind = T > 1 ? (int)((a.kind_mask >> h) & 1ull) : 0;
    // stored row of a position without a branch: a spatial head is the formula with location 0 and stride 1
    const unsigned magic = kind ? a.t_magic : 0u;
    const int stride = kind ? HW : 1;
    auto row_of = [&](int p) __attribute__((always_inline)) -> int {
        p = p < N ? p : N - 1;
        const int loc = DIV ? (kind ? p / T : 0) : (int)__umulhi((unsigned)p, magic);
        return (p - loc * T) * stride + loc;
    };
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i = lane & 15, g = lane >> 4;
    const float *qb = reinterpret_cast<const float *>(a.q) + (size_t)bh * N * D;
    const float *kb = reinterpret_cast<const float *>(a.k) + (size_t)bh * N * D + (lane % LPR) * 4;
    const float *vb = reinterpret_cast<const float *>(a.v) + (size_t)bh * N * D + i * (D / 16);
    const int qpos = tile * 16 + i;
    const int qrow = row_of(qpos);

    f32x4 qv[NX], kv[NK], vv[KT][4][D / 64];
#pragma unroll
    for (int x = 0; x < NX; ++x) qv[x] = *reinterpret_cast<const f32x4 *>(qb + (size_t)qrow * D + 16 * x + 4 * g);
    auto load_k = [&](int key0) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < NK; ++t) kv[t] = *reinterpret_cast<const f32x4 *>(kb + (size_t)row_of(key0 + t * RPI + lane / LPR) * D);
    };
    auto load_v = [&](int key0) __attribute__((always_inline)) {
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float *row = vb + (size_t)row_of(key0 + kt * 16 + 4 * g + r) * D;
#pragma unroll
                for (int x = 0; x < D / 64; ++x) vv[kt][r][x] = *reinterpret_cast<const f32x4 *>(row + 4 * x);
            }
    };

    f32x4 o[NX];
#pragma unroll
    for (int dt = 0; dt < NX; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m = -1e30f, l = 0.f;
    const int row = h * a.nb + tile / 4;
    const int e0 = a.row_ptr[row], units = 2 * (a.row_ptr[row + 1] - e0);
    auto first_key = [&](int u) __attribute__((always_inline)) -> int { return a.col_idx[e0 + (u >> 1)] * 64 + (u & 1) * 32; };
    int u = wave, key0 = 0;
    if (u < units) {
        key0 = first_key(u);
        load_k(key0);
    }
    // Without a reduce of the gate ahead of this launch every wave adds up the sample's partial sums itself, in the order of that
    // reduce, while its first keys are on their way: a launch less, layer call at H = 2, N = 1024 16.1 -> 13.6 us, H = 4, N = 2080 56.1 -> 53.0.
    const int smp = bh / a.H;
    float s_b = 0.f;
    if (a.gate_here) {
        if (a.gate_nparts) {
            static_assert(GATE_MAX_PARTS <= 512, "8 partial sums a lane");
            float t[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int x = j * 64 + lane;
                t[j] = x < a.gate_nparts ? a.gate_partial[(size_t)smp * a.gate_nparts + x] : 0.f;
            }
            s_b = ((t[0] + t[4]) + (t[2] + t[6])) + ((t[1] + t[5]) + (t[3] + t[7]));
#pragma unroll
            for (int x = 32; x > 0; x >>= 1) s_b += __shfl_xor(s_b, x);
            s_b /= (float)N;
        } else {
            s_b = a.s_dev[smp];
        }
        if (a.s_out && L == smp * a.H * ntiles && threadIdx.x == 0) a.s_out[smp] = s_b;
    }
    while (u < units) {
        load_v(key0);
#pragma unroll
        for (int t = 0; t < NK; ++t) *reinterpret_cast<f32x4 *>(&stage[wave][t * RPI + lane / LPR][(lane % LPR) * 4]) = kv[t];
        const int here = key0;
        u += 4;
        if (u < units) {                    // the next unit's keys travel under this unit's products
            key0 = first_key(u);
            load_k(key0);
        }
        __builtin_amdgcn_wave_barrier();    // the wave's own LDS operations execute in order
        f32x4 s[KT];
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) s[kt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int x = 0; x < NX; ++x) {
            f32x4 kf[KT];
#pragma unroll
            for (int kt = 0; kt < KT; ++kt) kf[kt] = *reinterpret_cast<const f32x4 *>(&stage[wave][kt * 16 + i][16 * x + 4 * g]);
#pragma unroll
            for (int y = 0; y < 4; ++y)
#pragma unroll
                for (int kt = 0; kt < KT; ++kt) s[kt] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[kt][y], qv[x][y], s[kt], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();
        float mb = -INFINITY;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[kt][r] = here + kt * 16 + 4 * g + r < N ? s[kt][r] * a.scale : -INFINITY;
                mb = fmaxf(mb, s[kt][r]);
            }
        mb = fmaxf(mb, __shfl_xor(mb, 16));
        mb = fmaxf(mb, __shfl_xor(mb, 32));
        const float mn = fmaxf(m, mb), alpha = __expf(m - mn);
        m = mn;
        l *= alpha;
#pragma unroll
        for (int dt = 0; dt < NX; ++dt) o[dt] *= alpha;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[kt][r] = here + kt * 16 + 4 * g + r < N ? __expf(s[kt][r] - mn) : 0.f;
                l += s[kt][r];
            }
        if (here + 32 > N) {                // keys past the end are copies of the last row: weight 0 alone would make NaN of an infinity
#pragma unroll
            for (int kt = 0; kt < KT; ++kt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (here + kt * 16 + 4 * g + r >= N)
#pragma unroll
                        for (int x = 0; x < D / 64; ++x) vv[kt][r][x] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int r = 0; r < 4; ++r)
#pragma unroll
                for (int dt = 0; dt < NX; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(vv[kt][r][dt / 4][dt % 4], s[kt][r], o[dt], 0, 0, 0);
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);

    // ---- the wave's partial result to LDS: tile dt, register r of lane (i, g) is channel (4 g + r) d/16 + dt of query i
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int x = 0; x < D / 64; ++x)
            *reinterpret_cast<f32x4 *>(&stage[wave][i][(4 * g + r) * (D / 16) + 4 * x]) = f32x4{o[4 * x][r], o[4 * x + 1][r], o[4 * x + 2][r], o[4 * x + 3][r]};
    if (g == 0) {
        msh[wave][i] = m;
        lsh[wave][i] = l;
    }
    // ---- linear branch: wave w owns output channels [w d/4, (w + 1) d/4); num^T = Hs^T relu(Q)^T in the same layout
    constexpr int CT = D / 64;
    const bool lin = a.use_linear && !(a.drop && a.drop[smp]);   // pruned sample (Sec. 4.3): out = O_s
    f32x4 num[CT];
    float inv_den = 0.f, cf = 0.f;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) num[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (lin) {
        const float *Hh = a.Hs + (size_t)bh * D * D + (size_t)(g * 4) * D + wave * (D / 4) + i;
        const float *Zh = a.Z + (size_t)bh * D + g * 4;
        float den = 0.f;
#pragma unroll
        for (int x = 0; x < NX; ++x)
#pragma unroll
            for (int y = 0; y < 4; ++y) {
                const float f = fmaxf(qv[x][y], 0.f);
                den = fmaf(f, Zh[16 * x + y], den);
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    num[ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(Hh[(size_t)(16 * x + y) * D + ct * 16], f, num[ct], 0, 0, 0);
            }
        den += __shfl_xor(den, 16);
        den += __shfl_xor(den, 32);
        inv_den = 1.f / (den + a.eps);
        cf = a.gate_here ? a.lambda * (a.head_scale ? a.head_scale[h] : 1.f) * s_b : a.coef[bh];
    }
    __syncthreads();
    // ---- merge, in wave order
    float mx = msh[0][i];
#pragma unroll
    for (int w = 1; w < 4; ++w) mx = fmaxf(mx, msh[w][i]);
    float wt[4], lt = 0.f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        wt[w] = __expf(msh[w][i] - mx);
        lt = fmaf(lsh[w][i], wt[w], lt);
    }
    const float inv_l = lt > 0.f ? 1.f / lt : 0.f;
    if (qpos >= N) return;
    const size_t ob = ((size_t)bh * N + qrow) * D;
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        const int c = wave * (D / 4) + ct * 16 + 4 * g;
        f32x4 os = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const f32x4 p = *reinterpret_cast<const f32x4 *>(&stage[w][i][c]);
#pragma unroll
            for (int r = 0; r < 4; ++r) os[r] = fmaf(wt[w], p[r], os[r]);
        }
        f32x4 ol, out;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            os[r] *= inv_l;
            ol[r] = num[ct][r] * inv_den;
            out[r] = lin ? fmaf(cf, ol[r], os[r]) : os[r];
        }
        *reinterpret_cast<f32x4 *>(reinterpret_cast<float *>(a.out) + ob + c) = out;
        if (a.o_sparse_dbg) *reinterpret_cast<f32x4 *>(a.o_sparse_dbg + ob + c) = os;
        if (a.o_linear_dbg && lin) *reinterpret_cast<f32x4 *>(a.o_linear_dbg + ob + c) = ol;
    }
}

hipError_t launch_sparse_attn_f32(const AttnArgs &a, hipStream_t st)
{
    const int ntiles = (a.N + 15) / 16;
    const long long total = (long long)a.B * a.H * ntiles;
    if (total > 0x7fffffffll) return hipErrorInvalidValue;
    // one grid dimension takes fewer than 2^32 threads: more tiles lie in slices of 2^23 along y
    const int per_xcd = (int)((std::min(total, 1ll << 23) + 7) / 8), slices = (int)((total + 8ll * per_xcd - 1) / (8ll * per_xcd));
    auto go = [&](auto kern) { launch_kernel(kern, dim3(per_xcd * 8, slices), dim3(256), 0, st, a, ntiles, (int)total, per_xcd); };
    const bool div = a.kind_mask != 0 && a.T > 1 && a.t_magic == 0;
    if (a.D == 128) div ? go(sparse_attn_f32_kernel<128, true>) : go(sparse_attn_f32_kernel<128, false>);
    else div ? go(sparse_attn_f32_kernel<64, true>) : go(sparse_attn_f32_kernel<64, false>);
    return take_launch_status();
}

}  // namespace salad
