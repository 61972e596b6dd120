// Block-sparse softmax attention (Eq. (2)) with the fused linear apply / scale / sum epilogue,
// d = 128 (and d = 64 on half-size tiles).  Large tile, deep LDS prefetch, softmax woven into the matrix stream.
//
//   * One workgroup = 8 waves = 256 query positions = 4 CSR rows of one (batch, head); one workgroup
//     per CU (LDS: 5 K + 4 V tiles of 16 KB plus the block list).  d = 64, where the tiles are 8 KB: two workgroups of 4 waves
//     per CU, a wave owning 64 queries, where there are tiles enough for both (query_sets).
//   * The union of the 4 rows' kept-block lists comes from a pre-pass (tile_lists_kernel), each entry carrying a 4-bit "kept by
//     query block i" mask, and is copied to LDS; no global or scalar load sits on the main loop's critical path.
//   * K and V tiles go straight from global memory into two rings of LDS slots, K four and V two blocks ahead
//     (global_load_lds_dwordx4, bank swizzle applied on the global side).  The wait before the
//     per-block barrier is counted (s_waitcnt vmcnt(n)), so two blocks of loads stay in flight and
//     L2 / fabric latency is covered without a second resident workgroup.
//   * Products are 32x32x16 or, for long lists in calls that fill the chip, 16x16x32 ones (long_list): an instantiation holds both ways from the
//     queries' operands to the epilogue, and a tile takes one by its list's length, its gaps and its round.
//   * The unit of work is half a block (32 keys).  While a wave multiplies (S of one half, then O += V^T P of another), the
//     fma / exp / pack of a third half sit between its MFMAs, a few vector instructions after each.  A block's
//     K and V loads are issued between its two halves.  One barrier per KV block (it also protects the rings).
//   * What bounds the loop is the energy of its instructions: the chip is at its power limit, and fewer cycles for the same
//     instructions only lower the clock.  So whatever is the same for a whole wave is on the scalar unit, and the tiles in LDS
//     are laid out so that operand addresses are one register and an immediate.  Layer calls at B = 1, N = 32760 with that, the row
//     sums on the matrix pipe and, for 64-wide heads, two query sets a wave: 12 heads of 128 dense 5863 -> 5477 us, at 90 % 694 -> 664, 24 heads
//     of 64 at 90 % 862 -> 712; with the smaller products (another card) 5604 -> 5257 (1.25 PFLOP/s), 671 -> 645, 737 -> 704.
//   * V^T operands come from ds_read_b64_tr_b16, K rows are read through the kappa permutation so
//     that P never moves between lanes.  LDS operand reads are spread evenly between the MFMAs through a
//     small ring of fragment registers.
//   * Softmax with few vector instructions: logits live in the log2 domain (one fma and one v_exp_f32 per
//     element); row sums are taken from the bf16-rounded probabilities by a 16x16x32 MFMA against a matrix of zeros and
//     ones (row_sum); the block maximum is not computed unless a block's sums show that some logit exceeds the running
//     reference by more than 13 binades (the reference then moves to the true maximum and the block is redone).
//   * Epilogue: the bf16 fragments of the linear state are staged once per workgroup in LDS.
#include "linear_ride.h"
#include <type_traits>
#include <utility>

namespace salad {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

#define LDS_PTR(p) ((__attribute__((address_space(3))) void *)(p))
#define GLB_PTR(p) ((const __attribute__((address_space(1))) void *)(p))
#define TR_READ(p) __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3))) *)LDS_PTR(p))
#define INL __attribute__((always_inline))
// s_waitcnt with only vmcnt constrained (gfx9 encoding: vmcnt[3:0] | expcnt 7 << 4 | lgkmcnt 15 << 8)
#define WAIT_VM(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | ((n) >> 4) << 14)

// Least entries of a list for 16x16x32 products (the kernel's G), by head width.  Layer calls with 32x32x16 -> 16x16x32 products (us), by entries:
//   128-wide heads, 8, 10, 12, 16:  19 heads, N = 4096 (304 tiles) 53.7 -> 54.1, 59.0 -> 58.8, 64.2 -> 63.2, 74.8 -> 73.3;  50 heads, N = 4096 (800) 124.3 -> 124.2,
//     134.5 -> 133.8, 147.0 -> 144.3, 168.0 -> 164.0;  15 heads, N = 12480 (735) 92.1 -> 93.3, 101.2 -> 101.5, 110.2 -> 109.5, 127.9 -> 126.7;  12 heads, N = 32760 (1536)
//     198.6 -> 195.8, 215.0 -> 211.8, 234.1 -> 230.4, 271.0 -> 268.3
//   64-wide heads, 16, 20, 24, 34:  30 heads, N = 4096 (480) 52.8 -> 52.8, 59.8 -> 58.9, 68.2 -> 65.9, 87.2 -> 83.0;  38 heads (608) 69.5 -> 71.0, 78.7 -> 79.3, 88.2 -> 87.7,
//     112.1 -> 110.4;  24 heads, N = 12480 (1176) 110.4 -> 113.8, 128.9 -> 130.7, 148.1 -> 148.2, 202.3 -> 200.8;  30 heads (1470) 131.3 -> 131.2, 152.9 -> 151.0, 176.8 -> 172.5,
//     234.6 -> 225.2
// Long lists: 12 heads of 128, N = 32760, 54 entries 671 -> 645, 512 5604 -> 5257; 24 heads of 64, 54 entries 737 -> 704.
constexpr int long_list(int d) { return d == 128 ? 12 : 20; }
constexpr int SPLIT_MAX_PIECES = 8;
constexpr int SPLIT_MIN_ENTRIES = 6;     // least entries of a piece: what a cut costs (two passes over 128 KB, a prologue) is about as long

namespace {

__device__ inline int row_of_position5(int kind, int p, int T, int HW, unsigned magic)
{
    if (!kind) return p;
    const int loc = (int)__umulhi((unsigned)p, magic);   // exact p / T (the host checks the range)
    return (p - loc * T) * HW + loc;
}

__device__ inline uint32_t pack2e(float a, float b)
{
    f32x2 x = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2));
}

__device__ inline uint32_t relu2e(uint32_t x)
{
    s16x2 v = __builtin_bit_cast(s16x2, x);
    s16x2 z = {0, 0};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(v, z));
}

// One 16-byte-per-lane global -> LDS load (lane i lands at lds_addr + 16 i).  Issued through inline
// assembly so that the compiler's automatic "wait for every pending LDS load before any LDS read"
// does not apply: which loads must have landed is known exactly and waited for with WAIT_VM below.
__device__ inline void lds_dma16(const void *gptr, unsigned lds_addr_uniform)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(lds_addr_uniform), "v"(gptr)
                 : "memory", "m0");
}

// Same, addressed as (wave-uniform 64-bit base) + (per-lane unsigned 32-bit byte offset): no 64-bit
// vector arithmetic per load.
__device__ inline void lds_dma16_base(const void *base_uniform, unsigned byte_off, unsigned lds_addr_uniform)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(lds_addr_uniform), "v"(byte_off), "s"(base_uniform)
                 : "memory", "m0");
}

// One 4-byte-per-lane global -> LDS load (lane i lands at lds_addr + 4 i).
__device__ inline void lds_dma4(const void *gptr, unsigned lds_addr_uniform)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 :
                 : "s"(lds_addr_uniform), "v"(gptr)
                 : "memory", "m0");
}

// The same past the L2 of this XCD: for what a workgroup on another one has written in the same launch.
__device__ inline void lds_dma4_device(const void *gptr, unsigned lds_addr_uniform)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off sc1" : : "s"(lds_addr_uniform), "v"(gptr) : "memory", "m0");
}
__device__ inline void lds_dma16_device(const void *gptr, unsigned lds_addr_uniform)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off sc1" : : "s"(lds_addr_uniform), "v"(gptr) : "memory", "m0");
}

// x / d for any x and d >= 1, magic = floor(2^32 / d) (2^32 - 1 for d = 1): the multiply-high is at most one too small
__device__ inline unsigned div_by(unsigned x, unsigned d, unsigned magic)
{
    const unsigned q = __umulhi(x, magic);
    return x - q * d >= d ? q + 1 : q;
}

__device__ inline unsigned lds_addr_of(const void *p)
{
    return __builtin_amdgcn_readfirstlane((unsigned)(size_t)LDS_PTR(p));
}

// max of a value over the lanes that own keys of the same query (every G-th), on the VALU: a cross-lane shuffle would go through the LDS
// unit, which the operand reads of the CU's waves keep busy.
template <int G>
__device__ inline float max_of_query(float x)
{
    if constexpr (G == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
    }
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// The lane's number, computed where it is asked for: what follows from it is not kept in registers through the loop for a use behind it (TIGHT).
__device__ inline int lane_again()
{
    unsigned all = ~0u;
    asm volatile("" : "+s"(all));
    return (int)__builtin_amdgcn_mbcnt_hi(all, __builtin_amdgcn_mbcnt_lo(all, 0u));
}

// f(0) .. f(N - 1) with compile-time arguments: where the order of the instructions matters nothing is left for the optimiser to decide (it
// computes the arms of a condition on an unrolled loop's variable ahead of the loop's other work before it knows the variable).
template <class F, int... I>
__device__ inline INL void unrolled_(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ inline INL void unrolled(F &&f)
{
    unrolled_(f, std::make_integer_sequence<int, N>{});
}

union Frag5 {
    bf16x8 v;
    uint4 u;
    uint32_t w[4];
    s16x4 h[2];
};

}  // namespace

// Pre-pass: for every (head, tile of 4 query blocks) the union of the 4 CSR rows' kept blocks, each entry
// tagged with which of the 4 rows keep it.  One wave per tile: bitmap in LDS, ordered compaction with
// ballots, then the ascending list is rotated so that it starts at the entry whose block id is smallest
// modulo the list length.  Softmax does not care about the order, and with sliding windows the rotation makes
// neighbouring tiles (which run at the same time on one XCD and whose windows overlap) reach a given KV
// block at about the same iteration, so the block is fetched into that XCD's L2 once instead of once per
// tile.  The mask is static, but the layer call accepts any CSR, so this runs per call (a few microseconds).
__global__ __launch_bounds__(64) void tile_lists_kernel(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx,
                                                        int nb, int ntiles, int cap, uint32_t *__restrict__ lists,
                                                        int32_t *__restrict__ counts)
{
    extern __shared__ uint32_t bm[];          // [cap] bitmap, then [cap] compacted list
    uint32_t *lst = bm + cap;
    __shared__ uint32_t best;
    const int h = blockIdx.y, tile = blockIdx.x, lane = threadIdx.x;
    for (int i = lane; i < nb; i += 64) bm[i] = 0u;
    if (lane == 0) best = 0xffffffffu;
    __syncthreads();
    for (int i = 0; i < 4; ++i) {
        const int r = tile * 4 + i;
        if (r < nb) {
            const int b0 = row_ptr[h * nb + r], b1 = row_ptr[h * nb + r + 1];
            for (int e = b0 + lane; e < b1; e += 64) {
                const int c = col_idx[e];
                if (c >= 0 && c < nb) atomicOr(&bm[c], 1u << (24 + i));
            }
        }
    }
    __syncthreads();
    int count = 0;
    for (int base = 0; base < nb; base += 64) {
        const int b = base + lane;
        const uint32_t f = b < nb ? bm[b] : 0u;
        const unsigned long long bal = __ballot(f != 0u);
        const int pos = count + __popcll(bal & ((1ull << lane) - 1ull));
        if (f) lst[pos] = (uint32_t)b | f;
        count += __popcll(bal);
    }
    __syncthreads();
    // rotation point: the entry with the smallest (block id mod count); ties cannot occur within count
    // consecutive ids, and for any other list the lowest position wins
    for (int i = lane; i < count; i += 64) {
        const uint32_t key = (lst[i] & 0xffffffu) % (uint32_t)count;
        atomicMin(&best, (key << 13) | (uint32_t)i);      // at most LIST_MAX_ENTRIES entries (checked on the host)
    }
    __syncthreads();
    const int rot = count > 0 ? (int)(best & 0x1fffu) : 0;
    uint32_t *out = lists + ((size_t)h * ntiles + tile) * cap;
    for (int i = lane; i < count; i += 64) {
        int src = i + rot;
        if (src >= count) src -= count;
        out[i] = lst[src];
    }
    if (lane == 0) counts[h * ntiles + tile] = count;
}

int tile_list_cap(int nb) { return (nb + 63) & ~63; }

constexpr int V5_MAX_DYN = 160 * 1024 - 2048;       // the static part is rounded up to its 1 KB alignment
constexpr int v5_ring_bytes(int d) { return 9 * 64 * d * 2; }     // 5 K and 4 V tiles

bool large_tile_list_fits(int d, int nb)
{
    return tile_list_cap(nb) <= LIST_MAX_ENTRIES && v5_ring_bytes(d) + tile_list_cap(nb) * 4 <= V5_MAX_DYN;
}

hipError_t launch_tile_lists(const int32_t *row_ptr, const int32_t *col_idx, int H, int nb, uint32_t *lists,
                             int32_t *counts, hipStream_t st)
{
    const int ntiles = (nb + 3) / 4;
    const int cap = tile_list_cap(nb);
    launch_kernel(tile_lists_kernel, dim3(ntiles, H), dim3(64), (size_t)cap * 8, st, row_ptr, col_idx, nb, ntiles, cap, lists, counts);
    return take_launch_status();
}

// MODE 0: block rows (CSR) through the per-tile union lists.
// MODE 1: token-level Top-K mask (App. A.1.2).  The tile lists are per (sample, head, tile); an entry is
//   block | key-block index << 16 | wave mask << 24 (bit 24 + w: some query of wave w keeps the block); each lane
//   tests its own query's bit of a.topk_mask and contributes nothing for a block it did not select.
// MODE 2: Top-K regrouped by key block.  A query tile is a run of up to 256 gathered queries that all keep the same
//   key block; the list is that key block's 64-token blocks; the normalised partial result and its log-sum-exp go
//   to a.g_po / a.g_lse (one slot per kept (query, key block) pair) for the merge kernel.
// ROPE (MODE 0 only): rotary position embedding inside the linear branch (Sec. 4.1).  The state fragments then hold
//   sum_j (R_j relu(K_j))^T V_j, and the epilogue rotates this tile's relu(Q) fragments in registers (channel pair
//   (2p, 2p+1) of the query's stored row n by the angle word a.rope_tab[n * 64 + p] = fp16 cos | fp16 sin << 16) after
//   the normaliser has been taken from the unrotated features.
// D = 64 (MODE 0 without ROPE only): the same kernel on half-size tiles.  A row is 8 chunks of 16 bytes instead of 16,
// so a tile is half as many 1 KB pieces, and every fragment count halves.
// SPLIT (MODE 0 only): the tiles from a.sp_full on, which do not fill the chip, are cut along their visit lists into up to
// a.sp_pieces workgroups each, or, where that does not pay, by rows into two.  Every piece runs its own softmax over its entries,
// writes O, the reference and the row sum in fp32, and counts itself in; the piece that comes last reads the others back, combines
// all in piece order (so the result does not depend on which it was) and goes on to the epilogue.  Nobody waits for anybody.
// QS: sets of 32 queries that a wave owns.  With 2 every operand fragment read from LDS feeds two products, which halves the energy
// of the reads, and a workgroup has half the waves.  d = 64 has the registers for it and LDS for two such workgroups per CU, whose
// barriers are independent: N = 32760, 24 heads at 90 % 832 -> 725 us.  At d = 128 it needs 400 registers, so one wave per SIMD, and
// the loads, which hold a wave for 60 cycles each, and the scalar code have nothing to run under: dense 5421 -> 5564 us.
// EMIT (d = 128, MODE 0 without ROPE and DBG): the linear branch goes, unscaled, to a.emit_ol instead of being added to O_s.
// RIDE (MODE 0, QS = 1): the launch's first workgroups compute the linear branch's state and gate (linear_ride.h), for which the
// epilogue waits.
template <int D, bool DBG, int MODE = 0, bool ROPE = false, bool SPLIT = false, int QS = 1, bool EMIT = false, bool RIDE = false>
__global__ __launch_bounds__(512 / QS, 2) void sparse_attn_v5_kernel(AttnArgs a, int ntiles, int total, int per_xcd, int list_cap)
{
    static_assert(D == 128 || (D == 64 && MODE == 0 && !ROPE), "d = 64 has the CSR mode only");
    constexpr int CH = D / 8;                    // 16-byte chunks per row
    constexpr int NW = 8 / QS, NT = 64 * NW;     // waves, threads
    constexpr int CG = CH / 4, NPASS = 4 * CG / NW;   // groups of 4 chunks per row; loads of a thread per tile
    constexpr int TILE = 64 * D;                 // elements
    constexpr int NK = 5, NV = 4;                // K and V tiles in LDS
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];
    u16 *Kb = reinterpret_cast<u16 *>(smem);                       // NK tiles
    u16 *Vb = Kb + NK * TILE;                                       // NV tiles
    uint32_t *blist = reinterpret_cast<uint32_t *>(Vb + NV * TILE);      // [list_cap] union list: blk | mask << 24

    constexpr bool TOPK = MODE == 1, GATHER = MODE == 2;
    // Which kernels have both kinds of products (G below).  Riders' calls are one round.  64-wide heads with one query set a wave are calls of up to
    // 384 tiles, the most of which are cut, and those of more than 1792 blocks, whose lists leave no room for a second workgroup: for them, as for the
    // modes of the dynamic mask, the smaller products have not been built.
    constexpr bool BOTH = MODE == 0 && !RIDE && (D == 128 || QS == 2);
    // chunk swizzle of the output staging
    auto oswz = [](int row) INL -> int { return D == 128 ? (row & 15) : ((row >> 1) & 7); };
    float (*ride_small)[32] = nullptr;
    if constexpr (RIDE) {
        static_assert(MODE == 0 && QS == 1, "the riders are 512 threads, and have no use in the modes of the dynamic mask");
        __shared__ float small[DIRECT_WAVES][32];
        ride_small = small;
        if ((int)blockIdx.x < a.ride.wgs) {
            if ((int)blockIdx.x < a.B * (a.H * slices_per_head(D) + a.ride.gate_tasks)) ride<D, ROPE>(blockIdx.x, smem, small);
            return;
        }
    }
    const int g = blockIdx.x - (RIDE ? a.ride.wgs : 0);
    int L, piece = 0, pieces = 1;
    if (SPLIT) {      // an XCD's share: its run of whole tiles, then its run of pieces
        const int fx = a.sp_full / 8, np = (total - a.sp_full) * a.sp_pieces, px = (np + 7) / 8;
        int r = (g >> 3) - fx;
        if (r < 0) {
            L = (g & 7) * fx + (g >> 3);
        } else {
            // QS 2: every sp_pieces-th of the run first, then the next ones.  Workgroups go to the compute units in turn, two to each, and those
            // without work leave at once; in plain order the first pieces, all that a short list has, came to lie in pairs on half of the
            // units.  24 heads of 64, 768 tiles, 6 entries 65.8 -> 60.9 us, 40 heads, 640 tiles, 6 entries 63.7 -> 56.9.  With one workgroup a
            // unit there is nothing to pair, but behind riders those with work have to come first.
            if (QS == 2 || RIDE) {
                const int col = (int)div_by((unsigned)r, (unsigned)a.sp_rows, a.rows_magic);
                r = (r - col * a.sp_rows) * a.sp_pieces + col;
            }
            const int q = (g & 7) * px + r;
            if (r >= px || q >= np) return;
            L = a.sp_full + (int)div_by((unsigned)q, (unsigned)a.sp_pieces, a.pieces_magic);
            piece = q - (L - a.sp_full) * a.sp_pieces;
            pieces = a.sp_pieces;
        }
    } else {
        L = (g & 7) * per_xcd + (g >> 3);
        if (L >= total) return;
    }
    int bh = (int)div_by((unsigned)L, (unsigned)ntiles, a.tiles_magic), tile = L - bh * ntiles;
    int g_J = 0, g_slot0 = 0, g_cnt = 0;
    if (GATHER) {
        const uint4 dsc = a.g_desc[L];
        bh = (int)dsc.x; g_J = (int)dsc.y; g_slot0 = (int)dsc.z; g_cnt = (int)dsc.w;
        if (g_cnt == 0) return;            // unused descriptor
        tile = 0;
    }
    const int smp = (int)div_by((unsigned)bh, (unsigned)a.H, a.heads_magic), h = bh - smp * a.H;
    const int N = a.N, T = a.T, HW = a.HW, nb = a.nb;
    const int kind = (T > 1 && !TOPK) ? (int)((a.kind_mask >> h) & 1ull) : 0;
    const unsigned magic = a.t_magic;
    constexpr uint32_t BLKMASK = TOPK ? 0xffffu : 0xffffffu;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int l32 = lane & 31, hh = lane >> 5;       // a lane's query of a set and half of a row, where rows are read and written
    const u16 *qb = reinterpret_cast<const u16 *>(a.q) + (size_t)bh * N * D;
    const u16 *kb = reinterpret_cast<const u16 *>(a.k) + (size_t)bh * N * D;
    const u16 *vb = reinterpret_cast<const u16 *>(a.v) + (size_t)bh * N * D;

    // ---- The start of a tile is a chain of memory latencies with nothing to run under them (9000 cycles of 57000 for a 13-entry
    // tile), so everything whose address is known is asked for at once: the count and the first entries by scalar loads, the
    // queries and the list straight into LDS, and, as soon as the first entries are there, the first blocks.
    // Where a list is not worth cutting, two workgroups take two of the tile's rows each.  All waves fetch, but with one computing
    // wave per SIMD an iteration is 2100 cycles long instead of 2900.  Cutting in p costs 19000 cycles (scratch, merge; d = 64: 12000),
    // so it takes n 2900 / p + 19000 < n 2100: two pieces from 30 entries on (d = 64: 19), three always.  N = 1950, 12 heads, 11 entries
    // 33.7 -> 29.8 us, 17 entries 39.5 (in two) -> 35.6 (rows); 25 entries 42.8 (rows) -> 38.8 (in four).  Not with two sets of
    // queries a wave: the two workgroups of a compute unit are one computing wave per SIMD each as it is.
    constexpr bool ROW_PAIRS = SPLIT && QS == 1;
    int my_rows = -1;                            // ROW_PAIRS: which two, or all
    const int g_blk0 = g_J * a.g_bpb;
    const uint32_t *src = GATHER ? nullptr : a.tile_lists + ((size_t)(TOPK ? bh : h) * ntiles + tile) * list_cap;
    int n = GATHER ? min(min(nb, g_blk0 + a.g_bpb) - g_blk0, list_cap) : a.tile_counts[(TOPK ? bh : h) * ntiles + tile], list0 = 0;
    auto pieces_of_list = [&]() INL -> int {
        int by_length = min(a.sp_pieces, n / SPLIT_MIN_ENTRIES);
        if (QS == 2) {
            // A piece alone on its compute unit takes 0.9 us an entry, one that shares it 1.6, a cut costs 4.8 and 11 us (fitted to calls of 520
            // to 768 tiles): the best of no cut, as many pieces as have a unit each, and all that there is room for.  Cut wherever pieces had
            // 6 entries: 24 heads, 768 tiles, 12 entries 84.4 -> 75.7 us; 40 heads, 640 tiles, 40 entries 147.1 -> 138.3 (in two, not four).
            const int own = min(a.sp_alone, by_length);
            const int p = own > 1 && 18 * n * (own - 1) > 95 * own ? own : 1;
            if (by_length <= own || (18 * n + (p > 1 ? 95 * p : 0)) * by_length < (32 * n + 220 * by_length) * p) by_length = p;
        }
        return by_length;
    };
    // Two query sets a wave, ahead of a last round that is cut: whether waves raise and lower their priority (part).  Not where each piece of that
    // round, if its lists are as long as this one, may have a compute unit to itself.
    const bool turns = SPLIT && QS == 2 && pieces_of_list() * (total - a.sp_full) > 256;
    if (SPLIT && pieces > 1) {
        const int by_length = pieces_of_list();
        if (by_length > 1 && (!ROW_PAIRS || n * (21 * by_length - 29) > (D == 64 ? 120 : 190) * by_length)) {
            pieces = by_length;
            if (piece >= pieces) return;
            list0 = n * piece / pieces;      // this piece's first entry
            n = n * (piece + 1) / pieces - list0;
        } else {                             // not worth cutting
            const bool rows = ROW_PAIRS && !(RIDE && a.ride.crowded);
            pieces = 1;
            if (piece >= (rows ? 2 : 1)) return;
            if (rows) my_rows = piece;
        }
    }
    constexpr int AK = NK - 1, AV = NV - 2;     // how far ahead of an iteration K and V are fetched
    uint32_t eq[AK];                             // entries j .. j+3 of iteration j; the first one's past the end of the list
#pragma unroll
    for (int b = 0; b < AK; ++b) eq[b] = GATHER ? (uint32_t)min(g_blk0 + b, nb - 1) | 0xff000000u : src[SPLIT ? min(list0 + b, list_cap - 1) : b];
    // How many rows keep the list's first entries: for the choice of the products (G), and asked for here with the others.
    constexpr int LOOKED_AT = 8;
    int kept_bits = 0;
    if (BOTH)
#pragma unroll
        for (int b = 0; b < LOOKED_AT; ++b) kept_bits += __popc(src[b] >> 24);

    // what chunk c of row r of a K or Q piece is swapped with (below)
    auto kswz = [](int row) INL -> int { return -(row >> 2) & 3; };
    const unsigned wave_u = (unsigned)__builtin_amdgcn_readfirstlane(wave);
    // Queries go through LDS, too, each wave's own into a part of the ring that nothing else uses yet: read from memory in operand order,
    // 32 bytes of 32 rows at a time, they pass the 64 bytes a clock of the load path four times.  Laid out like a K tile (below).
    auto q_lds = [&](int u) INL -> unsigned char * {
        const int unit = (int)wave_u * QS + u;
        return reinterpret_cast<unsigned char *>(unit < 6 ? Kb + (2 + (unit >> 1)) * TILE : Vb + (NV - 1) * TILE) + (unit & 1) * (32 * D * 2);
    };
    auto fetch_q = [&]() INL {
#pragma unroll
        for (int u = 0; u < QS; ++u)
#pragma unroll
            for (int rg = 0; rg < 2; ++rg) {
                const int i = ((int)wave_u * QS + u) * 32 + rg * 16 + (lane >> 2);      // query of the tile
                int row;
                if (GATHER) row = min(max(a.g_idx[(size_t)bh * N * a.g_kk + g_slot0 + (i < g_cnt ? i : 0)], 0), N - 1);
                else row = row_of_position5(kind, min(tile * 256 + i, N - 1), T, HW, magic);
                const unsigned off = (unsigned)row * (unsigned)(D * 2) + (unsigned)(((lane & 3) ^ kswz(lane >> 2)) * 16);
                const unsigned dst = lds_addr_of(q_lds(u)) + (unsigned)(rg * CG * 1024);
#pragma unroll
                for (int c = 0; c < CG; ++c) lds_dma16_base(qb + c * 32, off, dst + c * 1024u);
            }
    };
    if (!GATHER) fetch_q();
    // the list's whole row of list_cap slots (built by the pre-pass), without waiting for the count: slots past it hold stale words
    // that are never used
    if (!GATHER)
        for (int i = (int)wave_u * 64; i < list_cap; i += NT)
            lds_dma4(src + (SPLIT ? min(i + lane + list0, list_cap - 1) : i + lane), lds_addr_of(blist + i));

    // ---- All else depends on the products.  16x16x32 ones read and write half the accumulators of 32x32x16 ones for the same work (a loop of
    // them alone reaches 12 % more at the power limit, with this softmax between them 8 %), and the loop of a call that fills the chip is held by
    // the power limit.  But each has its own start to line up with the vector instructions: a block takes 3140 cycles instead of 2960, and a
    // call of one round, or a tile that is half prologue and output, is held by those.  So G = 16 where the list is long_list(D) entries or more and
    // the call more than one round (a.many), and not in a last round that is cut, with a wave to a SIMD for 64-wide heads and dealt out by constants
    // that are of the larger products: N = 12480, that round with 16x16x32 -> 32x32x16 products 11 heads of 128, 23 and 101 entries 142.8 -> 139.4,
    // 428.6 -> 421.4 us; 12 heads of 64, 23 and 43 entries 85.6 -> 83.0, 127.8 -> 124.7.
    // And only where the rows keep five eighths of their tile's list.  A wave's entry that does not follow on another of its own is computed out of
    // the woven part (start_cur, finish_prev), its products and its softmax one after the other, and the wave that does that is the one that the others
    // wait for.  Eight entries in a row of a window that has more are kept by 20 of 32 rows or more.  Layer calls, N = 12480, 32x32x16 ->
    // 16x16x32 products in all tiles (us), rows of random blocks, by the share that they keep of their tile's list: 15 heads of 128 0.39 509 -> 554,
    // 0.53 673 -> 706, 0.62 746 -> 752, 0.71 884 -> 855, 0.80 968 -> 923; 30 heads of 64 0.39 615 -> 653, 0.53 819 -> 827, 0.62 913 -> 890, 0.80 1084 -> 1035;
    // of random runs of four blocks: 15 heads 0.39 539 -> 610, 0.62 755 -> 784, 0.80 965 -> 937.
    auto rest = [&](auto g_, auto turns_) INL {
    constexpr int G = decltype(g_)::value;
    constexpr int KD = 512 / G, NS = D / KD;     // channels of a product of S, its steps
    constexpr int NDT = D / G;                   // G-channel tiles of O^T
    constexpr int QG = 32 / G * QS;              // groups of G queries that a wave owns: the columns of one product
    constexpr int NKG = 32 / G;                  // products of S for the 32 keys of a half
    constexpr int NP = G / 16;                   // P's operands for them
    constexpr bool TURNS = decltype(turns_)::value;
    // Two query sets a wave take all registers for the loop.  What the epilogue and a call's last block need is then computed there, and flags are
    // one for the wave: else 17 to 32 registers were in memory, some loaded again behind a block's loads, which the wait for them then waits for,
    // too.  24 heads of 64, N = 12480: 23 entries 160.8 -> 155.4 us, rows that keep every second block 590 -> 567, a random 10 % 275 -> 263.  With one
    // set there are registers for it all, and the same costs time: 12 heads, N = 1950 24.5 -> 24.8, 480p dense 5064 -> 5099.
    constexpr bool TIGHT = QS == 2;
    constexpr int EL = G / 2;                    // logits of a half that a lane owns, a group
    constexpr int AR = G * G / 64;               // accumulators of a lane
    typedef float acc_t __attribute__((ext_vector_type(AR)));
    const int lq = lane % G, ls = lane / G;          // a lane's query of a group and share of 8 channels or 4 rows in the products
    unsigned mybit = 0u;
    Frag5 qf[QG][NS];
    uint32_t qm_lo[QG] = {}, qm_hi[QG] = {};     // TOPK: this lane's queries' key-block bits
    auto rows_active = [&](int unit) INL -> bool { return !ROW_PAIRS || my_rows < 0 || my_rows == unit >> 2; };
    // Stored row of query i of the wave's set u (a valid one also where there is none), and whether there is one.  GATHER: the place in the run.
    auto query_row = [&](int u, int i, bool &valid) INL -> int {
        const int unit = (int)wave_u * QS + u, p = GATHER ? unit * 32 + i : tile * 256 + unit * 32 + i;
        valid = GATHER ? p < g_cnt : p < N && rows_active(unit);
        return GATHER ? p : row_of_position5(kind, min(p, N - 1), T, HW, magic);
    };
    bool valid0 = false;
    int row0 = 0;                                // this lane's query, unless TIGHT
    if (!TIGHT) row0 = query_row(0, l32, valid0);
#pragma unroll
    for (int u = 0; u < QS; ++u) {
        const int unit = wave * QS + u, qblk = tile * 4 + (unit >> 1);
        if (GATHER) mybit |= unit * 32 < g_cnt ? (1u << (24 + unit)) : 0u;
        else mybit |= qblk < nb && rows_active(unit) ? (1u << (24 + (TOPK ? unit : unit >> 1))) : 0u;
        if (TOPK)
#pragma unroll
            for (int c = 0; c < NKG; ++c) {     // spatial heads only: a position is its row
                const int row = qblk * 64 + (unit & 1) * 32 + c * G + lq;
                const unsigned long long m = qblk < nb && row < N ? a.topk_mask[(size_t)bh * N + row] : 0ull;
                qm_lo[NKG * u + c] = (uint32_t)m;
                qm_hi[NKG * u + c] = (uint32_t)(m >> 32);
            }
    }
    const float c2 = a.scale * 1.44269504088896340736f;   // logits are handled in the log2 domain

    // ---- global -> LDS.  A tile is laid out in pieces of 1 KB, 16 rows by 4 chunks (64 bytes) each, the CG pieces of 16 rows one
    // after the other; one load of a wave fills a piece.  Within a piece chunk c of row r is at r * 64 + ((c ^ x(r)) * 16), the swap being
    // made in the global address, so that each 256 bytes that a read takes at a time cover all banks once.  Those are, for the transposing reads
    // of V, 32 lanes in a row: 4 rows by 64 bytes (G = 32: no swap) or 8 rows by 32 bytes (G = 16: x = r / 4 % 2 * 2); for the 16-byte reads of
    // K and Q lanes 0-3, 12-15, 20-23 and 24-27, then 4-7, 8-11, 16-19 and 28-31: x = -(r / 4) % 4 (r / 4 % 4 does for G = 32, but with four
    // shares of channels side by side it costs twice the cycles of every read).  Of an operand's address only one or two bits of the chunk depend
    // on both lane and step; all else of the step is an immediate.
    // LDS destinations are wave-uniform scalars; global sources are a uniform base plus a 32-bit offset.
    const unsigned k_lds0 = lds_addr_of(Kb) + wave_u * (NPASS * 1024u);
    const unsigned v_lds0 = lds_addr_of(Vb) + wave_u * (NPASS * 1024u);
    const unsigned Tk = kind ? (unsigned)T : 0x7fffffffu;
    const int lr = wave * NPASS / CG * 16 + (lane >> 2);                       // this thread's row of a tile
    const int vchunk = (lane & 3) ^ (G == 16 ? (lane >> 4 & 1) * 2 : 0);
    const unsigned vchunk_b = (unsigned)(wave * NPASS % CG * 64 + vchunk * 16);
    const unsigned kv_b = (unsigned)((((lane & 3) ^ kswz(lane >> 2)) - vchunk) * 16);     // K's chunk less V's
    // byte offset of this thread's row of a block and its V chunk.  The division is by a scalar, of the block's first row; a lane's own
    // part is a constant, but for one wrap of the time axis.  Without a branch on the order (a spatial head is location 0, stride 1).
    const unsigned magic_u = kind ? magic : 0u, stride_b = (unsigned)((kind ? HW : 1) * D * 2), back_b = (unsigned)(D * 2) - (unsigned)T * stride_b;
    // (p - loc T) stride + loc, in rows of 2 D bytes
    auto row_bytes = [&](unsigned p) INL -> unsigned { return p * stride_b + __umulhi(p, magic_u) * back_b; };
    const unsigned ql = __umulhi((unsigned)lr, magic_u), rl = (unsigned)lr - ql * (unsigned)T * (kind ? 1u : 0u);
    const unsigned lane0 = (unsigned)lr * stride_b + ql * back_b + vchunk_b, lane1 = lane0 + (unsigned)(D * 2) - (unsigned)T * stride_b;
    auto rows_of = [&](int blk) INL -> unsigned {
        const unsigned p0 = (unsigned)__builtin_amdgcn_readfirstlane(blk * 64);
        if (__builtin_expect((int)p0 + 64 > N, 0)) return row_bytes((unsigned)min((int)p0 + lr, N - 1)) + vchunk_b;
        const unsigned q0 = __umulhi(p0, magic_u);
        const unsigned base = p0 * stride_b + q0 * back_b, left = Tk - (kind ? p0 - q0 * (unsigned)T : 0u);
        return base + (rl >= left ? lane1 : lane0);
    };
    auto fetch_k = [&](unsigned r, int slot) INL {
#pragma unroll
        for (int i = 0; i < NPASS; ++i) lds_dma16_base(kb + i * 32, r + kv_b, k_lds0 + (unsigned)slot * (unsigned)(TILE * 2) + i * 1024u);
    };
    auto fetch_v = [&](unsigned r, int slot) INL {
#pragma unroll
        for (int i = 0; i < NPASS; ++i) lds_dma16_base(vb + i * 32, r, v_lds0 + (unsigned)slot * (unsigned)(TILE * 2) + i * 1024u);
    };
    // list entries travel in a vector register (lane l holds entry 64 c + l of the current 64-entry
    // chunk c) and are picked with v_readlane: no LDS round trip per iteration
    uint32_t ev = 0u;
    const uint32_t tail_blk = (N & 63) ? (uint32_t)(N >> 6) : 0xffffffffu;             // the block that the sequence ends in
    auto entry = [&](int idx) INL -> uint32_t { return (uint32_t)__builtin_amdgcn_readlane((int)ev, idx & 63); };

    // first blocks: enough for iteration 0; the rest of what the loop expects in flight follows once these have landed
    unsigned rk[AK - AV + 1] = {};               // row offsets of blocks j+2 .. j+4, for the V fetches to come
    unsigned r1 = 0u;
    if (n > 0) {
        const unsigned r0 = rows_of((int)(eq[0] & BLKMASK));
        fetch_k(r0, 0);
        if (n > 1) {
            r1 = rows_of((int)(eq[1] & BLKMASK));
            fetch_k(r1, 1);
        }
        fetch_v(r0, 0);
    }

    // ---- LDS operand addresses.  P never moves between lanes: the logits that a lane gets are those of the keys whose P it has to hold.
    // G = 32 reads K's rows in the order that swaps bits 2 and 3 of the row (kappa); the accumulators are then the 8-key groups of P's operands.
    // With G = 16 a lane's logits of a half are keys 16 kg + 4 ls + t (kg the product, t the register), and V is read in that order of keys;
    // an operand of K is one piece of a tile, of V^T half the width of two.
    unsigned koff[2], voff[2];
    if constexpr (G == 16) {
        koff[0] = koff[1] = (unsigned)(lq * 64 + ((ls ^ kswz(lq)) << 4));
        voff[0] = (unsigned)((4 * ls + (lq >> 2)) * 64 + ((((lq & 3) >> 1) ^ (ls & 1) * 2) << 4) + 8 * (lq & 1));
        voff[1] = voff[0] ^ 32u;
    } else {
        const int kappa = (l32 & 0x13) | ((l32 & 4) << 1) | ((l32 & 8) >> 1);
#pragma unroll
        for (int p = 0; p < 2; ++p)
            koff[p] = (unsigned)((kappa >> 4) * (CG * 1024) + (kappa & 15) * 64 + (((2 * p + hh) ^ kswz(kappa)) << 4));
        voff[0] = voff[1] = (unsigned)((8 * hh + ((l32 >> 2) & 3)) * 64 + (2 * (l32 >> 4) + ((l32 & 3) >> 1)) * 16 + 8 * (l32 & 1));
    }
    // step t of the S products of a half, and of its O^T products
    auto k_frag = [&](const u16 *Kt, int half, int t) INL -> bf16x8 {
        const unsigned char *p = reinterpret_cast<const unsigned char *>(Kt) + half * (2 * CG * 1024);
        if constexpr (G == 16) return *(const bf16x8 *)(p + koff[0] + t / NS * (CG * 1024) + t % NS * 1024);
        else return *(const bf16x8 *)(p + koff[t & 1] + (t >> 1) * 1024);
    };
    auto v_frag = [&](Frag5 &f, const u16 *Vt, int half, int t) INL {
        const unsigned char *p = reinterpret_cast<const unsigned char *>(Vt) + half * (2 * CG * 1024);
        if constexpr (G == 16) p += voff[t & 1] + (t >> 1) * 1024;
        else p += voff[0] + t / NDT * (CG * 1024) + t % NDT * 1024;
        f.h[0] = TR_READ(p);
        f.h[1] = TR_READ(p + (G == 16 ? CG * 1024 : 256));
    };

    const f32x4 zero4 = {0.f, 0.f, 0.f, 0.f};
    acc_t zero;
#pragma unroll
    for (int r = 0; r < AR; ++r) zero[r] = 0.f;
    auto product = [&](const Frag5 &x, const Frag5 &y, acc_t c) INL -> acc_t {
        if constexpr (G == 16) return __builtin_amdgcn_mfma_f32_16x16x32_bf16(x.v, y.v, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x.v, y.v, c, 0, 0, 0);
    };
    acc_t o[QG][NDT];
    float m_run[QG], l_run[QG];
    // Whether m_run has been set from a block's true maximum: the same for all queries of a wave, which keep the same list entries, but for TOPK.
    constexpr int NREF = TIGHT ? 1 : QG;
    bool have_ref[NREF] = {};
#pragma unroll
    for (int u = 0; u < QG; ++u) {
#pragma unroll
        for (int i = 0; i < NDT; ++i) o[u][i] = zero;
        m_run[u] = l_run[u] = 0.f;
    }
    acc_t s[QG][2][NKG];                   // logits: group, half of the block, G keys of the half
    Frag5 pf[QG][2][NP];
    auto logit = [&](int u, int hf, int e) INL -> float { return s[u][hf][e / AR][e % AR]; };
    auto p_word = [&](int u, int hf, int pair) INL -> uint32_t & { return pf[u][hf][pair >> 2].w[pair & 3]; };
    // The unit of work is half a block (32 keys).  A part = the S products of one half (NKG NS operands, A = K rows) and the O^T
    // products of one half (NP NDT operands, A = V^T, two transposing 8-byte reads), each against every group of queries, with the
    // softmax of a third half woven between them.  Operand fragments move through a ring of RING register quads: step i takes ring[i % RING] and the read
    // of fragment i + RING is issued right after it; the last steps of a block read the next block's first K fragments.
    constexpr int RING = QS == 2 ? 2 : 4;         // 8: 5957 against 5842 us on the dense call; QS = 2 with 4: 731 against 725 us
    Frag5 ring[RING];
    constexpr int SS = NKG * NS, OS = NP * NDT, NPS = SS + OS;      // steps of a part
    static_assert((2 * NPS) % RING == 0, "a block's fragments go round the ring a whole number of times");
    auto read_frag = [&](int i, const u16 *Vt, const u16 *Kt, const u16 *Kn) INL {     // i counts a block's 2 NPS fragments
        Frag5 &f = ring[i % RING];
        const int pt = i / NPS, t = i % NPS;
        if (t < SS) f.v = k_frag(pt < 2 ? Kt : Kn, pt & 1, t);
        else v_frag(f, Vt, pt & 1, t - SS);
    };
    auto mfma_S = [&](int u, int pt, int t, const Frag5 &f) INL {
        acc_t &acc = s[u][pt][t / NS];
        acc = product(f, qf[u][t % NS], t % NS == 0 ? zero : acc);
    };
    auto mfma_PV = [&](int u, int pt, int t, const Frag5 &f) INL { o[u][t % NDT] = product(f, pf[u][pt][t / NDT], o[u][t % NDT]); };
    // TOPK: a lane whose query did not select the entry's key block gets P = 0 (scale 0, reference +inf) and takes no part
    // in the reference updates
    auto selected = [&](int u, uint32_t e) INL -> bool {
        if (!TOPK) return true;
        const int J = (int)((e >> 16) & 63u);
        return (((J & 32) ? qm_hi[u] : qm_lo[u]) >> (J & 31)) & 1u;
    };
    auto mask_tail = [&](int hf, uint32_t e) INL {           // keys past the sequence end (last block only)
        const int blk = (int)(e & BLKMASK);
        if (__builtin_expect((uint32_t)blk == tail_blk, 0)) {
            int first = blk * 64;
            asm volatile("" : "+s"(first));      // else the compares, the same in every such block, leave the loop and fill the scalar registers
            const int kbase = first + hf * 32 + (TIGHT ? lane_again() / G : ls) * (G / 4);
            auto mask = [&](int u, int e) INL {
                if (kbase + 16 * (e / (G / 4)) + e % (G / 4) >= N) s[u][hf][e / AR][e % AR] = TOPK ? -1e30f : -INFINITY;   // TOPK: stays finite times a zero scale
            };
            if constexpr (TIGHT) {               // a key's compare is used at once, not kept for the other groups
#pragma unroll
                for (int e = 0; e < EL; ++e)
#pragma unroll
                    for (int u = 0; u < QG; ++u) mask(u, e);
            } else {
#pragma unroll
                for (int u = 0; u < QG; ++u)
#pragma unroll
                    for (int e = 0; e < EL; ++e) mask(u, e);
            }
        }
    };
    // Sums of bf16 probabilities, every lane getting its query's, by 16x16x32 products.  With G = 16 the other operand is all ones.  With G = 32 a
    // fragment's lanes 0..15 and 32..47 are, as operand of such a product, keys of queries 0..15, the others keys of queries 16..31, and a
    // lane's results are the rows 4 (lane / 16) .. + 3 of column lane % 16: the A operand picks by row which of the two goes there.  Two rows
    // then share a column and are told apart by zeros only, which is good for finite probabilities: see sums_apart.
    // Four products a block and 32 queries take 64 cycles of the matrix pipe where 16 v_dot2c_f32_bf16 took 256 (plain adds of the unpacked
    // pairs take two more vector instructions per pair, and the loop is held by the energy of its instructions).  Layer call, B = 1, N = 32760:
    // 12 heads of 128 dense 5830 -> 5712 us, at 90 % 687 -> 672; the error against 64 bits is the same to six digits.
    Frag5 pick;
#pragma unroll
    for (int i = 0; i < 4; ++i) pick.w[i] = G == 16 || ((lane >> 2) & 1) == ((lane >> 4) & 1) ? 0x3f803f80u : 0u;
    asm volatile("" : "+v"(pick.w[0]), "+v"(pick.w[1]), "+v"(pick.w[2]), "+v"(pick.w[3]));
    auto row_sum = [&](int u, int hf, int i, f32x4 acc) INL -> f32x4 { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(pick.v, pf[u][hf][i].v, acc, 0, 0, 0); };
    auto row_sums = [&](int u, int hf) INL -> float {
        f32x4 acc = zero4;
#pragma unroll
        for (int i = 0; i < NP; ++i) acc = row_sum(u, hf, i, acc);
        return acc[0];
    };
    // The sums of a half, with the same bits, but each row by itself: with G = 32 a probability that is not finite (a NaN or an infinity in a
    // query, a logit far above the reference) times the zeros that part the rows makes the sum 16 lanes away a NaN as well.
    auto sums_apart = [&](int u, int hf) INL -> float {
        int l = lane;
        asm volatile("" : "+v"(l));                  // else the two masks live in registers all through the loop
        const uint32_t odd = (uint32_t)((int)((unsigned)l << 27) >> 31);       // all ones for the rows 16 .. 31
        uint32_t sum = 0u;
#pragma unroll
        for (int side = 0; side < 2; ++side) {       // the rows of the other side are zeros here
            const uint32_t mine = side ? odd : ~odd;
            f32x4 acc = zero4;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                Frag5 p;
#pragma unroll
                for (int j = 0; j < 4; ++j) p.w[j] = pf[u][hf][i].w[j] & mine;
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pick.v, p.v, acc, 0, 0, 0);
            }
            sum |= __float_as_uint(acc[0]) & mine;
        }
        return __uint_as_float(sum);
    };
    // P = 2^(S c2 - m) rounded to bf16, pair q of half hf; returns the packed pair
    auto pair_exp = [&](float t0, float t1) INL -> uint32_t { return pack2e(__builtin_amdgcn_exp2f(t0), __builtin_amdgcn_exp2f(t1)); };
    auto exp_pack = [&](int u, int hf, bool sel) INL -> float {
        const float cs = (TOPK && !sel) ? 0.f : c2, mref = (TOPK && !sel) ? INFINITY : m_run[u];
#pragma unroll
        for (int q = 0; q < EL / 2; ++q) p_word(u, hf, q) = pair_exp(fmaf(logit(u, hf, 2 * q), cs, -mref), fmaf(logit(u, hf, 2 * q + 1), cs, -mref));
        return row_sums(u, hf);
    };
    // The reference only has to keep 2^S in range, so the maximum is not computed unless the sums say that some logit rose
    // more than 13 binades above the reference (or no reference exists yet): then the reference moves to the true maximum
    // and the half is redone.  Every earlier half is in O and l by then.  whole: the block's second half of logits exists too and
    // counts, so that a row's first reference is the maximum of 64 keys, whose weight is then exactly 1 (keys past the sequence
    // end need no mask here: their K rows are copies of the last one, which is in the block).
    // With the maximum of the first 32 keys alone the error against 64 bits is up to 3 % larger (N = 1170, 95 %: 2.08e-3 -> 2.14e-3).
    // The sums are products over the wave's lanes, so the way here is the whole wave's, and what differs between lanes is selected, not
    // branched on (TOPK: a lane that did not select the entry keeps its reference and adds nothing, whatever the product put into its sum).
    // Only rows that did rise move, so that a row's result does not depend on the others of its wave; with G = 32 a sum that is not finite says so
    // for its own row or for the one 16 lanes away, and sums_apart tells which.
    auto settle = [&](int hf, bool whole, bool started, uint32_t e, const float (&ps)[QG]) INL {
        float psum[QG], all = 0.f;
        bool first[QG], any = false;
#pragma unroll
        for (int u = 0; u < QG; ++u) {
            psum[u] = ps[u];
            all += psum[u];                      // none is negative: within the bound only if each is
            first[u] = !started && !have_ref[TIGHT ? 0 : u];
            if (TOPK) first[u] = __any(selected(u, e) && first[u]);
            any = any || first[u];
        }
        if (__builtin_expect(any || __any(!(all <= 8192.f)), 0)) {
#pragma unroll
            for (int u = 0; u < QG; ++u)
                if (first[u] || __any(!(psum[u] <= 8192.f))) {
                    const bool known = started || have_ref[TIGHT ? 0 : u];
                    float own = psum[u];
                    if (G == 32 && (TOPK || known)) own = sums_apart(u, hf);
                    const bool rises = !known | !(own <= 8192.f), moves = TOPK ? rises & selected(u, e) : rises;
                    float mx = logit(u, hf, 0);
#pragma unroll
                    for (int r = 0; r < EL; ++r) mx = fmaxf(mx, logit(u, hf, r));
                    if (whole)
#pragma unroll
                        for (int r = 0; r < EL; ++r) mx = fmaxf(mx, logit(u, 1, r));
                    mx = fmaf(fmaxf(max_of_query<G>(mx), -1e30f), c2, -m_run[u]);   // maximum minus reference
                    const float shift = !moves ? 0.f : known ? fmaxf(mx, 0.f) : mx;   // new reference minus old reference
                    if (TOPK || known) {
                        const float alpha = TOPK && !known ? 1.f : __builtin_amdgcn_exp2f(-shift);
                        l_run[u] *= alpha;
#pragma unroll
                        for (int i = 0; i < NDT; ++i)
#pragma unroll
                            for (int r = 0; r < AR; ++r) o[u][i][r] *= alpha;
                    }
                    m_run[u] += shift;
                    if constexpr (!TIGHT) have_ref[u] = !TOPK || moves || have_ref[u];      // TOPK apart the same for all lanes, which the compiler is to see
                    psum[u] = exp_pack(u, hf, selected(u, e));
                    if (G == 32 && __builtin_expect(__any(!(psum[u] <= 8192.f)), 0)) psum[u] = sums_apart(u, hf);
                }
            if (TIGHT) have_ref[0] = true;       // behind all groups: each is to find it as it was
        }
#pragma unroll
        for (int u = 0; u < QG; ++u) l_run[u] += !TOPK || selected(u, e) ? psum[u] : 0.f;
    };
    // one part: S of half pt of the current block, O of half pt of the previous block, softmax of the other half in flight
    // (pt 0: the previous block's second half, pt 1: the current block's first half; entry e)
    auto part = [&](auto pt_, uint32_t e, const u16 *Vt, const u16 *Kt, const u16 *Kn) INL {
        constexpr int hf = 1 - decltype(pt_)::value;
        mask_tail(hf, e);
        float cs[QG], mref[QG];
#pragma unroll
        for (int u = 0; u < QG; ++u) {
            const bool sel = selected(u, e);
            cs[u] = (TOPK && !sel) ? 0.f : c2;
            mref[u] = (TOPK && !sel) ? INFINITY : m_run[u];
        }
        // Where the softmax's vector instructions stand, pair p of a part's logits: scaled behind product scaled(p), raised and packed after that.
        // G = 16: two waves a SIMD keep the matrix pipe busy (4 % more cycles than its own) with one exponential or two other instructions behind
        // every product; with the same ones in bunches, five behind every second product, it takes 53 % more.  So two pairs of logits take
        // seven products: scale two, exponential, exponential, the same again, pack all four.
        // G = 32: the steps of a pair one product apart, eight pairs over 13 products.
        constexpr int SLOTS = NPS * QG, GP = EL / 2, PAIRS = GP * QG;       // products of a part; pairs of a group, of all
        struct Row {
            static constexpr int at(int place) { return place * (SLOTS - 4) / (PAIRS / 2 * 7); }
            static constexpr int scaled(int p) { return G == 16 ? at(p / 2 * 7 + p % 2 * 3) : p * (SLOTS - 3 * QS) / PAIRS; }
            static constexpr int raised(int p, int b) { return G == 16 ? at(p / 2 * 7 + p % 2 * 3 + 1 + b) : scaled(p) + 1; }
            static constexpr int packed(int p) { return G == 16 ? at(p / 2 * 7 + 6) : scaled(p) + 2; }
        };
        float t[QG][EL];
        f32x4 ps[QG];
        unrolled<SLOTS>([&](auto slot_) INL {
            constexpr int slot = slot_, i = slot / QG, uu = slot % QG, u = (i & 1) ? QG - 1 - uu : uu, pt = decltype(pt_)::value, hf = 1 - pt;
            constexpr int g = pt * NPS + i;
            // G = 16: the wave that is behind goes first, so that the two of a SIMD come to the barrier together.  480p, 90 % 3240 -> 3180 cycles a
            // block (G = 32, where the oldest wave first has always been: 2957).  Where the two are of different workgroups (64-wide heads), both
            // workgroups of a unit end at the same time by that, and tiles behind them that are too few for two to each unit start in pairs
            // on half of the units.  N = 12480, with -> without: 12 heads, 43 entries 133.0 -> 124.7 us; 26 heads, 101 entries 558 -> 511; but 24 heads,
            // 43 entries, whose last round is cut into pieces for two to a unit, 226 -> 238.  Hence turns, in two copies: branches in here spill.
            if constexpr (G == 16 && TURNS && slot == 0) __builtin_amdgcn_s_setprio(pt ? 1 : 3);
            if constexpr (G == 16 && TURNS && slot == SLOTS / 2) __builtin_amdgcn_s_setprio(pt ? 0 : 2);
            if constexpr (i < SS) mfma_S(u, pt, i, ring[g % RING]); else mfma_PV(u, pt, i - SS, ring[g % RING]);
            if constexpr (uu == QG - 1) read_frag(g + RING, Vt, Kt, Kn);
            __builtin_amdgcn_sched_barrier(0);
            unrolled<PAIRS>([&](auto p_) INL {
                constexpr int p = p_, v = G == 16 ? p / GP : p % QG, q = G == 16 ? p % GP : p / QG, x = 2 * q;
                if constexpr (slot == Row::scaled(p)) {
                    t[v][x] = fmaf(logit(v, hf, x), cs[v], -mref[v]);
                    t[v][x + 1] = fmaf(logit(v, hf, x + 1), cs[v], -mref[v]);
                }
                if constexpr (slot == Row::raised(p, 0)) t[v][x] = __builtin_amdgcn_exp2f(t[v][x]);
                if constexpr (slot == Row::raised(p, 1)) t[v][x + 1] = __builtin_amdgcn_exp2f(t[v][x + 1]);
                if constexpr (slot == Row::packed(p)) p_word(v, hf, q) = pack2e(t[v][x], t[v][x + 1]);
                if constexpr (slot == Row::packed(p) + 1 && q % 4 == 3) ps[v] = row_sum(v, hf, q / 4, q < 4 ? zero4 : ps[v]);
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        float psum[QG];
#pragma unroll
        for (int u = 0; u < QG; ++u) psum[u] = ps[u][0];
        settle(hf, TOPK && hf == 0, !TOPK, e, psum);     // TOPK: a lane's first selected block may come here
    };
    // the same work for blocks that not both of two successive list entries give this wave (first and last entry, entries that
    // another query block of the tile keeps).  Lists of random or strided blocks live on it, so in the uncut d = 128 kernels start_cur has
    // the softmax of the first half between the S products of the second: every third block 1159 -> 1066 us at N = 12480, 24 heads.
    // The same in finish_prev lost (1182), and windows got slower by it where tiles are cut and at d = 64 (480p, 90 % 882 -> 895).
    // Layer calls there, every second / third / a random 30 % of the blocks: 1104 / 998 / 830 us; 24 heads of 64 572 / 535 / 495.
    // Operands are read four steps ahead here, too; only vector and scalar instructions may pass from one step to another.
    auto in_turn = [&](auto count, auto read, auto use) INL {
        Frag5 f[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) read(t, f[t]);
#pragma unroll
        for (int t = 0; t < count; ++t) {
            use(t, f[t % 4]);
            if (t + 4 < count) read(t + 4, f[t % 4]);
            __builtin_amdgcn_sched_barrier(0x406);
        }
    };
    auto finish_prev = [&](uint32_t e, const u16 *Vt) INL {
        mask_tail(1, e);
        in_turn(std::integral_constant<int, 2 * OS>{}, [&](int t, Frag5 &f) INL { v_frag(f, Vt, t / OS, t % OS); }, [&](int t, const Frag5 &f) INL {
            if (t == OS) {          // after the first half's products: the reference may move here
                float psum[QG];
#pragma unroll
                for (int u = 0; u < QG; ++u) psum[u] = exp_pack(u, 1, selected(u, e));
                settle(1, false, !TOPK, e, psum);
            }
#pragma unroll
            for (int u = 0; u < QG; ++u) mfma_PV(u, t / OS, t % OS, f);
        });
    };
    auto start_cur = [&](uint32_t e, const u16 *Kt) INL {
        constexpr bool woven = D == 128 && !SPLIT;
        float psum[QG];
        in_turn(std::integral_constant<int, 2 * SS>{}, [&](int t, Frag5 &f) INL { f.v = k_frag(Kt, t / SS, t % SS); }, [&](int t, const Frag5 &f) INL {
            if (woven && t == SS) mask_tail(0, e);
#pragma unroll
            for (int u = 0; u < QG; ++u) mfma_S(u, t / SS, t % SS, f);
            if (woven && t >= SS)
#pragma unroll
                for (int u = 0; u < QG; ++u) {
                    const bool sel = selected(u, e);
                    const float cs = (TOPK && !sel) ? 0.f : c2, mref = (TOPK && !sel) ? INFINITY : m_run[u];
#pragma unroll
                    for (int q = 0; q < EL / 2; ++q)
                        if ((u * (EL / 2) + q) * (SS - 1) / (EL / 2 * QG) == t - SS - 1)
                            p_word(u, 0, q) = pair_exp(fmaf(logit(u, 0, 2 * q), cs, -mref), fmaf(logit(u, 0, 2 * q + 1), cs, -mref));
                }
        });
        if constexpr (woven) {
#pragma unroll
            for (int u = 0; u < QG; ++u) psum[u] = row_sums(u, 0);
        } else {
            mask_tail(0, e);
#pragma unroll
            for (int u = 0; u < QG; ++u) psum[u] = exp_pack(u, 0, selected(u, e));
        }
        settle(0, true, false, e, psum);
    };

    bool lin = !GATHER && a.use_linear && !a.write_sparse_only && !(a.drop && a.drop[smp]);   // pruned sample (Sec. 4.3): out = O_s
    const u16 *hf = a.hfrag + (size_t)bh * D * D;
    float coef = lin && !RIDE && QS == 1 ? a.coef[bh] : 0.f;
    // RIDE: the sample's scale from the gate's partial sums, every wave for itself, in the order of finalize_kernel; tile 0 of a head writes it down
    auto reduce_gate = [&]() INL {
        CallRef c = call_args();
        float t[4] = {};
        const int nparts = c.ride.nparts;
        const float *p = c.ride.gate_sums + (size_t)smp * nparts * 4;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            for (int j = i * 64 + lane; j < nparts; j += 256)
                t[i] += (ride_loadf(p + j * 4) + ride_loadf(p + j * 4 + 1)) + (ride_loadf(p + j * 4 + 2) + ride_loadf(p + j * 4 + 3));
        float sum = (t[0] + t[2]) + (t[1] + t[3]);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        const float sc = nparts > 0 ? sum / (float)N : c.s_dev[smp];
        const bool dropped = c.ride.tau > 0.f && sc < c.ride.tau;      // Sec. 4.3: out = O_s
        coef = dropped ? 0.f : c.lambda * (c.head_scale ? c.head_scale[h] : 1.f) * sc;
        if (tile == 0 && tid == 0) {
            if (h == 0 && c.s_out) c.s_out[smp] = sc;
            c.coef_out[bh] = coef;
            if (h == 0 && c.ride.tau > 0.f) {
                c.ride.drop[smp] = dropped;
                if (c.ride.dropped_out) c.ride.dropped_out[smp] = dropped;
            }
        }
        if (__builtin_amdgcn_readfirstlane(dropped)) lin = false;
    };
    // the D x D linear-state fragments (32 KB at d = 128) for the epilogue, staged into the K ring once it is idle, and the normaliser's
    // sums into the V slot two after the last block's
    int v_last = 0;                         // V-ring slot of the last block: the only tile still read after the loop
    auto z_lds = [&]() INL -> float * { return reinterpret_cast<float *>(Vb + ((v_last + 2) & (NV - 1)) * TILE); };
    auto stage_state = [&]() INL {
        if constexpr (RIDE) {
            // counted at once: the word can go back to 0 before the riders are seen in it, which says the same
            if (tid == 0) {
                CallRef c = call_args();
                const uint64_t now = ride_count(c, bh, RIDE_TILE * (my_rows < 0 ? 2 : 1), c.ride.full), tag = c.ride.tag;
                const int riders = c.ride.riders;
                bool there = (int)(now & (RIDE_TILE - 1)) == riders;
                for (int i = c.ride.polls; !there && i > 0; --i) {
                    __builtin_amdgcn_s_sleep(2);
                    const uint64_t x = ride_load(ride_word(c, bh));
                    there = (x & ~RIDE_COUNT) != tag || (int)(x & (RIDE_TILE - 1)) == riders;
                }
                ride_small[0][0] = there ? 1.f : 0.f;
            }
            __syncthreads();
            if (__builtin_expect(__builtin_amdgcn_readfirstlane(ride_small[0][0] == 0.f), 0)) {
                __syncthreads();
                ride_alone<D, ROPE>(bh, smem, ride_small);
            }
            if ((int)wave_u * 64 < D) lds_dma4_device(a.Z + (size_t)bh * D + wave_u * 64 + lane, lds_addr_of(z_lds() + wave_u * 64));
#pragma unroll
            for (int i = 0; i < D * D / (NT * 8); ++i) lds_dma16_device(hf + (size_t)(i * NT + tid) * 8, lds_addr_of(Kb + (i * NT + wave * 64) * 8));
            return;
        }
        if ((int)wave_u * 64 < D) lds_dma4(a.Z + (size_t)bh * D + wave_u * 64 + lane, lds_addr_of(z_lds() + wave_u * 64));
#pragma unroll
        for (int i = 0; i < D * D / (NT * 8); ++i) lds_dma16(hf + (size_t)(i * NT + tid) * 8, lds_addr_of(Kb + (i * NT + wave * 64) * 8));
    };

    // ROPE: this lane's 32 angle words (its queries' rows of the table: pairs KD / 2 st + 4 ls + j), fetched under the last
    // PV product of the tile
    uint4 ang[QG][ROPE ? NS : 1];
    auto load_angles = [&]() INL {
        if (ROPE)
#pragma unroll
            for (int u = 0; u < QG; ++u) {
                const uint32_t *tr = a.rope_tab + (size_t)__shfl(row0, u * G + lq) * (D / 2) + ls * 4;
#pragma unroll
                for (int st = 0; st < NS; ++st) ang[u][st] = *reinterpret_cast<const uint4 *>(tr + st * (KD / 2));
            }
    };

    // ---- main loop over the union list.  Iteration j: S(j) and the softmax of its first half, the softmax of the second
    // half of block j-1 and its O products; fetch K of block j+4 and V of block j+2.  Block b lives in slot b % NK of the
    // K ring and b % NV of the V ring: K(b) is read at the end of iteration b-1 and in b, V(b) in b+1.  The barrier of
    // iteration j says that everything fetched up to iteration j-3 has landed (K(j+1) and V(j-1) among it), so two
    // iterations' loads stay in flight, and that iteration j-1 no longer reads the slots that j fetches into.
    // List, queries and K of block 0 are there, K of block 1 and V of block 0 still on their way; from here on the only vector-memory
    // operations in flight are the K/V fetches, whose completion is tracked by hand.
    if (GATHER) fetch_q();
    if (!GATHER && n > 1) WAIT_VM(2 * NPASS); else WAIT_VM(0);
    asm volatile("" ::: "memory");
    {
        // step st of group u: 8 channels from KD st + 8 ls of row lq of the group
#pragma unroll
        for (int u = 0; u < QG; ++u)
#pragma unroll
            for (int s = 0; s < NS; ++s)
                qf[u][s].u = *reinterpret_cast<const uint4 *>(q_lds(u / NKG) + (G == 16 ? u % NKG : lq >> 4) * (CG * 1024) + (lq & 15) * 64 + s * (KD / 8) / 4 * 1024 +
                                                              (((s * (KD / 8) % 4 + ls) ^ kswz(lq & 15)) << 4));
    }
#pragma unroll
    for (int u = 0; u < QG; ++u) {
#pragma unroll
        for (int s = 0; s < NS; ++s)
            asm volatile("" : "+v"(qf[u][s].w[0]), "+v"(qf[u][s].w[1]), "+v"(qf[u][s].w[2]), "+v"(qf[u][s].w[3]));
        asm volatile("" : "+v"(qm_lo[u]), "+v"(qm_hi[u]));
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    auto load_entries = [&](int first) INL {      // entries first .. first + 63
        if (GATHER) ev = (uint32_t)min(g_blk0 + first + lane, nb - 1) | 0xff000000u;
        else asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(ev) : "v"((unsigned)(size_t)LDS_PTR(blist + first + lane)) : "memory");
    };
    load_entries(0);
    if (n > 0) {
        static_assert(AK == 4 && AV == 2, "the waits below count the loads of two iterations");
        if (n > 2) fetch_k(rk[0] = rows_of((int)(eq[2] & BLKMASK)), 2);
        if (n > 3) fetch_k(rk[1] = rows_of((int)(eq[3] & BLKMASK)), 3);
        if (n > 1) fetch_v(r1, 1);
        uint32_t e_prev = 0u;                     // entry j-1
        int kslot = 0, vslot = 0;                 // j % NK, j % NV
        // The expectations keep the usual way through an iteration free of taken branches: dense 5525 -> 5455 us, 480p 90 % 652 -> 644.
        for (int j = 0; j < n; ++j) {
            if (__builtin_expect(j + AK <= n, 1)) WAIT_VM(4 * NPASS); else WAIT_VM(0);
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            const int jf = j + AK;
            uint32_t e_f = 0u;
            if (__builtin_expect(jf < n, 1)) {
                // waited for inside, so that the other turns of the loop need not wait for their operand reads
                if (__builtin_expect((jf & 63) == 0, 0)) load_entries(jf);
                e_f = entry(jf);
            }
            int kslot_f = kslot - 1; if (kslot_f < 0) kslot_f += NK;
            int kslot_n = kslot + 1; if (kslot_n >= NK) kslot_n -= NK;
            const int vslot_f = vslot ^ AV, vslot_prev = (vslot - 1) & (NV - 1);
            const uint32_t e_cur = eq[0];
            const bool kS = (e_cur & mybit) != 0, kP = (e_prev & mybit) != 0;
            const u16 *Kt = Kb + kslot * TILE, *Kn = Kb + kslot_n * TILE;
            const u16 *Vt = Vb + vslot_prev * TILE;
            auto dma = [&]() INL {
                if (__builtin_expect(jf < n, 1)) {
                    rk[2] = rows_of((int)(e_f & BLKMASK));
                    fetch_k(rk[2], kslot_f);
                }
                if (__builtin_expect(j + AV < n, 1)) fetch_v(rk[0], vslot_f);
            };
            if (__builtin_expect(kP && kS, 1)) {
                part(std::integral_constant<int, 0>{}, e_prev, Vt, Kt, Kn);
                dma();
                part(std::integral_constant<int, 1>{}, e_cur, Vt, Kt, Kn);
            } else {
                dma();
                if (kP) finish_prev(e_prev, Vt);
                if (kS) start_cur(e_cur, Kt);
#pragma unroll
                for (int i = 0; i < RING; ++i) read_frag(2 * NPS + i, Vt, Kt, Kn);
            }
            rk[0] = rk[1];
            rk[1] = rk[2];
            e_prev = e_cur;
#pragma unroll
            for (int b = 0; b + 1 < AK; ++b) eq[b] = eq[b + 1];
            eq[AK - 1] = e_f;
            kslot = kslot_n;
            vslot = (vslot + 1) & (NV - 1);
        }
        // tail: the last block's second half and its O products.  The K ring is idle from here on, so the epilogue's
        // state fragments are fetched into it under these MFMAs.
        WAIT_VM(0);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        v_last = vslot ? vslot - 1 : NV - 1;
        if (lin && !RIDE && !(SPLIT && pieces > 1)) stage_state();
        if (ROPE && lin && !(SPLIT && pieces > 1)) load_angles();
        if ((e_prev & mybit) != 0) finish_prev(e_prev, Vb + v_last * TILE);
    }

    if (SPLIT && G == 32 && pieces > 1) {
        const int first = (L - a.sp_full) * a.sp_pieces;      // the tile's pieces in the scratch
        constexpr int PER = NDT * (AR / 2) * 512;             // register pairs of a piece: pair r of thread tid at r * 512 + tid
        // The pieces of a tile may run on different XCDs, whose L2 caches do not see each other.  Instead of fences, which
        // write back and invalidate a whole L2 (101 against 37 us for a layer call of N = 1950), the scratch is written and
        // read with device-scope accesses, which go past it: a piece's stores are at the common level when they are
        // acknowledged, which every wave waits for before the workgroup counts itself in.
        auto put = [&](uint64_t *p, float x, float y) INL {
            __hip_atomic_store(p, (uint64_t)__float_as_uint(x) | (uint64_t)__float_as_uint(y) << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        auto get = [&](const uint64_t *p) INL -> float2 {
            const uint64_t v = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
        };
        uint64_t *mine = a.sp_o + (size_t)(first + piece) * PER + tid;
#pragma unroll
        for (int u = 0; u < QS; ++u) {
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                for (int r = 0; r < AR / 2; ++r) put(mine + (dt * (AR / 2) + r) * 512 + u * NT, o[u][dt][2 * r], o[u][dt][2 * r + 1]);
            // a wave that kept no entry of this piece has no reference, and nothing to add
            put(a.sp_ml + (size_t)(first + piece) * 512 + u * NT + tid, have_ref[TIGHT ? 0 : u] ? m_run[u] : -INFINITY, l_run[u]);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        WAIT_VM(0);
        __syncthreads();
        if (tid == 0) {
            // one round trip where the counter carries the call's tag, which the reduce ahead of this launch writes; without that
            // launch the first piece to arrive puts it there (a failed exchange means that another piece has got further)
            uint64_t *cnt = a.sp_count + (L - a.sp_full);
            uint64_t now = __hip_atomic_fetch_add(cnt, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
            while ((now & ~15ull) != a.sp_tag) {
                const uint64_t first = a.sp_tag + 1;
                if (__hip_atomic_compare_exchange_strong(cnt, &now, first, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) now = first;
                else if ((now & ~15ull) == a.sp_tag) now = __hip_atomic_fetch_add(cnt, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
            }
            const bool last = (int)(now & 15) == pieces;
            if (last) __hip_atomic_store(cnt, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            blist[0] = last;
        }
        __syncthreads();
        if (!blist[0]) return;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        float mx[QS];
#pragma unroll
        for (int u = 0; u < QS; ++u) {
            mx[u] = -INFINITY;
            for (int p = 0; p < pieces; ++p) mx[u] = fmaxf(mx[u], get(a.sp_ml + (size_t)(first + p) * 512 + u * NT + tid).x);
#pragma unroll
            for (int i = 0; i < NDT; ++i) o[u][i] = zero;
            l_run[u] = 0.f;
        }
        for (int p = 0; p < pieces; ++p)
#pragma unroll
            for (int u = 0; u < QS; ++u) {
                const float2 ml = get(a.sp_ml + (size_t)(first + p) * 512 + u * NT + tid);
                const float wt = ml.x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml.x - mx[u]);
                const uint64_t *src = a.sp_o + (size_t)(first + p) * PER + u * NT + tid;
                l_run[u] = fmaf(wt, ml.y, l_run[u]);
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int r = 0; r < AR / 2; ++r) {
                        const float2 v = get(src + (dt * (AR / 2) + r) * 512);
                        o[u][dt][2 * r] = fmaf(wt, v.x, o[u][dt][2 * r]);
                        o[u][dt][2 * r + 1] = fmaf(wt, v.y, o[u][dt][2 * r + 1]);
                    }
            }
#pragma unroll
        for (int u = 0; u < QS; ++u) m_run[u] = mx[u];
    }

    // ---- epilogue ---------------------------------------------------------------------------------
    float lin_scale[QG], inv_den[QG];
    if (lin) {
        const bool late = n == 0 || (SPLIT && pieces > 1);       // not under the last PV product
        if (RIDE || late) stage_state();
        if (ROPE && late) load_angles();
        if (RIDE) reduce_gate();
        if (QS == 2) coef = a.coef[bh];          // there is no register for it before
#pragma unroll
        for (int u = 0; u < QG; ++u)
#pragma unroll
            for (int st = 0; st < NS; ++st)
#pragma unroll
                for (int j = 0; j < 4; ++j) qf[u][st].w[j] = relu2e(qf[u][st].w[j]);
        WAIT_VM(0);
        __syncthreads();   // the staged fragments have landed in every wave's view
        float dpart[QG] = {};
        const float *Zh = z_lds() + (TIGHT ? lane_again() / G : ls) * 8;
#pragma unroll
        for (int st = 0; st < NS; ++st) {
            const float4 z0 = *reinterpret_cast<const float4 *>(Zh + st * KD), z1 = *reinterpret_cast<const float4 *>(Zh + st * KD + 4);
            const float zz[8] = {z0.x, z0.y, z0.z, z0.w, z1.x, z1.y, z1.z, z1.w};
#pragma unroll
            for (int u = 0; u < QG; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t w = qf[u][st].w[j];
                    dpart[u] = fmaf(__uint_as_float(w << 16), zz[2 * j], dpart[u]);
                    dpart[u] = fmaf(__uint_as_float(w & 0xffff0000u), zz[2 * j + 1], dpart[u]);
                }
        }
#pragma unroll
        for (int u = 0; u < QG; ++u) {
            if (G == 16) dpart[u] += __shfl_xor(dpart[u], 16);
            const float den = dpart[u] + __shfl_xor(dpart[u], 32) + a.eps;
            inv_den[u] = 1.f / den;
            lin_scale[u] = coef * inv_den[u];
        }
        if (ROPE) {
            // numerator operand: R_i relu(Q_i), rounded to bf16 like every MFMA operand (the normaliser above keeps the
            // unrotated features)
#pragma unroll
            for (int u = 0; u < QG; ++u)
#pragma unroll
                for (int st = 0; st < NS; ++st) {
                    const uint32_t cw[4] = {ang[u][st].x, ang[u][st].y, ang[u][st].z, ang[u][st].w};
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t w = qf[u][st].w[j];
                        const float x = __uint_as_float(w << 16), y = __uint_as_float(w & 0xffff0000u);
                        const f16x2 hcs = __builtin_bit_cast(f16x2, cw[j]);
                        const float cc = (float)hcs[0], ss = (float)hcs[1];
                        qf[u][st].w[j] = pack2e(x * cc - y * ss, x * ss + y * cc);
                    }
                }
        }
    }
    if (ROW_PAIRS && my_rows >= 0 && mybit == 0u) return;      // a wave of the other rows, no barrier follows
#pragma unroll
    for (int u = 0; u < QS; ++u) {
    const int unit = wave * QS + u, lane = TIGHT ? lane_again() : tid & 63, lq = lane % G, ls = lane / G, l32 = lane & 31, hh = lane >> 5;
    const int u0 = NKG * u;                  // this set's groups: u0 .. u0 + NKG - 1
    float inv_l[NKG];
#pragma unroll
    for (int c = 0; c < NKG; ++c) inv_l[c] = l_run[u0 + c] > 0.f ? 1.f / l_run[u0 + c] : 0.f;
    acc_t num[NKG][NDT];
    if (lin) {
        // the state's fragments are those of 32x32x16 products: with G = 16 this lane's 8 elements of a 16 x 32 one
        const int hoff = G == 16 ? (ls >> 1) * 512 + (ls & 1) * 256 + lq * 8 : lane * 8;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
#pragma unroll
            for (int c = 0; c < NKG; ++c) num[c][dt] = zero;
#pragma unroll
            for (int st = 0; st < NS; ++st) {
                const int idx = G == 16 ? ((dt >> 1) * (D / 16) + st * 2) * 512 + (dt & 1) * 128 : (dt * NS + st) * 512;
                Frag5 hi;
                hi.v = *reinterpret_cast<const bf16x8 *>(Kb + hoff + idx);
#pragma unroll
                for (int c = 0; c < NKG; ++c) num[c][dt] = product(hi, qf[u0 + c][st], num[c][dt]);
            }
        }
    }
    if (!DBG) {
        // bf16 results leave through LDS so that every global store is a run of full 256-byte rows: accumulator
        // layout (lane = query lq of a group; 4 consecutive columns per (dt, g4, ls)) -> half of a free tile of this set's own
        // (K slots 2..4, behind the state, and the V slot after the last block's: nobody reads them any more), 16-byte chunk c of row r at
        // r * 256 + ((c ^ (r & 15)) << 4) -> row layout (4 rows x 16 chunks per instruction).
        int vs = v_last + 1;
        if (vs >= NV) vs -= NV;
        u16 *free_tile = unit < 6 ? Kb + (2 + (unit >> 1)) * TILE : Vb + vs * TILE;
        constexpr int ROWB = D * 2;          // bytes of a row
        unsigned char *stg = reinterpret_cast<unsigned char *>(free_tile) + (unit & 1) * (32 * ROWB);
        auto stage = [&](int c, int dt, int g4, const float (&v)[4]) INL {       // columns dt G + 8 g4 + 4 ls .. + 3 of query lq of group c
            uint2 pk;
            pk.x = pack2e(v[0], v[1]);
            pk.y = pack2e(v[2], v[3]);
            const int row = c * G + lq;
            *reinterpret_cast<uint2 *>(stg + row * ROWB + (((dt * (G / 8) + g4 + (ls >> 1)) ^ oswz(row)) << 4) + (ls & 1) * 8) = pk;
        };
#pragma unroll
        for (int c = 0; c < NKG; ++c)
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                for (int g4 = 0; g4 < AR / 4; ++g4) {
                    float ov[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float os = o[u0 + c][dt][g4 * 4 + t] * inv_l[c];
                        ov[t] = lin && !EMIT ? fmaf(num[c][dt][g4 * 4 + t], lin_scale[u0 + c], os) : os;
                    }
                    stage(c, dt, g4, ov);
                }
        asm volatile("" ::: "memory");       // the wave's LDS operations execute in order
        // destination of row r: the stored row (or the pair slot) of the lane that owns query r
        bool valid = valid0;
        const int qrow = TIGHT ? query_row(u, l32, valid) : row0, dest_mine = !valid ? -1 : GATHER ? g_slot0 + qrow : qrow;
        constexpr int RPI = 64 / CH;          // rows per store instruction (4 rows x 16 chunks, or 8 x 8)
        const int r4 = lane / CH, c16 = lane % CH;
        u16 *dbase = GATHER ? a.g_po + (size_t)bh * N * a.g_kk * D : reinterpret_cast<u16 *>(a.out) + (size_t)bh * N * D;
#pragma unroll
        for (int i = 0; i < 32 / RPI; ++i) {
            const int r = RPI * i + r4;
            const uint4 v = *reinterpret_cast<const uint4 *>(stg + r * ROWB + ((c16 ^ oswz(r)) << 4));
            const int dest = __shfl(dest_mine, r);
            if (dest >= 0) *reinterpret_cast<uint4 *>(dbase + (size_t)dest * D + c16 * 8) = v;
        }
        if (EMIT && lin) {
            // the unscaled linear branch, for the full projection: through the same staging into 16-byte pieces of the lane's own row, the
            // order that the projection's operand wants (blocks of 32 stored rows x 128 channels, piece c of row r at
            // (c / 2 * 64 + c % 2 * 32 + r) * 16 bytes; whole kilobytes for a head in the stored order)
            asm volatile("" ::: "memory");
#pragma unroll
            for (int c = 0; c < NKG; ++c)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int g4 = 0; g4 < AR / 4; ++g4) {
                        float ol[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) ol[t] = num[c][dt][g4 * 4 + t] * inv_den[u0 + c];
                        stage(c, dt, g4, ol);
                    }
            asm volatile("" ::: "memory");
            u16 *blk = a.emit_ol + ((((size_t)smp * ((N + 31) >> 5) + (qrow >> 5)) * a.H + h) << 12) + (hh * 32 + (qrow & 31)) * 8;
#pragma unroll
            for (int i = 0; i < CH / 2; ++i) {
                const uint4 v = *reinterpret_cast<const uint4 *>(stg + l32 * ROWB + (((2 * i + hh) ^ oswz(l32)) << 4));
                if (valid) *reinterpret_cast<uint4 *>(blk + i * 512) = v;
            }
        }
        if (GATHER && valid && hh == 0) a.g_lse[(size_t)bh * N * a.g_kk + g_slot0 + qrow] = l_run[u] > 0.f ? m_run[u] + log2f(l_run[u]) : -INFINITY;
    } else {
#pragma unroll
        for (int c = 0; c < NKG; ++c) {
            bool valid;
            const int mine = TIGHT ? query_row(u, c * G + lq, valid) : __shfl(valid0 ? row0 : -1, c * G + lq);
            if (TIGHT ? valid : mine >= 0) {
                const size_t obase = ((size_t)bh * N + mine) * D;
                u16 *outp = reinterpret_cast<u16 *>(a.out) + obase;
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int g4 = 0; g4 < AR / 4; ++g4) {
                        const int col = dt * G + 8 * g4 + 4 * ls;
                        float os[4], ol[4], ov[4];
#pragma unroll
                        for (int t = 0; t < 4; ++t) {
                            os[t] = o[u0 + c][dt][g4 * 4 + t] * inv_l[c];
                            ol[t] = lin ? num[c][dt][g4 * 4 + t] : 0.f;
                            ov[t] = lin ? fmaf(ol[t], lin_scale[u0 + c], os[t]) : os[t];
                        }
                        uint2 pk;
                        pk.x = pack2e(ov[0], ov[1]);
                        pk.y = pack2e(ov[2], ov[3]);
                        *reinterpret_cast<uint2 *>(outp + col) = pk;
                        if (DBG && a.o_sparse_dbg)
                            *reinterpret_cast<float4 *>(a.o_sparse_dbg + obase + col) = make_float4(os[0], os[1], os[2], os[3]);
                        if (DBG && a.o_linear_dbg && lin)
                            *reinterpret_cast<float4 *>(a.o_linear_dbg + obase + col) =
                                make_float4(ol[0] * inv_den[u0 + c], ol[1] * inv_den[u0 + c], ol[2] * inv_den[u0 + c], ol[3] * inv_den[u0 + c]);
                    }
            }
        }
    }
    }
    };
    if constexpr (BOTH) {
        static_assert(long_list(D) >= LOOKED_AT, "a list has the entries that are looked at");
        const bool smaller = a.many && n >= long_list(D) && !(SPLIT && L >= a.sp_full) && 8 * kept_bits >= 5 * LOOKED_AT * min(4, nb - tile * 4);
        // the hint is for the registers and the order of the code: 480p dense without it 5262, with it 5215 us
        if (__builtin_expect(smaller, 1)) {
            if constexpr (!SPLIT || QS == 1) {
                rest(std::integral_constant<int, 16>{}, std::true_type{});
            } else if constexpr (DBG) {          // the same results, and one copy
                rest(std::integral_constant<int, 16>{}, std::false_type{});
            } else {
                if (turns) rest(std::integral_constant<int, 16>{}, std::true_type{});
                else rest(std::integral_constant<int, 16>{}, std::false_type{});
            }
        } else {
            rest(std::integral_constant<int, 32>{}, std::false_type{});
        }
    } else {
        rest(std::integral_constant<int, 32>{}, std::false_type{});
    }
}

// Sets of 32 queries of a wave (the kernel's QS): 2 at d = 64 where there are more tiles than compute units and two workgroups' LDS fits one.
// Up to half a round more than that, with 32 queries a wave the rest is cut in two or more and pairs of tiles on one unit are avoided: 64
// queries a wave against that take 98 % at 12 entries, 100 at 20, 106 at 32, 109 to 117 at 50, 124 at 104 (260 to 350 tiles).  A list holds
// at most nb entries, so with few of them 64 queries stay (280 tiles of 28 blocks: 96 to 101 %).
static int query_sets(int d, int nb, long long tiles)
{
    return d == 64 && tiles > (nb > 28 ? 384 : 256) && 2 * (v5_ring_bytes(d) + tile_list_cap(nb) * 4) <= V5_MAX_DYN ? 2 : 1;
}

SplitPlan split_plan(int BH, int nb, int d)
{
    // One workgroup per compute unit runs at a time, 256 in all, or two.  Whole rounds of tiles stay as they are; the rest, if it leaves
    // at least half of the chip idle, is cut into as many pieces as there is room for.
    // Layer call before -> after: 49 tiles of 12 heads (512 + 76 workgroups, 52 entries) 300 -> 269 us; 44 tiles, 42 entries, dense
    // 79 -> 46; 184 tiles of 2 x 12 heads 675 -> 629; 25 tiles of 5 heads 64 -> 55.  A list of 11 entries cut in two gained nothing
    // (37.4 -> 38.5), hence SPLIT_MIN_ENTRIES; with it calls that are not cut measure the same as before.
    const long long total = (long long)BH * ((nb + 3) / 4);
    const int round = 256 * query_sets(d, nb, total);
    SplitPlan p{};
    p.full = (int)(total / round * round);
    p.rest = (int)(total - p.full);
    p.pieces = p.rest ? round / p.rest : 1;
    if (p.pieces > SPLIT_MAX_PIECES) p.pieces = SPLIT_MAX_PIECES;
    p.cut = p.pieces > 1 && nb >= 2 * SPLIT_MIN_ENTRIES;
    if (p.cut && p.pieces > nb / SPLIT_MIN_ENTRIES) p.pieces = nb / SPLIT_MIN_ENTRIES;      // no list has entries for more
    if (!p.cut) p.pieces = p.pieces > 1 && round == 256 ? 2 : 1;      // no list of this length is cut, but rows can be dealt to two workgroups
    return p;
}

RidePlan ride_plan(int B, int H, int N, int d, const SplitPlan &split)
{
    // Where all tiles fit one round and riders, who read 192 bytes a token at some 30 GB/s, are not much later than the tiles come to their epilogues.
    // Layer calls, three launches -> one (us): 12 heads, N = 256 19.2 -> 11.5, 1024 23.8 -> 14.1, 1950 29.8 -> 24.8, 3000 32.4 -> 24.6, dense 83.7 -> 74.0;
    // 8 heads, N = 5200 37.2 -> 27.5, 6400 41.3 -> 43.2, dense 167 -> 171; 2 heads, N = 4000 32.0 -> 24.8, 9000 35.7 -> 39.0;
    // 40 heads, N = 256 31.6 -> 18.9, 1000 37.6 -> 25.2, 1500 42.7 -> 37.2; 64 heads, N = 512
    // 44.6 -> 35.4, 1000 (768 riders and tiles) 53.8 -> 53.7; 24 heads of 64, N = 1000 20.2 -> 13.8, 40 heads of 64, N = 512 20.2 -> 13.3.
    RidePlan p{};
    const int BH = B * H, nparts = gate_num_parts(N);
    const long long slices = (long long)BH * slices_per_head(d);
    if (N > 5400 || split.full || slices + split.rest > 640 || query_sets(d, (N + 63) / 64, split.rest) != 1) return p;
    // 32 shares of the gate, or 16 at the least where that gives every workgroup with work a compute unit: those of tiles dealt by rows, or else of
    // whole tiles (12 heads, N = 1500: 17.0 us with 16 and rows, 19.8 with 32 and whole tiles; 24 heads of 64, N = 1950: 18.7 and 24.5)
    int shares = 256 - (int)slices - 2 * split.rest;
    if (shares < 16) shares = 256 - (int)slices - split.rest;
    if (shares < 16 || shares > 32) shares = 32;
    p.gate_tasks = shares / B < 1 ? 1 : shares / B;
    if (p.gate_tasks > (nparts + 1) / 2) p.gate_tasks = (nparts + 1) / 2;
    const int riders = (int)slices + B * p.gate_tasks;
    p.wgs = (riders + 7) & ~7;
    p.crowded = p.wgs + 2 * split.rest > 256 && p.wgs + split.rest <= 256;
    return p;
}

template <bool DBG, int MODE = 0, bool ROPE = false, int D = 128, bool SPLIT = false, int QS = 1, bool EMIT = false, bool RIDE = false>
static hipError_t launch_v5(const AttnArgs &a, hipStream_t st)
{
    const int ntiles = (a.nb + 3) / 4;
    const int total = MODE == 2 ? a.g_max_tiles : a.B * a.H * ntiles;
    const int per_xcd = (total + 7) / 8;
    if (!large_tile_list_fits(D, a.nb)) return hipErrorInvalidValue;
    const int list_cap = tile_list_cap(a.nb);
    const size_t lds = v5_ring_bytes(D) + (size_t)list_cap * 4;
    auto kern = sparse_attn_v5_kernel<D, DBG, MODE, ROPE, SPLIT, QS, EMIT, RIDE>;
    static bool attr_done[16] = {};
    if (hipError_t e = dyn_lds_attr_once(reinterpret_cast<const void *>(kern), V5_MAX_DYN, attr_done); e != hipSuccess) return e;
    const int px = SPLIT ? ((total - a.sp_full) * a.sp_pieces + 7) / 8 : 0;      // pieces of an XCD
    auto magic = [](int d) { return d > 1 ? (unsigned)((1ull << 32) / (unsigned)d) : ~0u; };
    AttnArgs b = a;
    b.many = total > 256;
    b.tiles_magic = magic(ntiles); b.heads_magic = magic(a.H); b.pieces_magic = magic(a.sp_pieces);
    if (SPLIT) {
        b.sp_alone = 256 / (total - a.sp_full);
        b.sp_rows = (px + a.sp_pieces - 1) / a.sp_pieces; b.rows_magic = magic(b.sp_rows);
    }
    const int grid = SPLIT ? a.sp_full + (QS == 2 || RIDE ? b.sp_rows * a.sp_pieces : px) * 8 : per_xcd * 8;
    launch_kernel(kern, dim3(grid + (RIDE ? a.ride.wgs : 0)), dim3(512 / QS), lds, st, b, ntiles, total, per_xcd, list_cap);
    return take_launch_status();
}

hipError_t launch_sparse_attn_v5(const AttnArgs &a, hipStream_t st)
{
    const bool dbg = a.o_sparse_dbg || a.o_linear_dbg, split = a.sp_pieces > 1 && !a.g_desc && !a.topk_mask;
    if (a.D == 64) {
        if (a.g_desc || a.topk_mask || a.rope_tab) return hipErrorInvalidValue;
        if (query_sets(64, a.nb, (long long)a.B * a.H * ((a.nb + 3) / 4)) == 2) {
            if (split) return dbg ? launch_v5<true, 0, false, 64, true, 2>(a, st) : launch_v5<false, 0, false, 64, true, 2>(a, st);
            return dbg ? launch_v5<true, 0, false, 64, false, 2>(a, st) : launch_v5<false, 0, false, 64, false, 2>(a, st);
        }
        if (a.ride.wgs && split) return dbg ? launch_v5<true, 0, false, 64, true, 1, false, true>(a, st) : launch_v5<false, 0, false, 64, true, 1, false, true>(a, st);
        if (a.ride.wgs) return dbg ? launch_v5<true, 0, false, 64, false, 1, false, true>(a, st) : launch_v5<false, 0, false, 64, false, 1, false, true>(a, st);
        if (split) return dbg ? launch_v5<true, 0, false, 64, true>(a, st) : launch_v5<false, 0, false, 64, true>(a, st);
        return dbg ? launch_v5<true, 0, false, 64>(a, st) : launch_v5<false, 0, false, 64>(a, st);
    }
    if (a.g_desc) return launch_v5<false, 2>(a, st);
    if (a.topk_mask) return dbg ? launch_v5<true, 1>(a, st) : launch_v5<false, 1>(a, st);
    if (a.ride.wgs) {
        if (a.emit_ol && (dbg || a.rope_tab)) return hipErrorInvalidValue;
        if (a.emit_ol) return split ? launch_v5<false, 0, false, 128, true, 1, true, true>(a, st) : launch_v5<false, 0, false, 128, false, 1, true, true>(a, st);
        if (a.rope_tab && split) return dbg ? launch_v5<true, 0, true, 128, true, 1, false, true>(a, st) : launch_v5<false, 0, true, 128, true, 1, false, true>(a, st);
        if (a.rope_tab) return dbg ? launch_v5<true, 0, true, 128, false, 1, false, true>(a, st) : launch_v5<false, 0, true, 128, false, 1, false, true>(a, st);
        if (split) return dbg ? launch_v5<true, 0, false, 128, true, 1, false, true>(a, st) : launch_v5<false, 0, false, 128, true, 1, false, true>(a, st);
        return dbg ? launch_v5<true, 0, false, 128, false, 1, false, true>(a, st) : launch_v5<false, 0, false, 128, false, 1, false, true>(a, st);
    }
    if (a.emit_ol) {
        if (dbg || a.rope_tab) return hipErrorInvalidValue;
        return split ? launch_v5<false, 0, false, 128, true, 1, true>(a, st) : launch_v5<false, 0, false, 128, false, 1, true>(a, st);
    }
    if (split && a.rope_tab) return dbg ? launch_v5<true, 0, true, 128, true>(a, st) : launch_v5<false, 0, true, 128, true>(a, st);
    if (split) return dbg ? launch_v5<true, 0, false, 128, true>(a, st) : launch_v5<false, 0, false, 128, true>(a, st);
    if (a.rope_tab) return dbg ? launch_v5<true, 0, true>(a, st) : launch_v5<false, 0, true>(a, st);
    return dbg ? launch_v5<true>(a, st) : launch_v5<false>(a, st);
}

}  // namespace salad
