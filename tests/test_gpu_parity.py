"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded
inputs.  Integer work (the mask) must match bit for bit; floating point within max-abs 2e-2 and
relative L2 5e-3 (bf16 inputs, fp32 accumulation), per branch and combined."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2601_16515_amd import binding as sb
from paper_2601_16515_amd import workloads as wl
from tests.gpu_util import MAX_ABS, REL_L2, compare_layer, errors, gather_rows, run_layer, say, to_dev, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    assert torch.cuda.is_available(), "these tests need the MI355X"
    sb.lib()   # fails loudly if libsalad.so is missing


# --------------------------------------------------------------------------------------------- mask

@pytest.mark.parametrize("grid,kept", [
    ((4, 16, 16), [4, 4]), ((5, 6, 9), [1, 5, 3]), ((8, 30, 52), [49] * 12), ((21, 30, 52), [51] * 12),
    ((21, 30, 52), [512, 1, 26, 256]), ((1, 1, 1), [1]), ((21, 45, 80), [118] * 40),
])
def test_block_mask_bit_exact(oracle, grid, kept):
    say(f"mask grid={grid} kept[0]={kept[0]} H={len(kept)}")
    row_ptr, col_idx = sb.salad_block_mask(*grid, 64, kept)
    torch.cuda.synchronize()
    rp, ci = oracle.block_mask(*grid, 64, kept)
    assert np.array_equal(row_ptr.cpu().numpy(), rp)
    assert np.array_equal(col_idx.cpu().numpy(), ci)


@pytest.mark.parametrize("grid,kept", [
    ((4, 16, 16), [4, 5]), ((5, 6, 9), [1, 5, 3]), ((21, 30, 52), [51] * 12), ((21, 30, 52), [512, 1, 26, 255]),
    ((1, 1, 1), [1]), ((21, 45, 80), [118] * 40),
])
def test_block_mask_truncated_bit_exact(oracle, grid, kept):
    """The window cut at the sequence ends (rows of different lengths, first entries in closed form) against the oracle."""
    say(f"truncated mask grid={grid} kept[0]={kept[0]} H={len(kept)}")
    row_ptr, col_idx = sb.salad_block_mask_mode(*grid, 64, kept, sb.SALAD_WINDOW_TRUNCATED)
    torch.cuda.synchronize()
    rp, ci = oracle.block_mask(*grid, 64, kept, truncated=True)
    assert np.array_equal(row_ptr.cpu().numpy(), rp)
    assert np.array_equal(col_idx.cpu().numpy(), ci)
    assert sb.salad_block_mask_nnz_mode(*grid, 64, kept, sb.SALAD_WINDOW_TRUNCATED) == len(ci)
    same = sb.salad_block_mask_mode(*grid, 64, kept, sb.SALAD_WINDOW_SHIFTED)
    ref = sb.salad_block_mask(*grid, 64, kept)
    assert torch.equal(same[0], ref[0]) and torch.equal(same[1], ref[1])


def test_layer_with_truncated_window(oracle):
    """The layer on the truncated-window mask built on the device (short rows at both ends of every head, both head
    orders, prebuilt visit lists) against the oracle on its own truncated mask."""
    w = SMALL[7]                                      # N = 1170: 19 blocks, 3 heads
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4, 7, 5]
    row_ptr, col_idx = sb.salad_block_mask_mode(w.T, w.Hh, w.W, 64, kept, sb.SALAD_WINDOW_TRUNCATED)
    csr = (row_ptr.cpu().numpy(), col_idx.cpu().numpy())
    ref = _oracle_layer(oracle, w, inp, kept, kinds, truncated=True)
    assert np.array_equal(csr[0], ref["row_ptr"]) and np.array_equal(csr[1], ref["col_idx"])
    res = run_layer(w, inp, dev, kept, kinds, csr=csr)
    compare_layer(res, ref, label="truncated window")
    fast = run_layer(w, inp, dev, kept, kinds, csr=csr, dbg=False, prebuilt_lists=True)
    assert np.array_equal(fast["out"], res["out"])


# --------------------------------------------------------------------------------------------- gate

@pytest.mark.parametrize("B,N,D,dtype", [(1, 1024, 128, "f32"), (2, 270, 1536, "bf16"), (1, 4099, 5120, "bf16"),
                                         (3, 7, 64, "bf16"), (1, 1, 8, "f32"), (1, 12480, 1536, "bf16"),
                                         (2, 1031, 8192, "bf16"), (1, 300, 6152, "bf16"), (1, 77, 8192, "f32")])
def test_gate_parity(oracle, B, N, D, dtype):
    say(f"gate B={B} N={N} D={D} {dtype}")
    x = wl.normal(50, "x", (B, N, D))
    if dtype == "bf16":
        x = wl.round_to_bf16(x)
    wg = wl.normal(50, "w", (D,), std=0.05)
    for bias in (0.0, 0.7):
        s = sb.salad_gate_fwd(to_dev(x, dtype), torch.from_numpy(wg).cuda(), bias)
        torch.cuda.synchronize()
        ref = oracle.gate(x, wg, bias)
        assert np.abs(s.cpu().numpy().astype(np.float64) - ref).max() < 2e-6


# ------------------------------------------------------------------------------------- linear state

@pytest.mark.parametrize("B,H,N,d,dtype", [(1, 2, 270, 128, "bf16"), (2, 3, 1000, 128, "bf16"), (1, 2, 777, 64, "bf16"),
                                           (1, 1, 64, 128, "bf16"), (1, 1, 5, 64, "bf16"), (1, 2, 300, 64, "f32"),
                                           (1, 12, 12480, 128, "bf16")])
def test_linear_state_parity(oracle, B, H, N, d, dtype):
    say(f"state B={B} H={H} N={N} d={d} {dtype}")
    k = wl.normal(60, "k", (B, H, N, d))
    v = wl.normal(60, "v", (B, H, N, d))
    if dtype == "bf16":
        k, v = wl.round_to_bf16(k), wl.round_to_bf16(v)
    Hs, Z = sb.salad_linear_state_fwd(to_dev(k, dtype), to_dev(v, dtype))
    torch.cuda.synchronize()
    rH, rZ = oracle.linear_state(k, v)
    aH, eH = errors(Hs.cpu().numpy().astype(np.float64), rH)
    aZ, eZ = errors(Z.cpu().numpy().astype(np.float64), rZ)
    say(f"  Hs rel_l2={eH:.3e} Z rel_l2={eZ:.3e}")
    assert eH < 2e-6 and eZ < 2e-6          # exact bf16 products, fp32 accumulation


def test_linear_state_chunking_does_not_change_result(oracle):
    """Different numbers of token chunks (workgroups) only change the fp32 summation order."""
    k = wl.round_to_bf16(wl.normal(61, "k", (1, 2, 2000, 128)))
    v = wl.round_to_bf16(wl.normal(61, "v", (1, 2, 2000, 128)))
    rH, rZ = oracle.linear_state(k, v)
    try:
        for wgs in (2, 7, 64, 4096):
            sb.salad_tune("state_wgs", wgs)
            Hs, Z = sb.salad_linear_state_fwd(to_dev(k, "bf16"), to_dev(v, "bf16"))
            torch.cuda.synchronize()
            assert errors(Hs.cpu().numpy().astype(np.float64), rH)[1] < 2e-6
            assert errors(Z.cpu().numpy().astype(np.float64), rZ)[1] < 2e-6
    finally:
        sb.salad_tune("state_wgs", 256)


# -------------------------------------------------------------------------------------- whole layer

def _oracle_layer(oracle, w, inp, kept, kinds, sel=None, **kw):
    return oracle.salad_forward(inp["q"], inp["k"], inp["v"], inp["x_t"], inp["w_gate"], inp["head_scale"],
                                grid=(w.T, w.Hh, w.W), block=w.block, head_kind=kinds, kept=kept,
                                lam=kw.pop("lam", w.lam), eps=kw.pop("eps", w.eps), sel=sel, **kw)


SMALL = [
    wl.small("tail14-d128", 1, 2, 128, 5, 6, 9, "bf16", 0.5, seed=101),      # N=270: 5 blocks, 14-token tail
    wl.small("odd-blocks-d128", 2, 3, 128, 7, 9, 11, "bf16", 0.6, seed=102),  # N=693: 11 blocks, tail 53, B=2
    wl.small("d64", 1, 4, 64, 6, 10, 10, "bf16", 0.7, seed=103),              # N=600: 10 blocks, tail 24
    wl.small("one-block", 1, 2, 128, 2, 3, 5, "bf16", 0.0, seed=104),         # N=30 < one block
    wl.small("exact-blocks", 1, 2, 128, 4, 8, 16, "bf16", 0.75, seed=105),    # N=512, no tail
    wl.small("T-gt-block", 1, 2, 128, 70, 3, 2, "bf16", 0.5, seed=106),       # T=70 > 64: a location spans blocks
    wl.small("single-token", 1, 1, 128, 1, 1, 1, "bf16", 0.0, seed=109),      # N=1
    wl.small("five-tiles-d128", 1, 3, 128, 9, 10, 13, "bf16", 0.8, seed=110), # N=1170: 19 blocks = 5 tiles of 4, tail 18
    wl.small("d64-ragged", 2, 2, 64, 3, 11, 13, "bf16", 0.5, seed=111),       # N=429, d=64, B=2
    wl.small("d64-one-block", 1, 3, 64, 2, 3, 5, "bf16", 0.0, seed=114),      # N=30 < one block, d=64
    wl.small("d64-single-token", 2, 1, 64, 1, 1, 1, "bf16", 0.0, seed=115),   # N=1, d=64, B=2
    wl.small("d64-T-gt-block", 1, 2, 64, 70, 3, 3, "bf16", 0.5, seed=116),    # d=64, T=70 > 64: temporal rows far apart
]


@pytest.mark.parametrize("w", SMALL, ids=lambda w: w.name)
def test_layer_parity_small_bf16(oracle, w):
    say(f"layer {w.name} N={w.N} nb={w.nb}")
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    k = sb.salad_kept_from_sparsity(w.nb, w.sparsity)
    kept = [max(1, min(w.nb, k + (h % 2))) for h in range(w.H)]      # heads differ in window size
    res = run_layer(w, inp, dev, kept, kinds)
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    assert np.array_equal(res["row_ptr"], ref["row_ptr"]) and np.array_equal(res["col_idx"], ref["col_idx"])
    assert np.abs(res["s"] - ref["s"]).max() < 2e-6
    compare_layer(res, ref, label=w.name)


def test_layer_parity_tiny_config_fp32(oracle):
    w = wl.TINY
    say(f"layer {w.name} (fp32) N={w.N}")
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [sb.salad_kept_from_sparsity(w.nb, w.sparsity)] * w.H
    assert kept == [4, 4]
    res = run_layer(w, inp, dev, kept, kinds)
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    assert np.array_equal(res["col_idx"], ref["col_idx"])
    compare_layer(res, ref, tol_abs=1e-4, tol_rel=1e-5, label="tiny-f32")


def test_fp32_path_ragged_d128(oracle):
    w = wl.small("f32-d128", 1, 2, 128, 3, 7, 9, "f32", 0.4, seed=107)       # N=189
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [2, 3]
    res = run_layer(w, inp, dev, kept, kinds)
    compare_layer(res, _oracle_layer(oracle, w, inp, kept, kinds), tol_abs=1e-4, tol_rel=1e-5, label="f32-d128")


@pytest.mark.parametrize("B,H,d,grid,kept", [
    (1, 1, 64, (1, 1, 1), [1]),              # one token: 15 of a tile's 16 queries and 31 of a unit's 32 keys do not exist
    (1, 2, 64, (3, 1, 5), [1, 1]),           # 15 tokens, temporal head
    (2, 3, 64, (1, 1, 17), [1, 1, 1]),       # second tile of 1 query
    (1, 2, 128, (5, 13, 1), [2, 1]),         # 65 tokens: a block of one key, its second half empty
    (1, 2, 64, (4, 5, 8), [3, 2]),           # 160 tokens, 32-token tail: units of a row do not divide by the 4 waves
    (1, 2, 128, (7, 9, 11), [5, 11]),        # 693 tokens: every block kept by the second head
])
def test_fp32_tile_edges(oracle, B, H, d, grid, kept):
    """fp32 kernels at the edges of their 16-query tiles, 32-key units and 4-token groups."""
    w = wl.small(f"f32-{d}-{grid[0] * grid[1] * grid[2]}", B, H, d, *grid, "f32", 0.5, seed=300 + d + grid[2])
    inp = wl.make_inputs(w)
    kinds = wl.head_kinds(w)
    res = run_layer(w, inp, upload(w, inp), kept, kinds)
    compare_layer(res, _oracle_layer(oracle, w, inp, kept, kinds), tol_abs=1e-4, tol_rel=1e-5, label=w.name)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid,kept", [
    ((1, 1, 40), [1, 1]),                        # one block, both halves of it partly past the end
    ((2, 7, 5), [1, 2]),                         # 70 tokens: the tail block has 6 keys, its second half none
    ((3, 5, 13), [1, 2, 3, 4]),                  # 195 tokens, 4 blocks
    ((3, 13, 14), [1, 2, 3, 4, 5, 6, 7, 8, 9]),  # 546 tokens, 9 blocks: lists of 4 to 9 entries, around the 4 blocks fetched ahead
    ((5, 28, 31), [61, 62, 66, 68]),             # 4340 tokens, 68 blocks: lists of 64 and more entries, read in chunks of 64
])
def test_visit_list_lengths(oracle, d, grid, kept):
    """The attention kernel's pipeline at the ends of its visit lists: fewer entries than it fetches ahead, the wait at the
    last ones, the second chunk of a list, blocks without keys in their second half; both head orders, bf16."""
    w = wl.small(f"lists-{d}-{grid[0] * grid[1] * grid[2]}", 1, len(kept), d, *grid, "bf16", 0.5, seed=400 + d + grid[2])
    inp = wl.make_inputs(w)
    kinds = wl.head_kinds(w)
    for dbg in (True, False):
        res = run_layer(w, inp, upload(w, inp), kept, kinds, dbg=dbg)
        compare_layer(res, _oracle_layer(oracle, w, inp, kept, kinds), label=w.name)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("grid", [(2, 11, 13), (15, 4, 5), (63, 3, 5), (64, 3, 4), (65, 3, 5), (130, 2, 3)])
def test_time_axis_wraps_inside_a_block(oracle, d, grid):
    """Rows of a temporal head's block are found from its first row and a lane's own offset, which wraps the time axis at most
    once when the axis is longer than the 16 rows of a load and many times over the block when it is shorter."""
    w = wl.small(f"wrap-{d}-{grid}", 1, 2, d, *grid, "bf16", 0.5, seed=900 + d + grid[0])
    inp = wl.make_inputs(w)
    kept = [3, 3]
    for dbg in (True, False):
        res = run_layer(w, inp, upload(w, inp), kept, [1, 1], dbg=dbg)
        compare_layer(res, _oracle_layer(oracle, w, inp, kept, [1, 1]), label=w.name)


@pytest.mark.parametrize("B,H,grid,keep", [
    (1, 64, (3, 16, 17), 5),      # 256 tiles: 32 queries a wave
    (1, 43, (4, 17, 19), 9),      # 258 tiles: 64 queries a wave, one round, the last tile of a head with one block of 12 keys
    (1, 43, (4, 16, 29), 20),     # 344 tiles of 29 blocks: 32 queries a wave, 88 tiles cut in two
    (1, 43, (4, 16, 28), 20),     # of 28 blocks: 64 queries a wave
    (2, 64, (3, 13, 14), 2),      # 384 tiles, lists shorter than the blocks fetched ahead
    (3, 43, (3, 16, 17), 13),     # 516 tiles: the last four have room for 8 pieces each, and lists for one or two
    (1, 62, (6, 18, 21), 8),      # 558 tiles, 46 of them with room for 5 pieces: an XCD's run of pieces starts in the middle of a tile and ends short
    (1, 64, (3, 29, 32), 4),      # 704 tiles, 192 with room for two, lists too short to be cut
    (1, 53, (3, 37, 25), 30),     # 583 tiles, 71 with room for 7, of which 3 have a compute unit each
    (1, 55, (4, 24, 32), 40),     # 660 tiles, 148 cut in three that share units, but for those whose lists are short
])
def test_d64_sixty_four_queries_a_wave(oracle, B, H, grid, keep):
    """d = 64 around the number of tiles from which on a wave owns 64 queries; both head orders, guided batches, cut tiles."""
    w = wl.small(f"d64-{B}-{H}-{grid}", B, H, 64, *grid, "bf16", 0.5, seed=950 + H)
    inp = wl.make_inputs(w)
    kinds, kept = wl.head_kinds(w), [keep] * H
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    for dbg in (True, False):
        compare_layer(run_layer(w, inp, upload(w, inp), kept, kinds, dbg=dbg), ref, label=w.name)


@pytest.mark.parametrize("B,H,d,grid,kept", [
    (1, 3, 128, (5, 13, 17), [18, 5, 13]),       # 15 tiles in up to 8 pieces; lists of 18 (3 pieces), 8 (whole) and 16 (2 pieces) entries
    (2, 2, 64, (3, 29, 31), [43, 30]),           # 44 tiles in 5 pieces, the last tile of 3 blocks
    (1, 1, 128, (1, 7, 110), [13]),              # 13 blocks: the shortest list that is cut, one head, spatial
    (1, 64, 64, (2, 17, 32), [9 + h % 9 for h in range(64)]),   # 320 tiles: a whole round of 256, then 64 in 4 pieces
])
def test_last_round_cut_into_pieces(oracle, B, H, d, grid, kept):
    """Tiles of the last, partial round cut along their visit lists: against the oracle, the same bits on every call (whichever
    piece comes last combines them) on a workspace that held anything, with and without the linear branch."""
    w = wl.small(f"cut-{d}-{grid[0] * grid[1] * grid[2]}", B, H, d, *grid, "bf16", 0.5, seed=600 + d + grid[2])
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    res = run_layer(w, inp, dev, kept, kinds)
    compare_layer(res, _oracle_layer(oracle, w, inp, kept, kinds), label=w.name)
    row_ptr, col_idx = sb.salad_block_mask(w.T, w.Hh, w.W, w.block, kept)
    ws = sb.Workspace(B, H, w.N, d, sb.SALAD_BF16)
    ws.buf.fill_(0x5a)                           # the counters start from whatever the memory holds
    outs = {}
    for i in range(8):
        lam = 0.0 if i % 2 else w.lam
        out = sb.salad_sparse_linear_attn_fwd(dev["q"], dev["k"], dev["v"], grid, row_ptr, col_idx, kinds, lam=lam, head_scale=dev["head_scale"],
                                              x_t=dev["x_t"], w_gate=dev["w_gate"], eps=w.eps, workspace=ws)
        assert torch.equal(out, outs.setdefault(lam, out))
    assert torch.equal(outs[w.lam], res["out_t"])
    assert errors(outs[0.0].double().cpu().numpy(), res["o_sparse"])[1] < 4e-3      # one bf16 rounding (2^-9) of each value


@pytest.mark.parametrize("B,H,d,grid,keep", [
    (1, 2, 128, (1, 1, 40), 1),       # one row of 40 tokens: the second workgroup of the tile has no rows
    (1, 3, 64, (2, 7, 9), 2),         # 2 rows, the second of 62 tokens
    (2, 3, 128, (3, 5, 13), 3),       # 4 rows, the last of 3 tokens: alone in its workgroup with the third
    (1, 12, 128, (5, 15, 26), 8),     # 31 rows, lists of 8 to 11 entries
    (1, 12, 128, (5, 15, 26), 25),    # lists of 25 to 28: two pieces would not pay
    (1, 4, 128, (5, 15, 26), 9),      # lists of 9 to 12: room for 8 pieces, worth 2
    (1, 12, 128, (5, 15, 26), 31),    # lists of 31: two pieces do pay
    (1, 4, 64, (3, 13, 14), 9),       # all of 9 blocks
    (3, 43, 128, (3, 16, 17), 3),     # 512 whole tiles, four dealt by rows
])
def test_rows_of_a_tile_dealt_to_two_workgroups(oracle, B, H, d, grid, keep):
    """Tiles beyond a full round whose lists are too short to be cut; both head orders."""
    w = wl.small(f"rows-{d}-{grid}", B, H, d, *grid, "bf16", 0.5, seed=970 + H)
    inp = wl.make_inputs(w)
    kinds, kept = wl.head_kinds(w), [keep] * H
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    for dbg in (True, False):
        compare_layer(run_layer(w, inp, upload(w, inp), kept, kinds, dbg=dbg), ref, label=w.name)


@pytest.mark.parametrize("d", [64, 128])
def test_cut_tiles_with_the_options_of_the_call(oracle, d):
    """Lists that are cut (18 and 13 to 16 entries: 3 and 2 pieces) together with what the call can be asked for: branch dropping,
    the rotary linear branch with and without debug outputs, prebuilt lists, a CSR with empty rows and lists of every length, and
    replays of a captured graph; always on one workspace that first holds anything and then the last call's leavings."""
    w = wl.small(f"cut-options-{d}", 2, 2, d, 5, 13, 17, "bf16", 0.5, seed=650 + d)      # N = 1105: 20 tiles in up to 8 pieces
    inp = wl.make_inputs(w)
    wg = inp["w_gate"]
    inp["x_t"] = inp["x_t"].copy()
    inp["x_t"][1] = wl.round_to_bf16(inp["x_t"][1] + (2.0 * wg / float(np.dot(wg, wg))).astype(np.float32))   # pre-activations of sample 1 up by ~2
    dev = upload(w, inp)
    kinds, kept = wl.head_kinds(w), [18, 13]
    ws = sb.Workspace(w.B, w.H, w.N, d, sb.SALAD_BF16, rope=d == 128)
    ws.buf.fill_(0x5a)

    def layer(**kw):
        a = run_layer(w, inp, dev, kept, kinds, workspace=ws, dbg=False, **kw)
        b = run_layer(w, inp, dev, kept, kinds, workspace=ws, dbg=False, prebuilt_lists=True, **kw)
        c = run_layer(w, inp, dev, kept, kinds, workspace=ws, **kw)
        assert torch.equal(a["out_t"], b["out_t"]) and torch.equal(a["out_t"], c["out_t"])
        return c

    sparse_only = layer(lam=0.0)
    base = _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0)
    tau = float(0.5 * (base["s"][0] + base["s"][1]))
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0, drop_threshold=tau)
    drop = layer(lam=20.0, drop_threshold=tau)
    assert drop["dropped"].tolist() == [1, 0]
    compare_layer(drop, ref, check_linear=False, label="cut+drop")
    assert torch.equal(drop["out_t"][0], sparse_only["out_t"][0]) and not torch.equal(drop["out_t"][1], sparse_only["out_t"][1])
    if d == 128:
        cs, sn = wl.rope_tables(w.T, w.Hh, w.W, d)
        rope = layer(lam=20.0, rope=(torch.from_numpy(cs).cuda(), torch.from_numpy(sn).cuda()))
        compare_layer(rope, _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0, rope=(cs, sn)), label="cut+rope")

    # rows of 0 to 18 blocks: whole tiles empty, of one entry, with a single row that has any, and cut ones between them
    rng = np.random.default_rng(d)
    sizes = [[0, 0, 0, 0], [18, 0, 1, 0], [1, 1, 1, 1], [0, 0, 12, 0], [6, 5]]
    rows = [np.sort(rng.choice(w.nb, size=sz, replace=False)) for h in range(w.H) for t in (sizes if h else sizes[:4][::-1] + sizes[4:]) for sz in t]
    csr = (np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32), np.concatenate(rows).astype(np.int32))
    res = layer(csr=csr)
    o_s, rws = oracle.sparse_attn(inp["q"], inp["k"], inp["v"], (w.T, w.Hh, w.W), 64, kinds, *csr)
    got, ok = gather_rows(res["o_sparse"], rws)
    assert np.isfinite(got[ok]).all() and errors(got[ok], o_s[ok])[1] <= REL_L2

    row_ptr, col_idx = sb.salad_block_mask(w.T, w.Hh, w.W, w.block, kept)
    out, dropped = torch.zeros_like(dev["q"]), torch.zeros(w.B, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        p, keep = sb.make_fwd_params(dev["q"], dev["k"], dev["v"], out, (w.T, w.Hh, w.W), row_ptr, col_idx, kinds, lam=20.0,
                                     head_scale=dev["head_scale"], x_t=dev["x_t"], w_gate=dev["w_gate"], eps=w.eps, workspace=ws,
                                     drop_threshold=tau, dropped_out=dropped)
        sb.salad_fwd_call(p)
    for rep in range(4):
        out.fill_(float("nan"))
        if rep == 2:
            ws.buf.fill_(0x5a)
        assert torch.equal(layer(lam=0.0)["out_t"], sparse_only["out_t"])          # eager work on the same workspace between the replays
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, drop["out_t"]), f"replay {rep} differs from the eager call"


def test_workspace_without_room_for_the_pieces(oracle):
    """The scratch of cut tiles is optional: a workspace sized for a larger grid whose tiles fill whole rounds (no pieces)
    serves a smaller one, whose tiles then run whole, and the state alone never needs it."""
    H, d = 32, 64
    w = wl.small("uncut", 1, H, d, 4, 13, 16, "bf16", 0.5, seed=640)          # N = 832: 128 tiles, 2 pieces each
    large = sb.Workspace(1, H, 2048, d, sb.SALAD_BF16)                         # 256 tiles
    assert large.bytes < sb.salad_fwd_workspace_bytes(1, H, w.N, d, sb.SALAD_BF16)
    large.buf.fill_(0x5a)
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds, kept = wl.head_kinds(w), [13] * H
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    cut = run_layer(w, inp, dev, kept, kinds, dbg=False)
    row_ptr, col_idx = sb.salad_block_mask(w.T, w.Hh, w.W, w.block, kept)
    for lists in (None, sb.salad_tile_lists(row_ptr, col_idx, H, w.nb)):
        out = sb.salad_sparse_linear_attn_fwd(dev["q"], dev["k"], dev["v"], (w.T, w.Hh, w.W), row_ptr, col_idx, kinds, lam=w.lam,
                                              head_scale=dev["head_scale"], x_t=dev["x_t"], w_gate=dev["w_gate"], eps=w.eps,
                                              workspace=large, tile_lists=lists)
        got = out.float().cpu().numpy().astype(np.float64)
        compare_layer({"out": got}, ref, check_linear=False, label="uncut")
        assert errors(got, cut["out"])[1] < 4e-3                               # two independently rounded bf16 results
    Hs, Z = sb.salad_linear_state_fwd(dev["k"], dev["v"], large)
    assert errors(Hs.cpu().numpy().astype(np.float64), ref["Hs"])[1] < 2e-6
    assert errors(Z.cpu().numpy().astype(np.float64), ref["Z"])[1] < 2e-6


@pytest.mark.parametrize("B,H,d,grid,keep,opt", [
    (1, 2, 128, (1, 1, 40), 1, ""),            # one block, its riders with 3 of 8 waves' tokens; one gate share
    (3, 5, 128, (3, 5, 17), 2, "drop"),        # 255 tokens, a last group of 15; samples pruned and not
    (1, 12, 128, (4, 16, 16), 4, ""),          # whole groups, tiles dealt by rows
    (1, 12, 128, (5, 15, 26), 31, ""),         # lists that are cut, with riders on the compute units of other pieces
    (1, 8, 128, (5, 15, 26), 31, ""),          # cut in two, without riders in four
    (1, 2, 128, (4, 25, 40), 48, ""),          # in six and eight; a last block of 32
    (1, 16, 128, (5, 15, 26), 6, ""),          # more riders and tiles than compute units
    (1, 40, 128, (2, 9, 9), 2, "rope"),        # a row of 5120 channels
    (1, 64, 128, (1, 7, 9), 1, ""),            # 8192
    (2, 3, 128, (3, 5, 13), 3, "proj"),
    (1, 3, 64, (3, 13, 14), 9, "drop"),        # 64-wide heads; a row of 192 channels, a ragged chunk
    (1, 40, 64, (2, 16, 16), 8, "given"),      # the scale is given: no gate
    (1, 1, 64, (5, 30, 36), 20, ""),           # the longest sequence (5400)
])
def test_state_and_gate_within_the_attention_launch(B, H, d, grid, keep, opt):
    """Short sequences: riders in the attention's launch give the bits of the launches of their own that the per-stage timing mode makes (in
    another workspace), on a workspace that holds anything, then another call's leavings; and so does a tile that does not wait for them (a bound
    of 0 on its wait) or has none to wait for (-1: they leave at once, and the words of the heads are left as the tiles counted in them)."""
    w = wl.small(f"within-{H}-{d}", B, H, d, *grid, "bf16", 0.5, seed=700 + H)
    kinds, kept = wl.head_kinds(w), [min(keep, w.nb)] * H
    row_ptr, col_idx = sb.salad_block_mask(*grid, w.block, kept)
    ws, apart = (sb.Workspace(B, H, w.N, d, sb.SALAD_BF16, full_proj=opt == "proj", rope=opt == "rope") for _ in range(2))
    for seed in (1, 2):
        inp = {k: v.copy() for k, v in wl.make_inputs(wl.small("x", B, H, d, *grid, "bf16", 0.5, seed=700 + H + seed)).items()}
        dev = upload(w, inp)
        s_out, dropped = torch.zeros(B, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda")
        kw = dict(lam=20.0, eps=w.eps, s_out=s_out, head_scale=dev["head_scale"])
        if opt == "given":
            kw["s"] = torch.rand(B, device="cuda")
        else:
            kw.update(x_t=dev["x_t"], w_gate=dev["w_gate"])
        if opt == "drop":
            s = sb.salad_gate_fwd(dev["x_t"], dev["w_gate"])
            kw.update(drop_threshold=float(s.max()) if B > 1 else 1e-6, dropped_out=dropped)       # all but the largest, or none
        if opt == "rope":
            kw.update(zip(("rope_cos", "rope_sin"), (torch.from_numpy(t).cuda() for t in wl.rope_tables(*grid, d))))
        if opt == "proj":
            kw.update(head_scale=None, w_proj=torch.randn(H * d, H * d, device="cuda").bfloat16() / (H * d) ** 0.5)

        def call(polls=None, workspace=ws):
            out = torch.full_like(dev["q"], float("nan"))
            s_out.fill_(float("nan"))
            dropped.fill_(-1)
            p, keepalive = sb.make_fwd_params(dev["q"], dev["k"], dev["v"], out, grid, row_ptr, col_idx, kinds, workspace=workspace, **kw)
            sb._check(sb.lib().salad_sparse_linear_attn_fwd(C.byref(p)) if polls is None else sb.lib().salad_fwd_with_polls(C.byref(p), polls))
            torch.cuda.synchronize()
            return out, s_out.clone(), dropped.clone()

        sb.salad_timing_enable(1)
        try:
            ref = call(workspace=apart)
        finally:
            sb.salad_timing_read(True)
            sb.salad_timing_enable(0)
        for polls, leavings in ((None, seed > 1), (-1, False), (0, True), (-1, False), (None, True), (None, True), (0, False)):
            if not leavings:
                ws.buf.fill_(0x5a)
            for got, want in zip(call(polls), ref):
                assert torch.equal(got, want), (opt, polls, leavings, seed)
        if opt == "drop" and B > 1:
            assert sorted(ref[2].tolist()) == [0] + [1] * (B - 1)


def test_workspace_with_room_for_the_pieces_only():
    """A workspace with room for the pieces of cut tiles but not for state and gate within the attention's launch: tiles are cut as they
    are where the sparse branch runs alone."""
    H, d, grid = 2, 128, (4, 25, 40)
    w = wl.small("pieces-only", 1, H, d, *grid, "bf16", 0.5, seed=641)
    dev = upload(w, wl.make_inputs(w))
    kinds = wl.head_kinds(w)
    row_ptr, col_idx = sb.salad_block_mask(*grid, w.block, [48] * H)
    args = (dev["q"], dev["k"], dev["v"], grid, row_ptr, col_idx, kinds)
    alone = sb.salad_sparse_linear_attn_fwd(*args, lam=0.0)
    ws = sb.Workspace(1, H, w.N, d, sb.SALAD_BF16)
    kw = dict(lam=20.0, head_scale=dev["head_scale"], x_t=dev["x_t"], w_gate=dev["w_gate"], eps=w.eps, workspace=ws)
    whole = sb.salad_sparse_linear_attn_fwd(*args, **kw)
    ws.bytes -= 256
    assert torch.equal(sb.salad_sparse_linear_attn_fwd(*args, drop_threshold=2.0, **kw), alone)
    out = sb.salad_sparse_linear_attn_fwd(*args, **kw)
    assert errors(out.float().cpu().numpy().astype(np.float64), whole.float().cpu().numpy().astype(np.float64))[1] < 4e-3     # two independently rounded bf16 results


def test_sparse_branch_alone_is_one_launch():
    """lambda = 0 with prebuilt lists on a grid whose tiles may be cut: the attention kernel and nothing else, counted in a
    captured graph; replays on a workspace that held anything give the bits of the eager call."""
    w = wl.small("one-launch", 1, 3, 128, 5, 13, 17, "bf16", 0.5, seed=641)   # N = 1105: 15 tiles in up to 8 pieces
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    grid, kinds, kept = (w.T, w.Hh, w.W), wl.head_kinds(w), [18, 5, 13]
    row_ptr, col_idx = sb.salad_block_mask(*grid, w.block, kept)
    lists = sb.salad_tile_lists(row_ptr, col_idx, w.H, w.nb)
    eager = run_layer(w, inp, dev, kept, kinds, lam=0.0, dbg=False)["out_t"].clone()
    ws = sb.Workspace(w.B, w.H, w.N, w.d, sb.SALAD_BF16)
    ws.buf.fill_(0x5a)
    out = torch.zeros_like(dev["q"])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        p, keep = sb.make_fwd_params(dev["q"], dev["k"], dev["v"], out, grid, row_ptr, col_idx, kinds, lam=0.0, workspace=ws, tile_lists=lists)
        sb.salad_fwd_call(p)
    nodes = C.c_size_t(0)
    hip = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    assert C.CDLL(hip).hipGraphGetNodes(C.c_void_p(g.raw_cuda_graph()), None, C.byref(nodes)) == 0
    assert nodes.value == 1
    g.instantiate()
    for rep in range(3):
        out.fill_(float("nan"))
        (dev["x_t"].float().sum()).item()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), f"replay {rep} differs from the eager call"


@pytest.mark.parametrize("second_half", [True, False])
def test_softmax_reference_is_the_first_block_maximum(second_half):
    """Two keys carry the weight of every query, one in each half of the first block.  The reference is the larger of the two
    logits wherever it sits, so its weight is 1 and the other one's is rounded to bf16: O_s to fp32 precision (a reference
    taken from the first half alone rounds the other weight and is 1e-3 off)."""
    N, d = 64, 128
    a, b = (9, 41) if second_half else (41, 9)                     # logits 1.0 (key a) and 1.5 (key b), the others -300
    q = torch.zeros(1, 1, N, d); k = torch.zeros(1, 1, N, d)
    q[..., 0] = 1.0
    k[..., 0] = -300.0
    k[0, 0, a, 0], k[0, 0, b, 0] = 1.0, 1.5
    v = torch.from_numpy(wl.round_to_bf16(wl.normal(642, "v", (1, 1, N, d))))
    row_ptr, col_idx = sb.salad_block_mask(1, 8, 8, 64, [1])
    o_s = torch.empty(1, 1, N, d, device="cuda")
    sb.salad_sparse_linear_attn_fwd(q.bfloat16().cuda(), k.bfloat16().cuda(), v.bfloat16().cuda(), (1, 8, 8), row_ptr, col_idx, lam=0.0,
                                    softmax_scale=1.0, o_sparse_dbg=o_s)
    pa = float(torch.tensor(np.exp(-0.5)).bfloat16())              # 0.60653 lies 0.23 of a spacing from a rounding boundary
    want = (pa * v[0, 0, a].double() + v[0, 0, b].double()) / (pa + 1.0)
    got = o_s.double().cpu()[0, 0]
    assert float((got - want).abs().max()) < 1e-5


@pytest.mark.parametrize("B,H,grid", [(2, 2, (1, 1, 7)), (1, 3, (5, 16, 51)), (2, 1, (5, 16, 52)), (1, 2, (7, 24, 49))])
def test_fp32_gate_reduced_by_the_attention_kernel(B, H, grid):
    """1 to 512 partial sums, around the 255 and 261 where a second one falls to the same place: the dynamic scale of the layer
    call has the bits of the gate called alone, and a call that is given it the bits of the one that finds it."""
    N, d = grid[0] * grid[1] * grid[2], 64
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda") for _ in range(3))
    x, wg = torch.randn(B, N, H * d, generator=g, device="cuda"), torch.randn(H * d, generator=g, device="cuda") * 0.1
    rp, ci = sb.salad_block_mask(*grid, 64, [1] * H)
    hs, s = torch.rand(H, generator=g, device="cuda"), torch.full((B,), float("nan"), device="cuda")
    kw = dict(lam=0.5, head_scale=hs, eps=1e-6)
    out = sb.salad_sparse_linear_attn_fwd(q, k, v, grid, rp, ci, [h % 2 for h in range(H)], x_t=x, w_gate=wg, s_out=s, **kw)
    alone = sb.salad_gate_fwd(x, wg)
    given = sb.salad_sparse_linear_attn_fwd(q, k, v, grid, rp, ci, [h % 2 for h in range(H)], s=alone, **kw)
    assert torch.equal(s, alone) and torch.equal(out, given)


def _graph_nodes(g):
    nodes = C.c_size_t(0)
    hip = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64.so" in line)
    assert C.CDLL(hip).hipGraphGetNodes(C.c_void_p(g.raw_cuda_graph()), None, C.byref(nodes)) == 0
    return nodes.value


@pytest.mark.parametrize("H,grid,nodes", [(1, (1, 1, 40), 2), (2, (8, 64, 32), 2), (2, (41, 20, 20), 3)])
def test_fp32_gate_has_a_launch_of_its_own_in_large_calls(H, grid, nodes):
    """Up to 2048 query tiles of 16 the attention kernel reduces the gate (two launches), beyond that (here 2050) a third one does; a call
    that is given the scale needs no reduce at any size."""
    N, d = grid[0] * grid[1] * grid[2], 64
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v = (torch.randn(1, H, N, d, generator=g, device="cuda") for _ in range(3))
    x, wg = torch.randn(1, N, H * d, generator=g, device="cuda"), torch.randn(H * d, generator=g, device="cuda") * 0.1
    rp, ci = sb.salad_block_mask(*grid, 64, [1] * H)
    ws, out = sb.Workspace(1, H, N, d, sb.SALAD_F32), torch.empty_like(q)
    alone = sb.salad_gate_fwd(x, wg)
    outs = []
    for kw, want in ((dict(x_t=x, w_gate=wg), nodes), (dict(s=alone), 2)):
        graph = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(graph):
            p, keep = sb.make_fwd_params(q, k, v, out, grid, rp, ci, [h % 2 for h in range(H)], lam=0.5, workspace=ws, **kw)
            sb.salad_fwd_call(p)
        assert _graph_nodes(graph) == want
        graph.instantiate()
        graph.replay()
        outs.append(out.clone())
    assert torch.equal(*outs)


def test_fp32_infinite_value_in_the_last_row():
    """Keys past the end of the sequence do not exist: an infinite V element of the last token gives infinity in its channel
    and nothing anywhere else, whatever part of a 32-key unit the tail fills."""
    for N in (160, 144, 130):                                      # tails of 32, 16 and 2 keys
        q, k, v = (torch.from_numpy(wl.normal(643, t, (1, 1, N, 64))).cuda() for t in ("q", "k", "v"))
        v[0, 0, N - 1, 5] = float("inf")
        row_ptr, col_idx = sb.salad_block_mask(1, 1, N, 64, [3])
        out = sb.salad_sparse_linear_attn_fwd(q, k, v, (1, 1, N), row_ptr, col_idx, lam=0.0)
        v[0, 0, N - 1, 5] = 0.0
        want = sb.salad_sparse_linear_attn_fwd(q, k, v, (1, 1, N), row_ptr, col_idx, lam=0.0)
        want[..., 5] = float("inf")
        assert torch.equal(out, want), N


def test_fp32_state_and_gate_of_many_samples():
    """The state and the gate of 247000 samples: 16 state tiles and one gate workgroup of 1024 threads a sample are more than
    the 2^32 threads that one grid dimension holds (beyond, the runtime drops workgroups without an error)."""
    B, d = 247000, 64
    q, k, v, x = (torch.randn(B, 1, 1, d, generator=torch.Generator("cuda").manual_seed(s), device="cuda") for s in range(4))
    wg = torch.randn(d, generator=torch.Generator("cuda").manual_seed(4), device="cuda") * 0.05
    row_ptr, col_idx = sb.salad_block_mask(1, 1, 1, 64, [1])
    out = sb.salad_sparse_linear_attn_fwd(q, k, v, (1, 1, 1), row_ptr, col_idx, lam=1.0, x_t=x.view(B, 1, d), w_gate=wg)
    q, k, v, x = (t.double().view(B, d) for t in (q, k, v, x))
    dot = (q.clamp(min=0) * k.clamp(min=0)).sum(1, keepdim=True)
    want = v + torch.sigmoid(x @ wg.double())[:, None] * v * dot / (dot + 1e-6)
    assert float((out.view(B, d).double() - want).norm() / want.norm()) < 1e-5


def test_fp32_tiles_of_many_heads():
    """8.4 million heads of one token: as many tiles, more than one grid dimension of 256-thread workgroups took."""
    H, d = 64, 64
    B = 8388672 // H                                               # 2^31 / 256 tiles are 8388608
    v = torch.randn(B, H, 1, d, generator=torch.Generator("cuda").manual_seed(5), device="cuda")
    row_ptr, col_idx = sb.salad_block_mask(1, 1, 1, 64, [1] * H)
    out = sb.salad_sparse_linear_attn_fwd(v, v, v, (1, 1, 1), row_ptr, col_idx, lam=0.0)
    assert torch.equal(out, v)                                     # one key: its value


@pytest.mark.parametrize("B,H,d,grid,dtype", [
    (2, 1, 64, (1, 3, 5), "bf16"), (1, 5, 128, (3, 7, 11), "bf16"), (3, 12, 128, (2, 5, 13), "bf16"), (1, 16, 128, (1, 1, 1), "bf16"),
    (1, 40, 128, (2, 9, 9), "bf16"), (1, 41, 128, (2, 3, 3), "bf16"), (2, 2, 64, (2, 9, 11), "f32"), (1, 8, 128, (1, 4, 5), "f32"),
    (1, 9, 128, (1, 4, 5), "f32"),
])
def test_gate_rides_with_the_state(B, H, d, grid, dtype):
    """Gate and state in one launch (every row width the launch is built for, and the first beyond) give the bits of the two
    launches that the per-stage timing mode makes."""
    w = wl.small(f"ride-{H}-{d}", B, H, d, *grid, dtype, 0.5, seed=500 + H)
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    rope = tuple(torch.from_numpy(t).cuda() for t in wl.rope_tables(*grid, d)) if dtype == "bf16" and d == 128 else None
    kinds, kept = wl.head_kinds(w), [max(1, w.nb // 2)] * H
    for r in {None, rope}:
        got = run_layer(w, inp, dev, kept, kinds, dbg=False, rope=r)
        sb.salad_timing_enable(1)
        try:
            ref = run_layer(w, inp, dev, kept, kinds, dbg=False, rope=r)
        finally:
            sb.salad_timing_read(True)
            sb.salad_timing_enable(0)
        assert np.array_equal(got["s"], ref["s"]) and torch.equal(got["out_t"], ref["out_t"])


@pytest.mark.parametrize("d", [64, 128])
def test_sixty_four_heads(oracle, d):
    """The largest head count the boundary takes (64: the head-order mask is a 64-bit word, the last head temporal),
    every head with its own window size.  The gate runs over D = 4096 (d = 64) and D = 8192 (d = 128, the widest row the
    layer can have: gate weights in LDS)."""
    w = wl.small(f"heads64-d{d}", 1, 64, d, 3, 5, 21, "bf16", 0.5, seed=140 + d)      # N = 315: 5 blocks, tail 59
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    assert kinds[63] == 1
    kept = [1 + (h * 7) % 5 for h in range(w.H)]
    res = run_layer(w, inp, dev, kept, kinds)
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    assert np.abs(res["s"] - ref["s"]).max() < 2e-6
    assert np.array_equal(res["row_ptr"], ref["row_ptr"]) and np.array_equal(res["col_idx"], ref["col_idx"])
    compare_layer(res, ref, label=w.name)


def test_zero_static_scale_gives_sparse_branch_exactly(oracle):
    """Zero-initialised static scale (Sec. 4.2): the layer output is the sparse branch alone; the
    three ways of switching the linear branch off agree bit for bit."""
    w = SMALL[1]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4] * w.H
    r0 = run_layer(w, inp, dev, kept, kinds, lam=0.0, dbg=False)
    r1 = run_layer(w, inp, dev, kept, kinds, head_scale=torch.zeros(w.H, device="cuda"), dbg=False)
    r2 = run_layer(w, inp, dev, kept, kinds, s=torch.zeros(w.B, device="cuda"), dbg=False)
    assert torch.equal(r0["out_t"], r1["out_t"]) and torch.equal(r0["out_t"], r2["out_t"])
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=0.0)
    assert np.array_equal(ref["out"], ref["o_sparse"])
    compare_layer(r0, ref, label="lambda=0")


def test_linear_dominant_case(oracle):
    """On N(0,1) inputs the linear term is below the bf16 spacing of O_s, so a large static scale
    makes the combined output sensitive to the linear branch."""
    w = SMALL[0]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [3, 2]
    res = run_layer(w, inp, dev, kept, kinds, lam=100.0)
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=100.0)
    got, ok = gather_rows(res["out"], ref["rows"])
    lin_share = np.abs(ref["out"] - ref["o_sparse"])[ok].mean() / np.abs(ref["out"])[ok].mean()
    assert lin_share > 0.5
    a, r = errors(got[ok], ref["out"][ok])
    say(f"  linear-dominant: share={lin_share:.2f} max_abs={a:.3e} rel_l2={r:.3e}")
    assert r <= REL_L2


@pytest.mark.parametrize("kept_n", [19, 6], ids=["all-blocks", "window-6"])
@pytest.mark.parametrize("profile", ["rising", "falling", "mixed"])
def test_softmax_reference_moves_across_blocks(oracle, profile, kept_n):
    """Key magnitudes that change by large factors from one 64-token block to the next, so that the largest
    logit a query has seen so far jumps by tens of binades between blocks (rising), never again reaches the
    first block's (falling), or both (mixed): the running reference of the online softmax has to move, and
    what was accumulated before has to be rescaled, many times per row."""
    w = SMALL[7]                                   # N = 1170: 19 blocks, 3 heads (one temporal)
    inp = wl.make_inputs(w)
    blk = np.arange(w.N) // 64
    if profile == "rising":
        g = 1.0 + 3.0 * blk
    elif profile == "falling":
        g = 1.0 + 3.0 * (blk.max() - blk)
    else:
        g = np.array([1.0, 30.0, 2.0, 55.0, 8.0])[(blk * 7 + 3) % 5]
    inp["k"] = wl.round_to_bf16(inp["k"] * g[None, None, :, None].astype(np.float32))
    # With such keys the softmax is close to one-hot and the output is a single V row: values up to 4.5, where one
    # bf16 rounding alone is 1.6e-2 and the two roundings of the regrouped Top-K path (partial results are stored in
    # bf16) 3.1e-2.  A quarter of the magnitude keeps the absolute bar meaningful for every path; exact in bf16.
    inp["v"] = inp["v"] * np.float32(0.25)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [kept_n] * w.H
    res = run_layer(w, inp, dev, kept, kinds)
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    compare_layer(res, ref, label=f"{profile}/{kept_n}: ")
    if profile == "mixed":
        # the other attention kernels keep their own running maximum
        for variant in (1, 2):
            sb.salad_tune("attn_variant", variant)
            try:
                res = run_layer(w, inp, dev, kept, kinds)
            finally:
                sb.salad_tune("attn_variant", 0)
            compare_layer(res, ref, label=f"{profile}/{kept_n}/variant{variant}: ")
        # Top-K modes (stored order, all heads spatial): gathered queries and token mask
        kinds0 = np.zeros(w.H, dtype=np.uint8)
        ref_t = _oracle_layer(oracle, w, inp, [1] * w.H, kinds0, topk=3, key_block=128)
        for tv in (0, 1):
            sb.salad_tune("topk_variant", tv)
            try:
                res_t = run_layer(w, inp, dev, [1] * w.H, kinds0, topk=3, topk_key_block=128)
            finally:
                sb.salad_tune("topk_variant", 0)
            assert np.array_equal(res_t["topk_mask"], ref_t["topk_mask"])
            compare_layer(res_t, ref_t, label=f"{profile}/topk-variant{tv}: ")


@pytest.mark.parametrize("H,grid,keep", [(43, (4, 17, 19), 21), (43, (4, 17, 19), 6), (58, (4, 23, 25), 36)], ids=["whole", "whole-window-6", "cut"])
@pytest.mark.parametrize("profile", ["rising", "mixed"])
def test_references_of_two_query_sets_move_apart(oracle, profile, H, grid, keep):
    """64 queries a wave (d = 64, more than 256 tiles): the references of its two sets of 32 move independently.  Queries of one set, the
    second in every other head, are so small that they never move after the first block, those of the other rise or jump by
    tens of binades between blocks; in the last head both sets do."""
    w = wl.small(f"sets-{H}", 1, H, 64, *grid, "bf16", 0.5, seed=118)
    inp = wl.make_inputs(w)
    kinds = wl.head_kinds(w)
    blk = np.arange(w.N) // 64
    g = 1.0 + 3.0 * blk if profile == "rising" else np.array([1.0, 30.0, 2.0, 55.0, 8.0])[(blk * 7 + 3) % 5]
    small = np.arange(w.N) // 32 % 2
    for h in range(H):
        row = np.array([oracle.row_of_position(int(kinds[h]), p, w.T, w.Hh, w.W) for p in range(w.N)])
        inp["k"][:, h, row] *= g[:, None].astype(np.float32)
        if h < H - 1:
            inp["q"][:, h, row] *= np.where(small == h // 2 % 2, 0.02, 1.0)[:, None].astype(np.float32)
    for t in ("q", "k"):
        inp[t] = wl.round_to_bf16(inp[t])
    inp["v"] = inp["v"] * np.float32(0.25)                 # the softmax is close to one-hot: see test_softmax_reference_moves_across_blocks
    dev = upload(w, inp)
    ref = _oracle_layer(oracle, w, inp, [keep] * H, kinds)
    for dbg in (True, False):
        compare_layer(run_layer(w, inp, dev, [keep] * H, kinds, dbg=dbg), ref, label=f"{profile}/{H}/{keep}: ")


@pytest.mark.parametrize("H,d,grid,keep", [
    (43, 128, (4, 17, 19), 8),        # 258 tiles of 21 blocks, lists of at most 11 entries: the larger products
    (43, 128, (4, 17, 19), 9),        # lists of 9 to 12: both in one call
    (43, 128, (4, 17, 19), 16), (43, 128, (4, 17, 19), 17),
    (43, 128, (4, 17, 19), 21),       # 21, the last block of 12 keys
    (29, 128, (4, 23, 25), 36),       # 261 tiles: a round, and five in pieces
    (43, 64, (4, 17, 19), 16),        # lists of at most 19 entries: the larger products
    (43, 64, (4, 17, 19), 17),        # lists of 17 to 20: both in one call
    (58, 64, (4, 23, 25), 36),        # 522 tiles: a round, and ten in pieces that have a compute unit each
    (60, 64, (4, 25, 28), 44),        # 660: 148 in three pieces each, which share theirs
], ids=lambda x: str(x).replace(" ", ""))
def test_smaller_products_of_long_lists(oracle, topk_variant, H, d, grid, keep):
    """Calls of more than one round of tiles around the list length from which on a tile is computed with 16x16x32 products; key magnitudes
    that move the references of either group of 16 queries, and query rows that are not finite."""
    w = wl.small(f"columns-{H}-{d}", 1, H, d, *grid, "bf16", 0.5, seed=130 + keep)
    inp = wl.make_inputs(w)
    kinds = wl.head_kinds(w)
    blk = np.arange(w.N) // 64
    g = np.array([1.0, 30.0, 2.0, 55.0, 8.0])[(blk * 7 + 3) % 5]
    inp["k"] = wl.round_to_bf16(inp["k"] * g[None, None, :, None].astype(np.float32))
    inp["q"][:, :, np.arange(w.N) // 16 % 2 == 0] *= np.float32(2.0 ** -6)      # every other group of 16 stored rows stays where it is
    inp["v"] = inp["v"] * np.float32(0.25)                 # the softmax is close to one-hot: see test_softmax_reference_moves_across_blocks
    dev = upload(w, inp)
    ref = _oracle_layer(oracle, w, inp, [keep] * H, kinds)
    res = [run_layer(w, inp, dev, [keep] * H, kinds, dbg=dbg) for dbg in (True, False)]
    for r in res:
        compare_layer(r, ref, label=f"{H}/{d}/{keep}: ")
    assert torch.equal(res[0]["out_t"], res[1]["out_t"])
    test_non_finite_query_rows_stay_alone(topk_variant, 1, H, d, grid, keep, 0)


def test_precomputed_s_and_bias_and_scale_arguments(oracle):
    w = SMALL[2]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [3] * w.H
    s = torch.tensor([0.31], device="cuda")
    res = run_layer(w, inp, dev, kept, kinds, s=s, softmax_scale=0.2, eps=1e-3)
    ref = _oracle_layer(oracle, w, inp, kept, kinds, s_override=[0.31], scale=0.2, eps=1e-3)
    assert abs(res["s"][0] - 0.31) < 1e-7
    compare_layer(res, ref, label="s_dev")
    res = run_layer(w, inp, dev, kept, kinds, b_gate=-1.5)
    ref = _oracle_layer(oracle, w, inp, kept, kinds, b_gate=-1.5)
    assert np.abs(res["s"] - ref["s"]).max() < 2e-6 and ref["s"][0] < 0.25
    compare_layer(res, ref, label="b_gate")


def test_zero_queries_average_the_kept_values(oracle):
    """Q = 0: O_s is the plain mean of V over the kept, existing tokens (pins mask wiring, tail and
    token orders on the GPU without the oracle's softmax)."""
    w = SMALL[1]
    inp = wl.make_inputs(w)
    inp["q"] = np.zeros_like(inp["q"])
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [3, 4, 2]
    res = run_layer(w, inp, dev, kept, kinds, lam=0.0)
    rp, ci = oracle.block_mask(w.T, w.Hh, w.W, 64, kept)
    for h in range(w.H):
        order = np.array([oracle.row_of_position(int(kinds[h]), p, w.T, w.Hh, w.W) for p in range(w.N)])
        for i in range(w.nb):
            cols = ci[rp[h * w.nb + i]:rp[h * w.nb + i + 1]]
            krows = np.concatenate([order[j * 64:min((j + 1) * 64, w.N)] for j in cols])
            mean = inp["v"][:, h][:, krows].astype(np.float64).mean(axis=1)          # [B, d]
            qrows = order[i * 64:min((i + 1) * 64, w.N)]
            got = res["o_sparse"][:, h][:, qrows]                                      # [B, rows, d]
            assert np.abs(got - mean[:, None, :]).max() < 3e-3


def test_arbitrary_csr(oracle):
    """Any CSR with ascending unique block ids per row is accepted (e.g. a Top-K selection): rows
    of different lengths, non-contiguous ids, neighbouring query blocks with disjoint lists."""
    w = wl.small("csr", 1, 2, 128, 4, 10, 16, "bf16", 0.5, seed=108)    # N=640, nb=10
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    u = wl.uniform(108, "pick", (w.H * w.nb, w.nb))
    row_ptr, col_idx = [0], []
    for r in range(w.H * w.nb):
        cnt = (1 + (r * 7) % 5) if r != 3 else 0          # one empty row: its sparse output is defined as zero
        cols = sorted(np.argsort(u[r])[:cnt].tolist())
        col_idx += cols
        row_ptr.append(len(col_idx))
    csr = (np.array(row_ptr, np.int32), np.array(col_idx, np.int32))
    res = run_layer(w, inp, dev, None, kinds, csr=csr)
    o_s, rows = oracle.sparse_attn(inp["q"], inp["k"], inp["v"], (w.T, w.Hh, w.W), 64, kinds, *csr)
    got, ok = gather_rows(res["o_sparse"], rows)
    a, r = errors(got[ok], o_s[ok])
    say(f"  arbitrary CSR: o_sparse max_abs={a:.3e} rel_l2={r:.3e}")
    assert r <= REL_L2


@pytest.mark.parametrize("H,grid,longest", [
    (43, (4, 17, 19), 21),            # 258 tiles of 21 blocks
    (58, (4, 23, 25), 30),            # 522 tiles of 36 blocks, the last ten cut
])
def test_arbitrary_csr_with_two_query_sets_a_wave(oracle, H, grid, longest):
    """The same for 64 queries a wave (d = 64, more than 256 tiles), with a whole tile of empty rows in the last head."""
    w = wl.small(f"csr-{H}", 1, H, 64, *grid, "bf16", 0.5, seed=108)
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    u = wl.uniform(108, "pick", (w.H * w.nb, w.nb))
    row_ptr, col_idx = [0], []
    for r in range(w.H * w.nb):
        cnt = 1 + (r * 7) % longest
        if r == 3 or (w.H - 1) * w.nb + 4 <= r < (w.H - 1) * w.nb + 8:
            cnt = 0
        cols = sorted(np.argsort(u[r])[:cnt].tolist())
        col_idx += cols
        row_ptr.append(len(col_idx))
    csr = (np.array(row_ptr, np.int32), np.array(col_idx, np.int32))
    o_s, rows = oracle.sparse_attn(inp["q"], inp["k"], inp["v"], (w.T, w.Hh, w.W), 64, kinds, *csr)
    for got in (run_layer(w, inp, dev, None, kinds, csr=csr)["o_sparse"], run_layer(w, inp, dev, None, kinds, csr=csr, lam=0.0, dbg=False)["out"]):
        got, ok = gather_rows(got, rows)
        a, r = errors(got[ok], o_s[ok])
        say(f"  arbitrary CSR: o_sparse max_abs={a:.3e} rel_l2={r:.3e}")
        assert r <= REL_L2


@pytest.mark.parametrize("H,d,grid", [(29, 128, (4, 23, 25)), (58, 64, (4, 23, 25))])
def test_arbitrary_csr_in_calls_of_more_than_a_round(oracle, H, d, grid):
    """Random rows of long lists with few gaps, which the smaller products take, between ones with many, which the larger take; rows that share a tile
    and no block, an empty row, an empty tile; tiles of the last round in pieces."""
    w = wl.small(f"csr-{H}-{d}", 1, H, d, *grid, "bf16", 0.5, seed=109)
    inp = wl.make_inputs(w)
    dev, kinds = upload(w, inp), wl.head_kinds(w)
    u = wl.uniform(109, "pick", (w.H, w.nb, w.nb))
    keep = u < np.array([0.95, 0.85, 0.75, 0.3])[np.arange(w.H) % 4][:, None, None]
    keep[0, 3] = False
    keep[1, 8:12] = np.arange(w.nb) % 4 == np.arange(4)[:, None]
    keep[-2, 4:8] = False
    csr = (np.cumsum(np.concatenate([[0], keep.sum(2).ravel()])).astype(np.int32), np.nonzero(keep.reshape(-1, w.nb))[1].astype(np.int32))
    o_s, rows = oracle.sparse_attn(inp["q"], inp["k"], inp["v"], (w.T, w.Hh, w.W), 64, kinds, *csr)
    for got in (run_layer(w, inp, dev, None, kinds, csr=csr)["o_sparse"], run_layer(w, inp, dev, None, kinds, csr=csr, lam=0.0, dbg=False)["out"]):
        got, ok = gather_rows(got, rows)
        a, r = errors(got[ok], o_s[ok])
        say(f"  arbitrary CSR: o_sparse max_abs={a:.3e} rel_l2={r:.3e}")
        assert r <= REL_L2


def test_samples_with_the_smaller_products(oracle):
    """Two samples, one without its linear branch, in a call of more than a round: 260 tiles, lists of 20 to 23, the last four in pieces."""
    w = wl.small("pruned-columns", 2, 13, 128, 21, 10, 12, "bf16", 0.5, seed=143)
    inp = wl.make_inputs(w)
    wg = inp["w_gate"]
    inp["x_t"] = inp["x_t"].copy()
    inp["x_t"][1] = wl.round_to_bf16(inp["x_t"][1] + (2.0 * wg / float(np.dot(wg, wg))).astype(np.float32))   # pre-activations of sample 1 up by ~2
    dev, kinds, kept = upload(w, inp), wl.head_kinds(w), [20] * w.H
    sel = list(range(0, w.nb, 6)) + [w.nb - 1]
    s = _oracle_layer(oracle, w, inp, kept, kinds, sel=[0])["s"]
    tau = float(0.5 * (s[0] + s[1]))
    ref = _oracle_layer(oracle, w, inp, kept, kinds, sel=sel, lam=20.0, drop_threshold=tau)
    assert ref["dropped"].tolist() == [1, 0]
    sparse_only = run_layer(w, inp, dev, kept, kinds, lam=0.0, dbg=False)["out_t"]
    for dbg in (True, False):
        res = run_layer(w, inp, dev, kept, kinds, lam=20.0, drop_threshold=tau, dbg=dbg)
        assert res["dropped"].tolist() == [1, 0]
        compare_layer(res, ref, check_linear=False, label="pruned")
        assert torch.equal(res["out_t"][0], sparse_only[0]) and not torch.equal(res["out_t"][1], sparse_only[1])


def _heads_alone(w, dev, first, count, label):
    """The workload and inputs of some of its heads."""
    part, cols = wl.small(label, w.B, count, w.d, w.T, w.Hh, w.W, w.dtype, 0.5, seed=w.seed), slice(first * w.d, (first + count) * w.d)
    some = {t: dev[t][:, first:first + count].contiguous() for t in ("q", "k", "v")}
    return part, dict(some, x_t=dev["x_t"][..., cols].contiguous(), w_gate=dev["w_gate"][cols].contiguous(),
                      head_scale=dev["head_scale"][first:first + count].contiguous())


@pytest.mark.parametrize("d", [128, 64])
@pytest.mark.parametrize("step", [2, 3])
def test_products_of_rows_with_gaps(d, step):
    """Lists of 36 entries of which a row keeps every second or third one are computed with the same products in calls of any size: 504 tiles
    against 252 of them, with the same bits."""
    w = wl.small(f"gaps-{d}", 1, 56, d, 4, 23, 25, "bf16", 0.5, seed=141)
    dev, kinds = upload(w, wl.make_inputs(w)), wl.head_kinds(w)
    part, some = _heads_alone(w, dev, 0, 28, f"gaps-part-{d}")
    rows = [np.arange(i % 4 % step, w.nb, step) for i in range(w.nb)]
    got = []
    for x, y, k in ((w, dev, kinds), (part, some, kinds[:28])):
        csr = (np.cumsum([0] + [len(r) for r in rows] * x.H), np.concatenate(rows * x.H))
        got.append(run_layer(x, None, y, None, k, csr=csr)["o_sparse"])
    assert np.array_equal(got[0][:, :28], got[1])


@pytest.mark.parametrize("d,H,first", [(128, 22, 16), (64, 47, 32)])
def test_products_of_a_cut_last_round(d, H, first):
    """Tiles of a last round that leaves half of the chip idle, here with lists too short to be cut: with the same products, and bits, as in a call of
    their own.  16 tiles a head: 96 behind 256, or 240 behind 512 that go two to a compute unit."""
    w = wl.small(f"round-{d}", 1, H, d, 4, 32, 32, "bf16", 0.5, seed=142)
    dev, kinds = upload(w, wl.make_inputs(w)), wl.head_kinds(w)
    part, some = _heads_alone(w, dev, first, H - first, f"round-part-{d}")
    whole = run_layer(w, None, dev, [20] * H, kinds)["o_sparse"]
    alone = run_layer(part, None, some, [20] * part.H, kinds[first:])["o_sparse"]
    assert np.array_equal(whole[:, first:], alone)


def test_unfused_epilogue_matches(oracle):
    w = SMALL[1]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4] * w.H
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=30.0)
    res = run_layer(w, inp, dev, kept, kinds, lam=30.0, flags=sb.SALAD_FLAG_UNFUSED_EPILOGUE)
    compare_layer(res, ref, label="unfused")


@pytest.mark.parametrize("grid,kept,truncated", [((9, 10, 13), [4, 7, 5], False), ((9, 10, 13), [4, 7, 5], True),
                                                 ((21, 30, 52), [51] * 3, False), ((5, 6, 9), [1, 5], True)])
def test_tile_lists_layout(oracle, grid, kept, truncated):
    """salad_tile_lists against the documented layout, rebuilt here from the oracle's CSR: per (head, tile of 4 query
    blocks) the ascending union of the rows' kept blocks, each entry block | (kept-by-row bits << 24), rotated to start at
    the entry whose block id is smallest modulo the list length; counts after the lists at the next 256-byte boundary."""
    T, Hh, W = grid
    H, nb = len(kept), (T * Hh * W + 63) // 64
    rp, ci = oracle.block_mask(T, Hh, W, 64, kept, truncated=truncated)
    row_ptr, col_idx = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda()
    buf = sb.salad_tile_lists(row_ptr, col_idx, H, nb)
    torch.cuda.synchronize()
    raw = buf.cpu().numpy()
    ntiles, cap = (nb + 3) // 4, (nb + 63) // 64 * 64
    nlist = H * ntiles * cap * 4
    lists = raw[:nlist].view(np.uint32).reshape(H, ntiles, cap)
    counts = raw[(nlist + 255) // 256 * 256:][:H * ntiles * 4].view(np.int32).reshape(H, ntiles)
    for h in range(H):
        for t in range(ntiles):
            bits = {}
            for i in range(4):
                r = 4 * t + i
                if r < nb:
                    for c in ci[rp[h * nb + r]:rp[h * nb + r + 1]]:
                        bits[int(c)] = bits.get(int(c), 0) | (1 << (24 + i))
            asc = [b | m for b, m in sorted(bits.items())]
            n = len(asc)
            assert counts[h, t] == n
            rot = min(range(n), key=lambda i: ((asc[i] & 0xffffff) % n, i)) if n else 0
            assert lists[h, t, :n].tolist() == asc[rot:] + asc[:rot]


def test_prebuilt_tile_lists_give_the_same_bits(oracle):
    """salad_tile_lists builds the large-tile kernel's visit lists once per CSR; a layer call that is handed them skips
    its own pre-pass and must produce the bits of a call that builds them itself (window mask and an arbitrary CSR)."""
    w = SMALL[7]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4, 5, 4]
    a = run_layer(w, inp, dev, kept, kinds, dbg=False)
    b = run_layer(w, inp, dev, kept, kinds, dbg=False, prebuilt_lists=True)
    assert np.array_equal(a["out"], b["out"])
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    compare_layer(b, ref, label="prebuilt lists")
    rng = np.random.default_rng(5)
    rows = [np.sort(rng.choice(w.nb, size=int(rng.integers(1, 7)), replace=False)) for _ in range(w.H * w.nb)]
    row_ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    col_idx = np.concatenate(rows).astype(np.int32)
    a = run_layer(w, inp, dev, kept, kinds, dbg=False, csr=(row_ptr, col_idx))
    b = run_layer(w, inp, dev, kept, kinds, dbg=False, csr=(row_ptr, col_idx), prebuilt_lists=True)
    assert np.array_equal(a["out"], b["out"])


@pytest.mark.parametrize("variant", [1, 2], ids=["128-row-fallback", "first-generation"])
def test_fallback_attention_kernels(oracle, variant):
    """The d=128 kernels that serve as fallbacks (block list too long for LDS, huge N, inexact division)
    produce the same layer within the same tolerances; selected here through the tuning knob."""
    w = SMALL[7]                                      # five tiles of 4 query blocks, ragged tail, 3 heads
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4, 5, 4]
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    sb.salad_tune("attn_variant", variant)
    try:
        res = run_layer(w, inp, dev, kept, kinds)
    finally:
        sb.salad_tune("attn_variant", 0)
    compare_layer(res, ref, label=f"variant{variant}")


def test_run_to_run_bit_reproducible():
    w = SMALL[1]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    outs = [run_layer(w, inp, dev, [4] * w.H, kinds, dbg=False)["out_t"] for _ in range(3)]
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


@pytest.mark.parametrize("flags", [0, sb.SALAD_FLAG_UNFUSED_EPILOGUE], ids=["fused", "unfused"])
def test_branch_dropping(oracle, flags):
    """Sec. 4.3: with a threshold between the two samples' dynamic scales only the lower one loses its linear
    branch; its output is then the sparse branch alone, bit for bit what lambda = 0 gives."""
    w = SMALL[1]                                      # B = 2, 3 heads, 11 blocks
    inp = wl.make_inputs(w)
    wg = inp["w_gate"]
    inp["x_t"] = inp["x_t"].copy()
    inp["x_t"][1] = wl.round_to_bf16(inp["x_t"][1] + (2.0 * wg / float(np.dot(wg, wg))).astype(np.float32))   # pre-activations of sample 1 up by ~2
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4] * w.H
    base = _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0)
    s = base["s"]
    assert s[1] - s[0] > 0.2
    tau = float(0.5 * (s[0] + s[1]))
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0, drop_threshold=tau)
    assert ref["dropped"].tolist() == [1, 0]
    res = run_layer(w, inp, dev, kept, kinds, lam=20.0, flags=flags, drop_threshold=tau)
    assert res["dropped"].tolist() == [1, 0]
    assert np.abs(res["s"] - s).max() < 2e-6          # the reported scale is the gate's, pruned or not
    compare_layer(res, ref, check_linear=False, label="drop")
    sparse_only = run_layer(w, inp, dev, kept, kinds, lam=0.0, flags=0)["out_t"]
    assert torch.equal(res["out_t"][0], sparse_only[0])            # pruned sample: exactly the sparse branch
    assert not torch.equal(res["out_t"][1], sparse_only[1])        # the other one kept its linear branch
    # thresholds outside the range: nobody / everybody
    none = run_layer(w, inp, dev, kept, kinds, lam=20.0, flags=flags, drop_threshold=1e-6)
    full = run_layer(w, inp, dev, kept, kinds, lam=20.0, flags=flags)
    assert none["dropped"].tolist() == [0, 0] and torch.equal(none["out_t"], full["out_t"])
    assert full["dropped"].tolist() == [-1, -1]       # not written when dropping is off
    every = run_layer(w, inp, dev, kept, kinds, lam=20.0, flags=flags, drop_threshold=2.0)
    assert every["dropped"].tolist() == [1, 1] and torch.equal(every["out_t"], sparse_only)


def _random_shapes(count, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(count):
        T, Hh, W = int(rng.integers(1, 9)), int(rng.integers(1, 13)), int(rng.integers(1, 13))
        H, B, d = int(rng.integers(1, 5)), int(rng.integers(1, 3)), int(rng.choice([64, 128]))
        out.append(wl.small(f"rand{i}-T{T}x{Hh}x{W}-H{H}-B{B}-d{d}", B, H, d, T, Hh, W, "bf16", 0.5, seed=1000 + seed * 100 + i))
    return out


@pytest.mark.parametrize("w", _random_shapes(16, 1), ids=lambda w: w.name)
def test_layer_parity_random_shapes(oracle, w):
    """Seeded random small grids (1 to 1152 tokens), head counts, batch sizes, both head widths, random window sizes and
    head orders: the whole layer against the oracle, and the benchmark launch bit-equal to the call with per-branch outputs."""
    rng = np.random.default_rng(w.seed)
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = rng.integers(0, 2, size=w.H).astype(np.uint8)
    kept = [int(rng.integers(1, w.nb + 1)) for _ in range(w.H)]
    res = run_layer(w, inp, dev, kept, kinds)
    ref = _oracle_layer(oracle, w, inp, kept, kinds)
    assert np.array_equal(res["row_ptr"], ref["row_ptr"]) and np.array_equal(res["col_idx"], ref["col_idx"])
    assert np.abs(res["s"] - ref["s"]).max() < 2e-6
    compare_layer(res, ref, label=w.name)
    fast = run_layer(w, inp, dev, kept, kinds, dbg=False, prebuilt_lists=True)
    assert np.array_equal(fast["out"], res["out"])


def _random_shapes_d128(count, seed):
    rng = np.random.default_rng(seed)
    out = []
    for i in range(count):
        T, Hh, W = int(rng.integers(1, 9)), int(rng.integers(2, 13)), int(rng.integers(2, 13))
        H, B = int(rng.integers(1, 5)), int(rng.integers(1, 3))
        out.append(wl.small(f"randw{i}-T{T}x{Hh}x{W}-H{H}-B{B}", B, H, 128, T, Hh, W, "bf16", 0.5, seed=2000 + seed * 100 + i))
    return out


@pytest.mark.parametrize("w", _random_shapes_d128(12, 2), ids=lambda w: w.name)
def test_widened_rows_random_shapes(oracle, w):
    """Seeded random small shapes through the widened rows and their combinations: rotary linear branch (fused and with
    the separate apply pass), full projection with and without the rotation, Top-K masks (mixed head orders; mask bit for
    bit), each against the oracle."""
    rng = np.random.default_rng(w.seed)
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = rng.integers(0, 2, size=w.H).astype(np.uint8)
    kept = [int(rng.integers(1, w.nb + 1)) for _ in range(w.H)]
    cs, sn = wl.rope_tables(w.T, w.Hh, w.W, w.d)
    rope_dev = (torch.from_numpy(cs).cuda(), torch.from_numpy(sn).cuda())
    flags = sb.SALAD_FLAG_UNFUSED_EPILOGUE if rng.integers(0, 2) else 0
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=10.0, rope=(cs, sn))
    res = run_layer(w, inp, dev, kept, kinds, lam=10.0, rope=rope_dev, flags=flags)
    compare_layer(res, ref, label=f"{w.name} rope flags={flags}")
    D = w.H * w.d
    wp = wl.round_to_bf16((wl.normal(w.seed, "w_proj", (D, D)) / np.sqrt(D) * 4.0).astype(np.float32))
    wp_dev = torch.from_numpy(wp).cuda().to(torch.bfloat16)
    with_rope = bool(rng.integers(0, 2))
    ref = _oracle_layer(oracle, w, inp, kept, kinds, w_proj=wp.astype(np.float64), rope=(cs, sn) if with_rope else None)
    res = run_layer(w, inp, dev, kept, kinds, head_scale=None, w_proj=wp_dev, rope=rope_dev if with_rope else None, dbg=False)
    compare_layer(res, ref, check_linear=False, label=f"{w.name} proj rope={with_rope}")
    key_block = int(rng.choice([64, 128]))
    nbk = -(-w.N // key_block)
    topk = int(rng.integers(1, min(8, nbk) + 1))
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=5.0, topk=topk, key_block=key_block)
    res = run_layer(w, inp, dev, kept, kinds, lam=5.0, topk=topk, topk_key_block=key_block)
    assert np.array_equal(res["topk_mask"], ref["topk_mask"])
    compare_layer(res, ref, label=f"{w.name} topk={topk}/{key_block}")
    # without the debug outputs (topk <= 4: the partial results are merged inside the linear-apply pass)
    fast = run_layer(w, inp, dev, kept, kinds, lam=5.0, topk=topk, topk_key_block=key_block, dbg=False)
    assert np.array_equal(fast["topk_mask"], ref["topk_mask"])
    compare_layer(fast, ref, check_linear=False, label=f"{w.name} topk={topk}/{key_block} fast")


def test_d64_large_tile_modes(oracle):
    """bf16 d = 64 on the large-tile kernel through the modes of the layer call: lambda = 0 (sparse branch alone, bit
    equal to what a pruned sample gets), branch dropping with B = 2, the unfused epilogue, a precomputed s, and an
    arbitrary CSR with an empty row."""
    w = SMALL[8]                                      # d64-ragged: N = 429, B = 2, 2 heads
    inp = wl.make_inputs(w)
    wg = inp["w_gate"]
    inp["x_t"] = inp["x_t"].copy()
    inp["x_t"][1] = wl.round_to_bf16(inp["x_t"][1] + (2.0 * wg / float(np.dot(wg, wg))).astype(np.float32))
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [3, 4]
    base = _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0)
    tau = float(0.5 * (base["s"][0] + base["s"][1]))
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0, drop_threshold=tau)
    assert ref["dropped"].tolist() == [1, 0]
    sparse_only = run_layer(w, inp, dev, kept, kinds, lam=0.0)
    compare_layer(sparse_only, _oracle_layer(oracle, w, inp, kept, kinds, lam=0.0), check_linear=False, label="d64 lambda=0")
    for flags in (0, sb.SALAD_FLAG_UNFUSED_EPILOGUE):
        res = run_layer(w, inp, dev, kept, kinds, lam=20.0, flags=flags, drop_threshold=tau)
        assert res["dropped"].tolist() == [1, 0]
        compare_layer(res, ref, check_linear=False, label=f"d64 drop flags={flags}")
        assert torch.equal(res["out_t"][0], sparse_only["out_t"][0])
        full = run_layer(w, inp, dev, kept, kinds, lam=20.0, flags=flags)
        compare_layer(full, base, label=f"d64 flags={flags}")
    s_fixed = np.array([0.25, 0.75], dtype=np.float32)
    res_s = run_layer(w, inp, dev, kept, kinds, lam=3.0, s=torch.from_numpy(s_fixed).cuda())
    compare_layer(res_s, _oracle_layer(oracle, w, inp, kept, kinds, lam=3.0, s_override=s_fixed.astype(np.float64)), label="d64 s_dev")
    rng = np.random.default_rng(9)
    rows = [np.sort(rng.choice(w.nb, size=int(rng.integers(0 if r == 2 else 1, 5)), replace=False)) for r in range(w.H * w.nb)]
    csr = (np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32), np.concatenate(rows).astype(np.int32))
    res_c = run_layer(w, inp, dev, None, kinds, csr=csr)
    o_s, rws = oracle.sparse_attn(inp["q"], inp["k"], inp["v"], (w.T, w.Hh, w.W), 64, kinds, *csr)
    got, ok = gather_rows(res_c["o_sparse"], rws)
    assert errors(got[ok], o_s[ok])[1] <= REL_L2


def test_branch_dropping_fp32(oracle):
    w = wl.small("drop-f32", 2, 2, 64, 3, 6, 8, "f32", 0.5, seed=112)       # N = 144
    inp = wl.make_inputs(w)
    wg = inp["w_gate"]
    inp["x_t"] = inp["x_t"].copy()
    inp["x_t"][0] += (2.0 * wg / float(np.dot(wg, wg))).astype(np.float32)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [2, 2]
    base = _oracle_layer(oracle, w, inp, kept, kinds, lam=5.0)
    tau = float(0.5 * (base["s"][0] + base["s"][1]))
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=5.0, drop_threshold=tau)
    res = run_layer(w, inp, dev, kept, kinds, lam=5.0, drop_threshold=tau)
    assert ref["dropped"].tolist() == [0, 1] and res["dropped"].tolist() == [0, 1]
    compare_layer(res, ref, check_linear=False, tol_abs=1e-4, tol_rel=1e-5, label="drop-f32")


PROJ_SHAPES = [
    SMALL[1],                                                                    # B = 2, H = 3 (odd: one output head per workgroup), N = 693
    wl.small("proj-even-heads", 2, 4, 128, 7, 9, 11, "bf16", 0.6, seed=112),     # H = 4: two output heads per workgroup, 3 row tiles, tail
]


@pytest.mark.parametrize("w", PROJ_SHAPES, ids=lambda w: w.name)
def test_full_projection(oracle, w):
    """Alg. 1 "Proj" as a full D x D matrix across heads: O_s + lambda s_b (O_l W_p), against the oracle; the
    block-diagonal W_p reproduces the per-head form; pruned samples stay the sparse branch."""
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4] * w.H
    D = w.H * w.d
    wp = wl.round_to_bf16((wl.normal(113, "w_proj", (D, D)) / np.sqrt(D)).astype(np.float32))
    wp_dev = torch.from_numpy(wp).cuda().to(torch.bfloat16)
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=25.0, w_proj=wp.astype(np.float64))
    ref_ps = _oracle_layer(oracle, w, inp, kept, kinds, lam=25.0)
    assert errors(ref["out"], ref_ps["out"])[1] > 0.05                 # the projection is not a small effect here
    res = run_layer(w, inp, dev, kept, kinds, lam=25.0, head_scale=None, w_proj=wp_dev)
    compare_layer(res, ref, check_linear=False, label="full-proj")
    # W_p rearranged once for the layer (salad_proj_pack) and handed in instead of w_proj: the same bits
    packed = sb.salad_proj_pack(wp_dev, w.H, w.d)
    res_p = run_layer(w, inp, dev, kept, kinds, lam=25.0, head_scale=None, w_proj_packed=packed)
    assert np.array_equal(res_p["out"], res["out"])
    # block-diagonal projection = per-head scalars (a_h representable in bf16)
    a = wl.round_to_bf16(inp["head_scale"])
    wd = torch.from_numpy(np.kron(np.diag(a), np.eye(w.d, dtype=np.float32)).astype(np.float32)).cuda().to(torch.bfloat16)
    res_d = run_layer(w, inp, dev, kept, kinds, lam=25.0, head_scale=None, w_proj=wd)
    res_h = run_layer(w, inp, dev, kept, kinds, lam=25.0, head_scale=torch.from_numpy(a).cuda())
    assert errors(res_d["out"], res_h["out"])[1] < 3e-3
    # with branch dropping: the pruned sample is the sparse branch alone
    tau = 2.0
    res_dr = run_layer(w, inp, dev, kept, kinds, lam=25.0, head_scale=None, w_proj=wp_dev, drop_threshold=tau)
    sparse_only = run_layer(w, inp, dev, kept, kinds, lam=0.0)["out_t"]
    assert res_dr["dropped"].tolist() == [1, 1] and torch.equal(res_dr["out_t"], sparse_only)


@pytest.mark.parametrize("B,H,grid,keep", [
    (1, 2, (1, 1, 40), 1),            # a block of 32 rows and one of 8
    (2, 3, (3, 5, 13), 3),            # 195 rows, tiles dealt by rows, two samples
    (1, 4, (5, 15, 26), 31),          # 1950 rows, tiles cut along their lists
    (1, 13, (21, 12, 20), 8),    # 5040 rows, 260 tiles: whole ones and dealt ones
    (1, 13, (21, 12, 20), 24),   # lists of 24 to 27: a round with the smaller products, and four tiles in pieces
])
def test_full_projection_input_from_the_attention_epilogue(oracle, B, H, grid, keep):
    """Without debug outputs the attention kernel itself writes the projection's operand: both head orders, ragged last blocks,
    whole, cut and dealt tiles against the oracle; a pruned sample stays the sparse branch bit for bit."""
    w = wl.small(f"emit-{B}-{H}-{grid}", B, H, 128, *grid, "bf16", 0.5, seed=130 + H)
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds, kept, D = wl.head_kinds(w), [keep] * H, H * 128
    wp = wl.round_to_bf16((wl.normal(131, "w_proj", (D, D)) / np.sqrt(D)).astype(np.float32))
    wp_dev = torch.from_numpy(wp).cuda().to(torch.bfloat16)
    # lambda 5: outputs stay below 2 in magnitude, where the two bf16 roundings are at most 2 x 2^-8 = 0.8e-2 of the 2e-2 bar; with 25
    # those of the first shape reach 6.7, where one rounding alone can take 2^-6 = 1.6e-2
    lam = 5.0
    sel = None if w.nb <= 31 else list(range(0, w.nb, 9)) + [w.nb - 1]
    ref = _oracle_layer(oracle, w, inp, kept, kinds, sel=sel, lam=lam, w_proj=wp.astype(np.float64))
    res = run_layer(w, inp, dev, kept, kinds, lam=lam, head_scale=None, w_proj=wp_dev, dbg=False)
    assert np.abs(ref["out"][ref["rows"] >= 0]).max() < 2
    compare_layer(res, ref, check_linear=False, label=w.name)
    pruned = run_layer(w, inp, dev, kept, kinds, lam=lam, head_scale=None, w_proj=wp_dev, dbg=False, drop_threshold=2.0)
    assert torch.equal(pruned["out_t"], run_layer(w, inp, dev, kept, kinds, lam=0.0, dbg=False)["out_t"])


@pytest.mark.parametrize("variant", [0, 1], ids=["regrouped", "token-mask"])
@pytest.mark.parametrize("wi,key_block,topk", [(1, 64, 4), (7, 128, 2), (0, 64, 8), (6, 64, 1), (4, 64, 3)],
                         ids=["N693-B2-kb64-k4", "N1170-kb128-k2", "N270-all-blocks", "single-token", "N512-k3"])
def test_topk_mask_layer(oracle, topk_variant, wi, key_block, topk, variant):
    """Top-K dynamic mask (App. A.1.2): the per-query block selection matches the oracle bit for bit (both sides
    take the decision in the same fixed float32 order), and the layer output on that mask meets the bf16 bar, for
    both attention paths (queries regrouped by key block and merged; token mask on ordinary query tiles)."""
    topk_variant(variant)
    w = SMALL[wi]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = np.zeros(w.H, dtype=np.uint8)               # Top-K works on the stored order
    kept = [1] * w.H                                    # unused by the Top-K path
    ref = _oracle_layer(oracle, w, inp, kept, kinds, topk=topk, key_block=key_block)
    res = run_layer(w, inp, dev, kept, kinds, topk=topk, topk_key_block=key_block)
    assert np.array_equal(res["topk_mask"], ref["topk_mask"])
    nbk = -(-w.N // key_block)
    pop = np.array([bin(int(x)).count("1") for x in res["topk_mask"].reshape(-1)])
    assert (pop == min(topk, nbk)).all()
    compare_layer(res, ref, label=f"topk-{w.name}")
    # the same call without the debug outputs
    fast = run_layer(w, inp, dev, kept, kinds, topk=topk, topk_key_block=key_block, dbg=False)
    compare_layer(fast, ref, label=f"topk-{w.name}-fast")
    assert np.array_equal(fast["topk_mask"], ref["topk_mask"])
    if topk >= nbk:                                      # every block kept: the dense layer
        dense = run_layer(w, inp, dev, [w.nb] * w.H, kinds)
        assert errors(res["out"], dense["out"])[1] < 5e-3   # two independently rounded bf16 results


@pytest.mark.parametrize("B,H,d,grid,keep,topk", [
    (1, 43, 128, (3, 15, 16), 5, 0),      # 129 whole tiles
    (1, 2, 128, (2, 7, 19), 4, 0),        # dealt by rows
    (1, 3, 128, (5, 13, 17), 18, 0),      # cut along their lists
    (1, 43, 64, (3, 15, 16), 5, 0), (1, 2, 64, (2, 7, 19), 4, 0), (1, 3, 64, (5, 13, 17), 18, 0),
    (1, 43, 64, (4, 17, 19), 9, 0),       # 64 queries a wave: whole
    (1, 58, 64, (4, 23, 25), 36, 0),      # and cut
    (1, 3, 128, (5, 13, 17), 1, 3), (1, 3, 128, (5, 13, 17), 1, -3),     # Top-K: regrouped, token mask
], ids=lambda x: str(x).replace(" ", ""))
def test_non_finite_query_rows_stay_alone(topk_variant, B, H, d, grid, keep, topk):
    """A query row with a NaN, an infinity or values that overflow costs nobody else anything: every other row has the bits of
    the same call without it.  Key magnitudes rise and fall between blocks, so that references move in good rows as well."""
    N = grid[0] * grid[1] * grid[2]
    g = torch.Generator(device="cuda").manual_seed(N + d)
    q, k, v = (torch.randn(B, H, N, d, generator=g, device="cuda") for _ in range(3))
    k *= torch.tensor([1.0, 12.0, 2.0, 20.0, 5.0], device="cuda")[(torch.arange(N, device="cuda") // 64 * 7 + 3) % 5][:, None]
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    x, wg = torch.randn(B, N, H * d, generator=g, device="cuda").to(torch.bfloat16), torch.randn(H * d, generator=g, device="cuda") * 0.02
    bad = torch.zeros(B, H, N, dtype=torch.bool, device="cuda")
    q_bad = q.clone()
    for h in range(H):
        for first, value in ((3, float("nan")), (40, float("inf")), (71, -float("inf")), (101, 3e38), (N - 1, float("nan"))):
            n = (first + 5 * h) % N
            q_bad[:, h, n, (7 * h) % d:(7 * h) % d + 2] = value
            bad[:, h, n] = True
    rp, ci = sb.salad_block_mask(*grid, 64, [keep] * H)
    kw = dict(x_t=x, w_gate=wg, lam=0.5, eps=1e-6)
    kinds = [0 if topk else h % 2 for h in range(H)]
    if topk:
        topk_variant(0 if topk > 0 else 1)
        kw.update(topk=abs(topk), topk_key_block=64)
    for dbg in (False, True):
        outs = []
        for t in (q, q_bad):
            more = dict(o_sparse_dbg=torch.zeros(B, H, N, d, device="cuda"), o_linear_dbg=torch.zeros(B, H, N, d, device="cuda")) if dbg else {}
            outs.append([sb.salad_sparse_linear_attn_fwd(t, k, v, grid, rp, ci, kinds, **kw, **more)] + list(more.values()))
        for clean, got in zip(*outs):
            assert bool(torch.isfinite(clean).all())
            assert torch.equal(got[~bad], clean[~bad]), int((got[~bad] != clean[~bad]).any(-1).sum())
        assert bool(torch.isnan(outs[1][0][:, torch.arange(H), (3 + 5 * torch.arange(H)) % N]).any(-1).all())


def test_token_mask_rows_beside_a_row_out_of_range(oracle, topk_variant):
    """Before a query has a softmax reference, logits 150 to 300 binades above 0 make its first sum infinite; the queries next to it
    in the wave did not select that block and must not notice.  Neighbours take different blocks, whose keys point along a
    channel of their own; the same call on the regrouped path, which never has both in one tile."""
    w = wl.small("beside", 2, 2, 128, 4, 12, 16, "bf16", 0.5, seed=645)      # N = 768: 12 blocks
    inp = wl.make_inputs(w)
    blk = np.arange(w.N) // 64
    inp["k"] = inp["k"] * np.float32(0.25)
    inp["k"][:, :, np.arange(w.N), blk] += 32 + 4.0 * (blk % 3)
    for i in range(2):                                     # two blocks of its own for every query, others for the next 15 and for the one 16 on
        inp["q"][:, :, np.arange(w.N), (np.arange(w.N) % 16 + np.arange(w.N) // 16 * 3 + 5 * i) % w.nb] += 48 - 8 * i
    for t in ("q", "k"):
        inp[t] = wl.round_to_bf16(inp[t].astype(np.float32))
    inp["v"] = inp["v"] * np.float32(0.25)                 # two bf16 roundings of values up to 4.5 would take the absolute bar; exact in bf16
    dev = upload(w, inp)
    kinds = np.zeros(w.H, dtype=np.uint8)
    ref = _oracle_layer(oracle, w, inp, [1] * w.H, kinds, topk=2, key_block=64)
    for variant in (0, 1):
        topk_variant(variant)
        for dbg in (True, False):
            res = run_layer(w, inp, dev, [1] * w.H, kinds, topk=2, topk_key_block=64, dbg=dbg)
            assert np.array_equal(res["topk_mask"], ref["topk_mask"])
            compare_layer(res, ref, label=f"variant {variant}")


@pytest.mark.parametrize("wi,key_block,topk", [(1, 64, 4), (7, 128, 2), (5, 64, 3), (0, 64, 2)],
                         ids=["N693-B2-kb64-k4", "N1170-kb128-k2", "T70-gt-block-k3", "N270-tail14-k2"])
def test_topk_mask_temporal_heads(oracle, wi, key_block, topk):
    """Top-K with temporal heads (App. A.1.1 order inside App. A.1.2): the key blocks of an odd head are runs of its
    location-major order, so its block means, its selection and the keys it attends to differ from the stored-order
    ones; mask bit for bit, output to the bf16 bar, ragged last key block included."""
    w = SMALL[wi]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    assert kinds.any() and w.T > 1
    kept = [1] * w.H
    ref = _oracle_layer(oracle, w, inp, kept, kinds, topk=topk, key_block=key_block)
    ref_stored = _oracle_layer(oracle, w, inp, kept, np.zeros(w.H, dtype=np.uint8), topk=topk, key_block=key_block)
    assert not np.array_equal(ref["topk_mask"], ref_stored["topk_mask"])          # the order matters on these inputs
    res = run_layer(w, inp, dev, kept, kinds, topk=topk, topk_key_block=key_block)
    assert np.array_equal(res["topk_mask"], ref["topk_mask"])
    compare_layer(res, ref, label=f"topk-temporal-{w.name}")
    fast = run_layer(w, inp, dev, kept, kinds, topk=topk, topk_key_block=key_block, dbg=False)
    compare_layer(fast, ref, label=f"topk-temporal-{w.name}-fast")


@pytest.mark.parametrize("flags", [0, sb.SALAD_FLAG_UNFUSED_EPILOGUE], ids=["fused", "unfused"])
@pytest.mark.parametrize("wi", [1, 7, 0, 4], ids=["N693-B2", "N1170", "N270-tail14", "N512"])
def test_rotary_linear_branch(oracle, wi, flags):
    """RoPE inside the linear branch (Sec. 4.1; numerator rotated, normaliser not): the layer against the oracle,
    with a static scale large enough that the linear branch carries weight; zero angles reproduce the plain layer.
    fused: the attention kernel's epilogue rotates relu(Q) in registers; unfused: the separate apply kernel does."""
    w = SMALL[wi]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [3] * w.H if w.nb >= 3 else [1] * w.H
    cs, sn = wl.rope_tables(w.T, w.Hh, w.W, w.d)
    rope_dev = (torch.from_numpy(cs).cuda(), torch.from_numpy(sn).cuda())
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0, rope=(cs, sn))
    ref_plain = _oracle_layer(oracle, w, inp, kept, kinds, lam=20.0)
    res = run_layer(w, inp, dev, kept, kinds, lam=20.0, rope=rope_dev, flags=flags)
    compare_layer(res, ref, label=f"rope-{w.name}")
    fast = run_layer(w, inp, dev, kept, kinds, lam=20.0, rope=rope_dev, flags=flags, dbg=False)
    assert np.array_equal(fast["out"], res["out"])
    if w.N > 1:
        assert errors(ref["o_linear"], ref_plain["o_linear"])[1] > 0.05          # the rotation is not a small effect
    one = torch.ones_like(rope_dev[0]); zero = torch.zeros_like(rope_dev[0])
    res0 = run_layer(w, inp, dev, kept, kinds, lam=20.0, rope=(one, zero), flags=flags)
    plain = run_layer(w, inp, dev, kept, kinds, lam=20.0, flags=flags)
    assert torch.equal(res0["out_t"], plain["out_t"])                            # identity rotation: the same bits


@pytest.mark.parametrize("keep", [8, 24])
def test_rotary_linear_branch_in_calls_of_more_than_a_round(oracle, keep):
    """260 tiles of 5040 rows: with lists of 24 to 27 the smaller products rotate their queries, and the four tiles of the last round, in pieces, theirs."""
    w = wl.small("rope-columns", 1, 13, 128, 21, 12, 20, "bf16", 0.5, seed=144)
    inp = wl.make_inputs(w)
    dev, kinds, kept = upload(w, inp), wl.head_kinds(w), [keep] * w.H
    cs, sn = wl.rope_tables(w.T, w.Hh, w.W, w.d)
    rope_dev = (torch.from_numpy(cs).cuda(), torch.from_numpy(sn).cuda())
    ref = _oracle_layer(oracle, w, inp, kept, kinds, sel=list(range(0, w.nb, 9)) + [w.nb - 1], lam=20.0, rope=(cs, sn))
    res = run_layer(w, inp, dev, kept, kinds, lam=20.0, rope=rope_dev)
    compare_layer(res, ref, label="rope-columns")
    assert torch.equal(run_layer(w, inp, dev, kept, kinds, lam=20.0, rope=rope_dev, dbg=False)["out_t"], res["out_t"])


@pytest.mark.parametrize("w", PROJ_SHAPES, ids=lambda w: w.name)
def test_full_projection_with_rotary_linear_branch(oracle, w):
    """Alg. 1 "Proj" as a full matrix over the rotary linear branch (the paper's layer has both): the emit pass writes the
    rotated O_l, the GEMM projects it; small shapes with B = 2 and a ragged tail, against the oracle."""
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [3, 4, 3, 4][:w.H]
    D = w.H * w.d
    wp = wl.round_to_bf16((wl.normal(w.seed, "w_proj", (D, D)) / np.sqrt(D) * 8.0).astype(np.float32))
    wp_dev = torch.from_numpy(wp).cuda().to(torch.bfloat16)
    cs, sn = wl.rope_tables(w.T, w.Hh, w.W, w.d)
    rope_dev = (torch.from_numpy(cs).cuda(), torch.from_numpy(sn).cuda())
    res = run_layer(w, inp, dev, kept, kinds, head_scale=None, w_proj=wp_dev, rope=rope_dev, dbg=False)
    ref = _oracle_layer(oracle, w, inp, kept, kinds, w_proj=wp.astype(np.float64), rope=(cs, sn))
    ref_plain = _oracle_layer(oracle, w, inp, kept, kinds, w_proj=wp.astype(np.float64))
    assert errors(ref["out"], ref_plain["out"])[1] > 1e-2             # the rotation changes the projected branch
    compare_layer(res, ref, check_linear=False, label="proj+rope")


def test_wan13_480p_rotary_sampled(oracle):
    """The rotary linear branch at the headline size: full rotated state and sampled rows against the oracle."""
    w = wl.WAN13_480P
    say("480p-rope: generating inputs")
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [sb.salad_kept_from_sparsity(w.nb, w.sparsity)] * w.H
    cs, sn = wl.rope_tables(w.T, w.Hh, w.W, w.d)
    rope_dev = (torch.from_numpy(cs).cuda(), torch.from_numpy(sn).cuda())
    say("480p-rope: GPU call")
    res = run_layer(w, inp, dev, kept, kinds, rope=rope_dev)
    sel = wl.sample_blocks(w.nb, 4, w.seed)
    say(f"480p-rope: oracle on {len(sel)} query blocks per head")
    ref = _oracle_layer(oracle, w, inp, kept, kinds, sel=sel, rope=(cs, sn))
    compare_layer(res, ref, label="480p-rope")
    assert np.isfinite(res["out"]).all()


@pytest.mark.parametrize("grid,key_block", [((70, 2, 3), 192), ((64, 3, 5), 320), ((21, 5, 6), 192), ((2, 15, 17), 128)],
                         ids=["frames-over-64-tail36", "64-frames", "21-frames-tail54", "2-frames-tail126"])
def test_topk_means_walk_the_temporal_order(oracle, grid, key_block):
    """Mean keys over several steps of 64 positions, where the frame count is above, equal to and below the step, with last
    key blocks whose remainder goes by eights and ones; the selection turns on every bit of the means, so masks are exact."""
    w = wl.small("topk-means", 1, 2, 128, *grid, "bf16", 0.5, seed=307)
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = np.array([0, 1], dtype=np.uint8)
    kept = [1] * w.H
    ref = _oracle_layer(oracle, w, inp, kept, kinds, topk=1, key_block=key_block)
    res = run_layer(w, inp, dev, kept, kinds, topk=1, topk_key_block=key_block)
    assert np.array_equal(res["topk_mask"], ref["topk_mask"])
    compare_layer(res, ref, label=f"topk-means-T{w.T}")


@pytest.mark.parametrize("grid,key_block,topk", [((10, 10, 20), 64, 5), ((10, 20, 20), 64, 4), ((7, 11, 13), 192, 6),
                                                 ((16, 16, 16), 64, 8), ((4, 33, 31), 64, 8)],
                         ids=["32-key-blocks-k5", "63-key-blocks-k4", "6-key-blocks-k6-all", "64-key-blocks-k8",
                              "64-key-blocks-ragged-k8"])
def test_topk_selection_kernel_instantiations(oracle, grid, key_block, topk):
    """Shapes that reach the other instantiations of the selection kernel (up to 32 and up to 64 key blocks, four
    and eight kept slots), a ragged everything (N = 2000, 4000, 1001) and the limits: 64 key blocks (bit 63 of the
    mask word) with 8 kept, N = 4096 and N = 4092 (last key block of 60 tokens)."""
    w = wl.small("topk-shapes", 1, 2, 128, *grid, "bf16", 0.5, seed=211 + topk)
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = np.zeros(w.H, dtype=np.uint8)
    kept = [1] * w.H
    ref = _oracle_layer(oracle, w, inp, kept, kinds, topk=topk, key_block=key_block)
    res = run_layer(w, inp, dev, kept, kinds, topk=topk, topk_key_block=key_block)
    assert np.array_equal(res["topk_mask"], ref["topk_mask"])
    compare_layer(res, ref, label=f"topk-N{w.N}-kb{key_block}-k{topk}")


@pytest.mark.parametrize("H,grid,key_block,topk", [
    (2, (1, 5, 100), 64, 4),          # 8 blocks
    (1, (3, 9, 13), 64, 5),           # 6 blocks: one is left out; 5 of 8 slots; a last workgroup of 95 queries
    (2, (1, 4, 128), 64, 8),          # all of 8 blocks
    (1, (4, 16, 33), 64, 4),          # 33 blocks: a second tile of one row
    (2, (4, 32, 32), 64, 1),          # 64 blocks
])
@pytest.mark.parametrize("kind", ["normal", "ties", "one block in all", "zero queries", "wide range", "infinite", "cancelling", "cancelling, small",
                                  "leading channel", "common part"])
def test_topk_scores_from_the_matrix_cores(oracle, H, grid, key_block, topk, kind):
    """Masks bit for bit where scores from the matrix cores cannot decide, for a few queries of a wave and for all of them: equal means, zero
    queries, values at both ends of bf16, infinite ones; scores that are nothing but rounding, also where the product of the squared norms is
    below what fp32 holds; partial sums that are at full size from the first channel on; means that differ little from each other."""
    N, d = grid[0] * grid[1] * grid[2], 128
    q, k = (wl.round_to_bf16(wl.normal(77 + N, t, (1, H, N, d))) for t in ("q", "k"))
    if kind == "ties":
        k[:, :, key_block:2 * key_block] = k[:, :, :key_block]        # the first two blocks, for every query that one of them is last for
        q[:, :, ::17] = np.round(q[:, :, ::17])
    elif kind == "one block in all":
        k[:] = np.resize(k[0, 0, 0], k.shape)
    elif kind == "zero queries":
        q[:, :, 5:300] = 0
    elif kind == "wide range":
        q *= np.where(np.arange(N) % 3 == 0, 1e-30, 1e18).astype(np.float32)[:, None]
        k *= np.where(np.arange(N) // key_block % 2 == 0, 1e-19, 1e-3).astype(np.float32)[:, None]
        q, k = wl.round_to_bf16(q), wl.round_to_bf16(k)
    elif kind == "infinite":
        k[0, 0, N // 2, 3] = np.inf
        q[0, 0, 70:90, 3] = np.inf                                      # the same channel: scores are infinite, none is a NaN
    elif kind.startswith("cancelling"):                                 # channel c + 64 of the product is minus channel c
        scale = np.float32(1e-13 if kind.endswith("small") else 1)
        q[..., 64:], k[..., 64:] = q[..., :64], -k[..., :64]
        q, k = wl.round_to_bf16(q * scale), wl.round_to_bf16(k * scale)
    elif kind == "leading channel":
        # the first product is 1, and each of the next 126 is a little more than half a unit in the last place (the chain rounds up) or, where the
        # block is among the first topk, less (down); those are ahead by the last one, up to 1.2e-4, the same for the 64 queries of a wave, of which
        # the chain takes away 1.5e-5
        J, n = np.arange(N) // key_block, np.arange(N)
        ahead = J < topk
        q[:], k[:] = 2.0 ** -12, (2.0 ** -12 * (1 + np.where(ahead, -1, 1) / 64))[:, None]
        q[..., 0], k[..., 0] = 1, 1
        q[..., 127], k[..., 127] = 2.0 ** -12 * 12 * (n // 64 * 64 / N), np.where(ahead, 0.04, 0)
        q, k = wl.round_to_bf16(q), wl.round_to_bf16(k)
    elif kind == "common part":
        k = wl.round_to_bf16(k + np.float32(10) * np.sign(np.sin(np.arange(d) * 1.7 + 0.5)).astype(np.float32))
    ref = oracle.topk_select(q, k, key_block, topk, [0] * H, grid)
    got = torch.zeros((1, H, N), dtype=torch.int64, device="cuda")
    qd, kd = (torch.from_numpy(x).cuda().bfloat16() for x in (q, k))
    sb.salad_sparse_linear_attn_fwd(qd, kd, kd, grid, None, None, [0] * H, lam=0.0, topk=topk, topk_key_block=key_block, topk_mask_out=got)
    torch.cuda.synchronize()
    same = got.cpu().numpy().view(np.uint64) == ref
    assert same.all(), (kind, int((~same).sum()), np.argwhere(~same)[:4].tolist())


def test_topk_rotary_dropping_together(oracle):
    """The widened pieces in one call: Top-K mask for the sparse branch, rotary linear branch, and branch dropping
    with a threshold between the two samples' dynamic scales (sample 0 keeps its branch, sample 1 loses it)."""
    w = SMALL[1]                                        # B = 2, H = 3, N = 693
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = np.zeros(w.H, dtype=np.uint8)
    kept = [1] * w.H
    cs, sn = wl.rope_tables(w.T, w.Hh, w.W, w.d)
    rope_dev = (torch.from_numpy(cs).cuda(), torch.from_numpy(sn).cuda())
    s = oracle.gate(inp["x_t"], inp["w_gate"], 0.0)
    tau = float(0.5 * (s.min() + s.max()))
    assert s.min() < tau < s.max()
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=10.0, topk=3, key_block=128, rope=(cs, sn), drop_threshold=tau)
    res = run_layer(w, inp, dev, kept, kinds, lam=10.0, topk=3, topk_key_block=128, rope=rope_dev, drop_threshold=tau)
    assert res["dropped"].tolist() == ref["dropped"].tolist() and sorted(res["dropped"].tolist()) == [0, 1]
    assert np.array_equal(res["topk_mask"], ref["topk_mask"])
    compare_layer(res, ref, check_linear=False, label="topk+rope+drop")
    b_drop = int(np.argmax(ref["dropped"]))
    sparse_only = run_layer(w, inp, dev, kept, kinds, lam=0.0, topk=3, topk_key_block=128)["out_t"]
    assert torch.equal(res["out_t"][b_drop], sparse_only[b_drop])
    # the same call without the debug outputs
    fast = run_layer(w, inp, dev, kept, kinds, lam=10.0, topk=3, topk_key_block=128, rope=rope_dev, drop_threshold=tau, dbg=False)
    compare_layer(fast, ref, check_linear=False, label="topk+rope+drop-fast")
    assert torch.equal(fast["out_t"][b_drop], sparse_only[b_drop])


@pytest.mark.parametrize("topk,key_block", [(4, 64), (2, 128), (1, 64)], ids=["k4", "k2", "k1"])
def test_topk_merge_inside_the_apply_pass(oracle, topk, key_block):
    """Regrouped Top-K path without debug outputs, projection or rotation: the partial results of a query are merged
    by the linear-apply pass itself (fp32, one rounding of the sum).  Against the oracle, with one of the two samples
    pruned (Sec. 4.3): that sample must come out as the merge kernel writes it for lambda = 0, bit for bit, and the
    call with debug outputs (merge kernel, then the apply pass) must agree with the oracle as well."""
    w = SMALL[1]                                        # B = 2, H = 3, N = 693: three passes of 256 rows, ragged
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = np.zeros(w.H, dtype=np.uint8)
    kept = [1] * w.H
    s = oracle.gate(inp["x_t"], inp["w_gate"], 0.0)
    tau = float(0.5 * (s.min() + s.max()))
    ref = _oracle_layer(oracle, w, inp, kept, kinds, lam=10.0, topk=topk, key_block=key_block, drop_threshold=tau)
    ref_all = _oracle_layer(oracle, w, inp, kept, kinds, lam=10.0, topk=topk, key_block=key_block)
    fast = run_layer(w, inp, dev, kept, kinds, lam=10.0, topk=topk, topk_key_block=key_block, drop_threshold=tau, dbg=False)
    assert fast["dropped"].tolist() == ref["dropped"].tolist() and sorted(fast["dropped"].tolist()) == [0, 1]
    assert np.array_equal(fast["topk_mask"], ref["topk_mask"])
    compare_layer(fast, ref, check_linear=False, label="topk-merge-in-apply+drop")
    b_drop = int(np.argmax(ref["dropped"]))
    sparse_only = run_layer(w, inp, dev, kept, kinds, lam=0.0, topk=topk, topk_key_block=key_block, dbg=False)["out_t"]
    assert torch.equal(fast["out_t"][b_drop], sparse_only[b_drop])
    assert not torch.equal(fast["out_t"][1 - b_drop], sparse_only[1 - b_drop])
    # nobody pruned: both ways of merging against the oracle, and against each other (they differ by one bf16 rounding of O_s)
    fast_all = run_layer(w, inp, dev, kept, kinds, lam=10.0, topk=topk, topk_key_block=key_block, dbg=False)
    slow_all = run_layer(w, inp, dev, kept, kinds, lam=10.0, topk=topk, topk_key_block=key_block)
    e_fast = compare_layer(fast_all, ref_all, check_linear=False, label="topk-merge-in-apply")["out"]
    e_slow = compare_layer(slow_all, ref_all, label="topk-merge-kernel")["out"]
    assert e_fast[1] <= e_slow[1] * 1.05               # one rounding less cannot be less accurate
    assert errors(fast_all["out"], slow_all["out"])[1] < 5e-3


@pytest.fixture
def topk_variant():
    yield lambda v: sb.salad_tune("topk_variant", v)
    sb.salad_tune("topk_variant", 0)


def test_layer_call_under_graph_capture():
    """The layer call allocates nothing and never synchronises, so it can be captured into a HIP graph.
    Replays (with eager work and synchronisation in between) give the bits of the eager call."""
    w = SMALL[7]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4, 5, 4]
    eager = run_layer(w, inp, dev, kept, kinds, dbg=False)["out_t"].clone()
    grid = (w.T, w.Hh, w.W)
    row_ptr, col_idx = sb.salad_block_mask(*grid, w.block, kept)
    q, k, v = dev["q"], dev["k"], dev["v"]
    out = torch.zeros_like(q)
    ws = sb.Workspace(w.B, w.H, w.N, w.d, sb.SALAD_BF16, q.device)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        p, keep = sb.make_fwd_params(q, k, v, out, grid, row_ptr, col_idx, kinds, lam=w.lam, head_scale=dev["head_scale"],
                                     x_t=dev["x_t"], w_gate=dev["w_gate"], eps=w.eps, workspace=ws)
        sb.salad_fwd_call(p)
    for rep in range(3):
        out.fill_(float("nan"))                      # eager work between replays
        (dev["x_t"].float().sum()).item()            # ... and a synchronisation
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), f"replay {rep} differs from the eager call"


def test_stream_handle_is_the_current_streams():
    side = torch.cuda.Stream()
    assert sb._stream() == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert sb._stream() == side.cuda_stream
    assert sb._stream() == torch.cuda.current_stream().cuda_stream


def test_timing_modes_leave_results_alone():
    """Per-stage timing (mode 1), attention-only timing (mode 2) and no timing give the same bits; mode 2 reports
    the attention stage alone."""
    w = SMALL[7]
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [4, 5, 4]
    ref = run_layer(w, inp, dev, kept, kinds, dbg=False)["out_t"].clone()
    try:
        for mode in (1, 2):
            sb.salad_timing_read(reset=True)
            sb.salad_timing_enable(mode)
            outs = [run_layer(w, inp, dev, kept, kinds, dbg=False)["out_t"].clone() for _ in range(3)]
            sb.salad_timing_enable(0)
            kt = sb.salad_timing_read(reset=True)
            assert all(torch.equal(o, ref) for o in outs)
            assert kt.calls == 3 and kt.attn_ms > 0
            if mode == 1:
                assert kt.gate_ms > 0 and kt.state_ms > 0 and kt.finalize_ms > 0
            else:
                assert kt.gate_ms == 0 and kt.state_ms == 0 and kt.finalize_ms == 0 and kt.epilogue_ms == 0
    finally:
        sb.salad_timing_enable(0)
        sb.salad_timing_read(reset=True)


# ------------------------------------------------------------------- benchmark configurations

def _sampled_parity(oracle, w, nsel, label):
    say(f"{label}: generating inputs N={w.N} H={w.H}")
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [sb.salad_kept_from_sparsity(w.nb, w.sparsity)] * w.H
    say(f"{label}: GPU call, kept={kept[0]} of {w.nb}")
    res = run_layer(w, inp, dev, kept, kinds)
    sel = wl.sample_blocks(w.nb, nsel, w.seed)
    say(f"{label}: oracle on {len(sel)} query blocks per head")
    ref = _oracle_layer(oracle, w, inp, kept, kinds, sel=sel)
    assert np.array_equal(res["row_ptr"], ref["row_ptr"]) and np.array_equal(res["col_idx"], ref["col_idx"])
    assert np.abs(res["s"] - ref["s"]).max() < 2e-6
    compare_layer(res, ref, label=label)
    # properties that hold at any size: finite everywhere, every row written
    assert np.isfinite(res["out"]).all() and np.isfinite(res["o_sparse"]).all() and np.isfinite(res["o_linear"]).all()
    # the launch the benchmark times (no per-branch outputs: results leave through LDS as whole rows) gives the same
    # bits as the call above with its per-lane stores
    say(f"{label}: benchmark launch (no per-branch outputs)")
    fast = run_layer(w, inp, dev, kept, kinds, dbg=False)
    assert np.array_equal(fast["out"], res["out"])
    return res, ref, inp, dev, kinds, kept


def test_mid_config_sampled(oracle):
    _sampled_parity(oracle, wl.MID, 12, "mid")


def test_d64_large_tile_kernel_sampled(oracle):
    """bf16 d = 64 on the large-tile kernel at a size that fills the chip (N = 12480: 195 blocks, tail 0, 24 heads,
    odd heads temporal): sampled query blocks against the oracle, the benchmark launch bit-equal to the call with
    per-branch outputs, prebuilt visit lists bit-equal too, and the first-generation d = 64 kernel (the fallback,
    selected through the knob) within the same bars."""
    w = wl.small("d64-mid", 1, 24, 64, 8, 30, 52, "bf16", 0.75, seed=113)
    res, ref, inp, dev, kinds, kept = _sampled_parity(oracle, w, 10, "d64-mid")
    pre = run_layer(w, inp, dev, kept, kinds, dbg=False, prebuilt_lists=True)
    assert np.array_equal(pre["out"], res["out"])
    sb.salad_tune("attn_variant", 2)
    try:
        old = run_layer(w, inp, dev, kept, kinds)
    finally:
        sb.salad_tune("attn_variant", 0)
    compare_layer(old, ref, label="d64-mid/first-generation")


@pytest.mark.timeout(600)
def test_wan13_480p_90_sampled(oracle):
    """The headline configuration at full size, in the launch configuration the benchmark times; the oracle
    evaluates every one of the 512 query blocks of every head (all 393 120 output rows are compared), plus the
    full linear state and gate."""
    res, ref, inp, dev, kinds, kept = _sampled_parity(oracle, wl.WAN13_480P, wl.WAN13_480P.nb, "480p-90")
    Hs, Z = sb.salad_linear_state_fwd(dev["k"], dev["v"])
    torch.cuda.synchronize()
    assert errors(Hs.cpu().numpy().astype(np.float64), ref["Hs"])[1] < 2e-6
    assert errors(Z.cpu().numpy().astype(np.float64), ref["Z"])[1] < 2e-6


def test_wan13_480p_full_projection_sampled(oracle):
    """Alg. 1 "Proj" with the full D x D matrix at the headline size (H = 12, N = 32760: 128 row tiles of the
    projection GEMM, the last one with 248 rows), in the launch configuration the benchmark times; the oracle
    evaluates sampled query blocks of every head (first, last = tail, middle, seeded picks)."""
    w = wl.WAN13_480P
    say("480p-proj: generating inputs")
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = wl.head_kinds(w)
    kept = [sb.salad_kept_from_sparsity(w.nb, w.sparsity)] * w.H
    D = w.H * w.d
    wp = wl.round_to_bf16((wl.normal(w.seed, "w_proj", (D, D)) / np.sqrt(D)).astype(np.float32))
    wp_dev = torch.from_numpy(wp).cuda().to(torch.bfloat16)
    say("480p-proj: GPU call")
    res = run_layer(w, inp, dev, kept, kinds, head_scale=None, w_proj=wp_dev, dbg=False)
    sel = wl.sample_blocks(w.nb, 4, w.seed)
    say(f"480p-proj: oracle on {len(sel)} query blocks per head")
    ref = _oracle_layer(oracle, w, inp, kept, kinds, sel=sel, w_proj=wp.astype(np.float64))
    ref_ps = _oracle_layer(oracle, w, inp, kept, kinds, sel=sel)
    assert errors(ref["out"], ref_ps["out"])[1] > 1e-3                 # the projection changes the result
    compare_layer(res, ref, check_linear=False, label="480p-proj")
    assert np.isfinite(res["out"]).all()


def test_wan13_480p_topk_sampled(oracle):
    """Top-K mask at the headline size and sparsity: 40 key blocks of 832 tokens (13 blocks of 64; the last one
    312 tokens), 4 kept per query token = 90 % sparsity.  The full mask is compared bit for bit, the output on
    sampled query blocks."""
    w = wl.WAN13_480P
    say("480p-topk: generating inputs")
    inp = wl.make_inputs(w)
    dev = upload(w, inp)
    kinds = np.zeros(w.H, dtype=np.uint8)
    kept = [1] * w.H
    say("480p-topk: GPU call")
    res = run_layer(w, inp, dev, kept, kinds, topk=4, topk_key_block=832, dbg=False)
    sel = wl.sample_blocks(w.nb, 4, w.seed)
    say(f"480p-topk: oracle selection for every query, attention on {len(sel)} query blocks per head")
    ref = _oracle_layer(oracle, w, inp, kept, kinds, sel=sel, topk=4, key_block=832)
    assert np.array_equal(res["topk_mask"], ref["topk_mask"])
    compare_layer(res, ref, check_linear=False, label="480p-topk")
    assert np.isfinite(res["out"]).all()


@pytest.mark.timeout(600)
@pytest.mark.parametrize("case", ["list-too-long", "inexact-division"])
def test_long_sequence_takes_the_fallback_by_itself(oracle, case):
    """Shapes the large-tile kernel does not take, so that the dispatcher has to pick the 128-row kernel without being
    told (the tuning knob stays at automatic).  list-too-long: 6152 key blocks per head, more than the per-tile block
    list may hold in LDS.  inexact-division: N T >= 2^32, where the temporal order's multiply-high division by T is no
    longer exact (the list would fit).  One spatial and one temporal head, 5 kept blocks per row, ragged last block."""
    if case == "list-too-long":
        w = wl.small("long-seq", 1, 2, 128, 31, 100, 127, "bf16", 1.0 - 5.0 / 6152.0, seed=131)
        assert w.N == 393700 and w.nb == 6152 and w.N % 64 == 36
    else:
        w = wl.small("long-T", 1, 2, 128, 11078, 5, 7, "bf16", 1.0 - 5.0 / 6059.0, seed=132)
        assert w.N == 387730 and w.nb == 6059 and w.N % 64 == 18 and w.N * w.T >= 1 << 32
        assert ((w.nb + 63) & ~63) * 4 <= 24 * 1024
    assert sb.salad_kept_from_sparsity(w.nb, w.sparsity) == 5
    _sampled_parity(oracle, w, 8, w.name)


@pytest.mark.timeout(600)
@pytest.mark.parametrize("nb,grid", [(3584, (40, 63, 91)), (3585, (40, 155, 37)), (3563, (19000, 3, 4))])
def test_edge_of_the_large_tile_kernel_at_d128(oracle, nb, grid):
    """d = 128: the large-tile kernel's rings leave room for lists of 3584 entries; the first sequence beyond has to go to the
    128-row kernel, lists passed in or not, and so does a shorter one whose temporal order it cannot divide (N T >= 2^32).  One
    spatial and one temporal head, 5 kept blocks per row, ragged last block."""
    w = wl.small(f"list-{nb}", 1, 2, 128, *grid, "bf16", 1.0 - 5.0 / nb, seed=133)
    assert w.nb == nb and w.N % 64 and sb.salad_kept_from_sparsity(nb, w.sparsity) == 5
    assert (w.N * w.T >= 1 << 32) == (nb == 3563)
    res, _, inp, dev, kinds, kept = _sampled_parity(oracle, w, 8, w.name)
    pre = run_layer(w, inp, dev, kept, kinds, dbg=False, prebuilt_lists=True)
    assert np.array_equal(pre["out"], res["out"])


@pytest.mark.parametrize("rho", [0.0, 0.5, 0.75, 0.95])
def test_wan13_480p_sweep_sampled(oracle, rho):
    """The other points of the sparsity sweep at the 480p shape (same seeded inputs)."""
    w = wl.WAN13_480P.with_sparsity(rho)
    _sampled_parity(oracle, w, 4 if rho < 0.7 else 8, f"480p-{rho:g}")


@pytest.mark.timeout(900)
def test_wan14_720p_90_sampled(oracle):
    """Wan-14B-shaped 720p configuration: H=40, N=75600 (16-token tail), gate over D=5120."""
    _sampled_parity(oracle, wl.WAN14_720P, 4, "720p-90")
