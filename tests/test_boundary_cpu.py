"""C-ABI checks that need no GPU: the library loads, exports every declared symbol, and rejects
bad arguments on the host before any HIP call."""
import ctypes as C
import os
import re

import pytest

from paper_2601_16515_amd import binding as sb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(sb.LIB_PATH):
        sb.build_library()
    return sb.lib()


def _declared_symbols():
    text = open(os.path.join(ROOT, "include", "salad.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(salad_[a-z_0-9]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = _declared_symbols()
    assert set(names) == set(sb.EXPORTS)
    for n in names:
        assert getattr(lib, n) is not None


def test_kept_from_sparsity_host_arithmetic(lib, oracle):
    for nb in (1, 2, 16, 195, 512, 1182):
        for rho in (0.0, 0.5, 0.75, 0.9, 0.95, 1.0, 0.333):
            assert sb.salad_kept_from_sparsity(nb, rho) == oracle.kept_from_sparsity(nb, rho)
    assert sb.salad_kept_from_sparsity(0, 0.5) == 0
    assert sb.salad_kept_from_sparsity(512, 0.9) == 51


def test_mask_nnz(lib):
    assert sb.salad_block_mask_nnz(21, 30, 52, 64, [51] * 12) == 313344
    assert sb.salad_block_mask_nnz(4, 16, 16, 64, [4, 4]) == 128
    assert sb.salad_block_mask_nnz(4, 16, 16, 64, [4, 17]) == -1
    assert sb.salad_block_mask_nnz(4, 16, 16, 64, [0, 4]) == -1
    assert sb.salad_block_mask_nnz(0, 16, 16, 64, [1]) == -1


def test_mask_nnz_of_the_truncated_window(lib, oracle):
    # the closed form of the header against the oracle's count, and the mode argument's range
    for grid, kept in (((21, 30, 52), [51] * 12), ((4, 16, 16), [4, 5]), ((5, 6, 9), [1, 5, 3]), ((3, 8, 8), [3, 3])):
        _, ci = oracle.block_mask(*grid, 64, kept, truncated=True)
        assert sb.salad_block_mask_nnz_mode(*grid, 64, kept, sb.SALAD_WINDOW_TRUNCATED) == len(ci)
        assert sb.salad_block_mask_nnz_mode(*grid, 64, kept, sb.SALAD_WINDOW_SHIFTED) == sb.salad_block_mask_nnz(*grid, 64, kept)
    assert sb.salad_block_mask_nnz_mode(4, 16, 16, 64, [4, 4], 2) == -1
    assert sb.salad_block_mask_nnz_mode(4, 16, 16, 64, [4, 17], sb.SALAD_WINDOW_TRUNCATED) == -1
    kept = (C.c_int32 * 2)(4, 4)
    fake = 0x1000   # never dereferenced
    assert lib.salad_block_mask_mode(4, 16, 16, 64, 2, kept, 7, fake, fake, 128, None) == sb.SALAD_EINVAL
    assert "window_mode" in lib.salad_last_error().decode()
    assert lib.salad_block_mask_mode(4, 16, 16, 64, 2, kept, sb.SALAD_WINDOW_TRUNCATED, fake, fake, 119, None) == sb.SALAD_ENOSPC    # nnz = 120
    assert lib.salad_block_mask_mode(4, 16, 16, 64, 2, kept, sb.SALAD_WINDOW_TRUNCATED, None, fake, 128, None) == sb.SALAD_EINVAL


def test_proj_pack_argument_errors(lib):
    assert lib.salad_proj_pack_bytes(12, 128) == 2 * (12 * 128) ** 2
    assert lib.salad_proj_pack_bytes(12, 64) == 0 and lib.salad_proj_pack_bytes(0, 128) == 0 and lib.salad_proj_pack_bytes(65, 128) == 0
    fake = 0x1000   # never dereferenced
    need = lib.salad_proj_pack_bytes(3, 128)
    assert lib.salad_proj_pack(None, 3, 128, fake, need, None) == sb.SALAD_EINVAL
    assert lib.salad_proj_pack(fake, 3, 64, fake, need, None) == sb.SALAD_ENOTSUP
    assert lib.salad_proj_pack(fake, 3, 128, fake + 16, need, None) == sb.SALAD_EINVAL
    assert "aligned" in lib.salad_last_error().decode()
    assert lib.salad_proj_pack(fake, 3, 128, fake, need - 1, None) == sb.SALAD_ENOSPC


def _err(lib):
    return lib.salad_last_error().decode()


def test_block_mask_argument_errors(lib):
    kept = (C.c_int32 * 2)(4, 4)
    fake = 0x1000   # never dereferenced: every check happens before the first HIP call
    assert lib.salad_block_mask(4, 16, 16, 64, 2, kept, None, fake, 128, None) == sb.SALAD_EINVAL
    assert "null" in _err(lib)
    assert lib.salad_block_mask(4, 16, 16, 32, 2, kept, fake, fake, 128, None) == sb.SALAD_ENOTSUP
    assert lib.salad_block_mask(4, 16, 16, 64, 2, kept, fake, fake, 127, None) == sb.SALAD_ENOSPC
    assert "127" in _err(lib)
    assert lib.salad_block_mask(4, 0, 16, 64, 2, kept, fake, fake, 128, None) == sb.SALAD_EINVAL
    bad = (C.c_int32 * 2)(4, 99)
    assert lib.salad_block_mask(4, 16, 16, 64, 2, bad, fake, fake, 1 << 20, None) == sb.SALAD_EINVAL
    many = (C.c_int32 * 65)(*([1] * 65))
    assert lib.salad_block_mask(4, 16, 16, 64, 65, many, fake, fake, 1 << 20, None) == sb.SALAD_ENOTSUP


def _params(**over):
    p = sb.FwdParams()
    p.B, p.H, p.N, p.d, p.dtype = 1, 2, 1024, 64, sb.SALAD_BF16
    p.T, p.Hh, p.W, p.block = 4, 16, 16, 64
    for f in ("q", "k", "v", "row_ptr", "col_idx", "x_t", "w_gate"):
        setattr(p, f, 0x1000)
    p.out = 0x2000
    p.workspace = 0x4000
    p.workspace_bytes = 1 << 30
    p.lam = 1.0
    p.eps = 1e-6
    for k, v in over.items():
        setattr(p, k, v)
    return p


@pytest.mark.parametrize("over,status,needle", [
    (dict(d=96), sb.SALAD_ENOTSUP, "d=96"),
    (dict(block=128), sb.SALAD_ENOTSUP, "block"),
    (dict(N=1000), sb.SALAD_EINVAL, "T*Hh*W"),
    (dict(q=None), sb.SALAD_EINVAL, "non-null"),
    (dict(out=0x1000), sb.SALAD_EINVAL, "alias"),
    (dict(row_ptr=None), sb.SALAD_EINVAL, "CSR"),
    (dict(phi=3), sb.SALAD_ENOTSUP, "feature map"),
    (dict(dtype=7), sb.SALAD_EINVAL, "dtype"),
    (dict(B=0), sb.SALAD_EINVAL, "positive"),
    (dict(H=65), sb.SALAD_ENOTSUP, "H=65"),
    (dict(eps=-1.0), sb.SALAD_EINVAL, "eps"),
    (dict(x_t=None), sb.SALAD_EINVAL, "s_dev"),
    (dict(workspace=None), sb.SALAD_EINVAL, "workspace"),
    (dict(workspace=0x4001), sb.SALAD_EINVAL, "aligned"),
    (dict(workspace_bytes=16), sb.SALAD_ENOSPC, "workspace"),
    (dict(flags=8), sb.SALAD_EINVAL, "flags"),
    (dict(flags=1, dtype=sb.SALAD_F32), sb.SALAD_ENOTSUP, "bf16"),
    (dict(lam=float("nan")), sb.SALAD_EINVAL, "lambda"),
    (dict(drop_threshold=float("nan")), sb.SALAD_EINVAL, "drop_threshold"),
    (dict(w_proj=0x8000), sb.SALAD_ENOTSUP, "w_proj"),                                   # d = 64
    (dict(w_proj=0x8000, d=128, head_scale=0x9000), sb.SALAD_EINVAL, "exclude"),
    (dict(w_proj_packed=0x8000), sb.SALAD_ENOTSUP, "w_proj"),                            # packed W_p alone, d = 64
    (dict(w_proj_packed=0x8000, d=128, head_scale=0x9000), sb.SALAD_EINVAL, "exclude"),
    (dict(w_proj_packed=0x8010, d=128), sb.SALAD_EINVAL, "w_proj_packed not 256-byte aligned"),
    (dict(topk=-1), sb.SALAD_EINVAL, "topk"),
    (dict(topk=4, topk_key_block=128), sb.SALAD_ENOTSUP, "d = 128"),                     # d = 64
    (dict(topk=9, topk_key_block=128, d=128), sb.SALAD_ENOTSUP, "above 8"),
    (dict(topk=4, topk_key_block=100, d=128), sb.SALAD_EINVAL, "multiple of 64"),
    (dict(topk=4, topk_key_block=0, d=128), sb.SALAD_EINVAL, "multiple of 64"),
    (dict(topk=4, topk_key_block=64, d=128, N=8192, T=32), sb.SALAD_ENOTSUP, "key blocks"),   # 128 key blocks
    (dict(topk=4, topk_key_block=128, d=128, workspace_bytes=1 << 16), sb.SALAD_ENOSPC, "workspace"),
    (dict(topk=4, topk_key_block=3648, d=128, N=229400, T=40, Hh=155, W=37, workspace_bytes=256), sb.SALAD_ENOTSUP, "too long"),   # 3585 blocks
    (dict(topk=4, topk_key_block=3648, d=128, N=229320, T=40, Hh=63, W=91, workspace_bytes=256), sb.SALAD_ENOSPC, "workspace"),    # 3584 blocks
    (dict(rope_cos=0xa000, d=128), sb.SALAD_EINVAL, "together"),                          # cosine table without the sine table
    (dict(rope_sin=0xa000, d=128), sb.SALAD_EINVAL, "together"),
    (dict(rope_cos=0xa000, rope_sin=0xb000), sb.SALAD_ENOTSUP, "rotary"),                # d = 64
    (dict(rope_cos=0xa000, rope_sin=0xb000, d=128, dtype=sb.SALAD_F32), sb.SALAD_ENOTSUP, "rotary"),
])
def test_fwd_argument_errors(lib, over, status, needle):
    p = _params(**over)
    assert lib.salad_sparse_linear_attn_fwd(C.byref(p)) == status
    assert needle in _err(lib)


def test_fwd_null_params_and_head_kind(lib):
    assert lib.salad_sparse_linear_attn_fwd(None) == sb.SALAD_EINVAL
    hk = (C.c_uint8 * 2)(0, 5)
    p = _params(head_kind_host=C.cast(hk, C.c_void_p))
    assert lib.salad_sparse_linear_attn_fwd(C.byref(p)) == sb.SALAD_EINVAL
    assert "head_kind" in _err(lib)


def test_topk_temporal_heads_and_csr_pointers(lib):
    hk = (C.c_uint8 * 2)(0, 1)
    # temporal heads are taken by the default (regrouped) Top-K path: the next check that fails is the workspace size
    p = _params(topk=2, topk_key_block=128, d=128, head_kind_host=C.cast(hk, C.c_void_p), workspace_bytes=256)
    assert lib.salad_sparse_linear_attn_fwd(C.byref(p)) == sb.SALAD_ENOSPC
    # the token-mask variant works on the stored order only
    assert lib.salad_tune(b"topk_variant", 1) == sb.SALAD_OK
    try:
        p = _params(topk=2, topk_key_block=128, d=128, head_kind_host=C.cast(hk, C.c_void_p))
        assert lib.salad_sparse_linear_attn_fwd(C.byref(p)) == sb.SALAD_ENOTSUP
        assert "stored token order" in _err(lib)
    finally:
        assert lib.salad_tune(b"topk_variant", 0) == sb.SALAD_OK
    # the CSR pointers may be null with topk: the next check that fails is a different one (workspace size)
    p = _params(topk=2, topk_key_block=128, d=128, row_ptr=None, col_idx=None, workspace_bytes=256)
    assert lib.salad_sparse_linear_attn_fwd(C.byref(p)) == sb.SALAD_ENOSPC


def test_workspace_query(lib):
    base = sb.salad_fwd_workspace_bytes(1, 12, 32760, 128, sb.SALAD_BF16)
    assert sb.salad_fwd_workspace_bytes(1, 12, 32760, 128, sb.SALAD_BF16, full_proj=True) > base + 2 * 12 * 32760 * 128
    assert sb.salad_fwd_workspace_bytes(1, 12, 32760, 128, sb.SALAD_BF16, topk=4) > base + 2 * 4 * 12 * 32760 * 128
    assert sb.salad_fwd_workspace_bytes(1, 12, 32760, 128, sb.SALAD_BF16) > 12 * (128 * 128 + 128) * 4
    assert sb.salad_fwd_workspace_bytes(1, 2, 1024, 64, sb.SALAD_F32) > 0
    assert sb.salad_fwd_workspace_bytes(1, 2, 1024, 96, sb.SALAD_BF16) == 0
    assert sb.salad_fwd_workspace_bytes(1, 2, 1024, 64, sb.SALAD_BF16) % 256 == 0


def test_state_chunks(lib):
    """The workspace holds one partial state per chunk of tokens: as many chunks as the knob asks for, except that its default leaves
    out those too short to be worth one, which depends on the head width."""
    def partial(BH, chunks, d):
        return BH * chunks * (d * d + d) * 4

    def more_chunks(BH, N, d, wgs, chunks):      # the workspace with the knob at wgs is larger by so many partial states a head
        rest = sb.salad_fwd_workspace_bytes(1, BH, N, d, sb.SALAD_BF16)
        try:
            sb.salad_tune("state_wgs", wgs)
            return abs(sb.salad_fwd_workspace_bytes(1, BH, N, d, sb.SALAD_BF16) - rest - partial(BH, chunks, d)) < 256
        finally:
            sb.salad_tune("state_wgs", 256)

    assert more_chunks(12, 1950, 128, 12 * 31, 31 - 8)            # 31 tiles, 4 a chunk by default
    assert more_chunks(12, 1950, 64, 12 * 31, 31 - 11)            # 3 a chunk
    assert more_chunks(2, 2000, 128, 4096, 32 - 16)
    assert more_chunks(40, 4096, 128, 257, 0)                     # 11 a chunk: what spreads 40 heads over the chip is longer already


def test_d64_tiles_just_past_a_round_are_cut(lib):
    """d = 64, 344 tiles: with lists of more than 28 blocks the 88 beyond a round of 256 are cut in two and the workspace has room for the
    pieces' results; with shorter lists, and from 385 tiles on, a round is 512 tiles and nothing is cut."""
    room = 88 * 2 * (256 * 64 * 4 + 512 * 8)
    long_lists, short_lists = (sb.salad_fwd_workspace_bytes(1, 43, nb * 64, 64, sb.SALAD_BF16) for nb in (29, 28))
    assert long_lists > room > short_lists
    assert sb.salad_fwd_workspace_bytes(1, 43, 36 * 64, 64, sb.SALAD_BF16) < room      # 387 tiles


def test_step_entry_points_reject_bad_arguments(lib):
    fake = 0x1000
    assert lib.salad_linear_state_fwd(None, fake, 1, 2, 64, 64, sb.SALAD_BF16, fake, fake, fake, 1 << 30, None) == sb.SALAD_EINVAL
    assert lib.salad_linear_state_fwd(fake, fake, 1, 2, 64, 48, sb.SALAD_BF16, fake, fake, 0x4000, 1 << 30, None) == sb.SALAD_EINVAL
    assert lib.salad_linear_state_fwd(fake, fake, 1, 2, 64, 64, sb.SALAD_BF16, fake, fake, 0x4000, 8, None) == sb.SALAD_ENOSPC
    assert lib.salad_gate_fwd(fake, fake, 0.0, 1, 64, 12, sb.SALAD_BF16, fake, 0x4000, 1 << 20, None) == sb.SALAD_EINVAL
    assert lib.salad_gate_fwd(fake, fake, 0.0, 1, 64, 8200, sb.SALAD_BF16, fake, 0x4000, 1 << 20, None) == sb.SALAD_ENOTSUP
    assert lib.salad_gate_fwd(fake, None, 0.0, 1, 64, 128, sb.SALAD_BF16, fake, 0x4000, 1 << 20, None) == sb.SALAD_EINVAL
    assert lib.salad_timing_read(None, 0) == sb.SALAD_EINVAL
    assert lib.salad_timing_enable(3) == sb.SALAD_EINVAL and lib.salad_timing_enable(-1) == sb.SALAD_EINVAL
    assert lib.salad_timing_enable(0) == sb.SALAD_OK
    assert lib.salad_tune(b"no_such_knob", 1) == sb.SALAD_EINVAL
    assert lib.salad_tune(None, 1) == sb.SALAD_EINVAL


def test_tune_keys_are_the_declared_ones_and_range_checked(lib):
    """Every key the header documents is accepted inside its range and refused outside; keys of earlier builds that the
    header does not declare are refused."""
    text = open(os.path.join(ROOT, "include", "salad.h")).read()
    declared = set(re.findall(r'^ \*\s+"([a-z_]+)"', text, flags=re.M))
    assert declared == {"state_wgs", "attn_variant", "topk_variant"}
    for key, ok, bad in ((b"state_wgs", (1, 512, 65536), (0, -3, 65537)), (b"attn_variant", (0, 1, 2), (-1, 3, 7, 5 + 16)),
                         (b"topk_variant", (0, 1), (-1, 2))):
        for v in bad:
            assert lib.salad_tune(key, v) == sb.SALAD_EINVAL, (key, v)
            assert "outside" in _err(lib)
        for v in ok:
            assert lib.salad_tune(key, v) == sb.SALAD_OK, (key, v)
    assert lib.salad_tune(b"state_wgs", 256) == sb.SALAD_OK and lib.salad_tune(b"attn_variant", 0) == sb.SALAD_OK
    assert lib.salad_tune(b"topk_variant", 0) == sb.SALAD_OK
    for key in (b"gate_parts", b"gate_tok"):
        assert lib.salad_tune(key, 1) == sb.SALAD_EINVAL


def test_tile_lists_argument_errors(lib):
    fake = 0x1000
    need = lib.salad_tile_lists_bytes(12, 512)
    assert need == 12 * 128 * 512 * 4 + 12 * 128 * 4 and need % 256 == 0
    assert lib.salad_tile_lists_bytes(12, 6145) == 0 and lib.salad_tile_lists_bytes(0, 8) == 0 and lib.salad_tile_lists_bytes(65, 8) == 0
    assert lib.salad_tile_lists(None, fake, 12, 512, 0x4000, need, None) == sb.SALAD_EINVAL
    assert lib.salad_tile_lists(fake, fake, 12, 512, 0x4001, need, None) == sb.SALAD_EINVAL
    assert lib.salad_tile_lists(fake, fake, 12, 512, 0x4000, need - 1, None) == sb.SALAD_ENOSPC
    assert lib.salad_tile_lists(fake, fake, 12, 7000, 0x4000, 1 << 30, None) == sb.SALAD_ENOTSUP
    p = _params(tile_lists=0x4010, d=128)
    assert lib.salad_sparse_linear_attn_fwd(C.byref(p)) == sb.SALAD_EINVAL and "tile_lists" in _err(lib)


def test_static_scratch_gate_argument_errors(lib):
    fake = 0x1000
    assert lib.salad_gate_fwd_static(None, fake, 0.0, 1, 64, 128, sb.SALAD_BF16, fake, None) == sb.SALAD_EINVAL
    assert lib.salad_gate_fwd_static(fake, fake, 0.0, 1, 64, 12, sb.SALAD_BF16, fake, None) == sb.SALAD_EINVAL
    assert lib.salad_gate_fwd_static(fake, fake, 0.0, 64, 32760, 128, sb.SALAD_BF16, fake, None) == sb.SALAD_ENOSPC
    assert "static" in _err(lib)


def test_binding_refuses_to_run_without_library(monkeypatch, tmp_path):
    monkeypatch.setattr(sb, "_lib", None)
    monkeypatch.setattr(sb, "LIB_PATH", str(tmp_path / "missing.so"))
    with pytest.raises(RuntimeError, match="no fallback"):
        sb.lib()


def test_product_does_not_import_the_oracle():
    pkg = os.path.join(ROOT, "paper_2601_16515_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "salad_oracle" not in text and "from oracle" not in text and "import oracle" not in text, f
    for f in os.listdir(os.path.join(ROOT, "oracle")):
        if f.endswith((".py", ".c")):
            text = open(os.path.join(ROOT, "oracle", f)).read()
            assert "paper_2601_16515_amd" not in text and "libsalad.so" not in text, f


def test_bench_refuses_more_than_one_gpu():
    """bench.py is a one-GPU program: any other --gpus value ends with a message before anything touches a device."""
    import subprocess
    import sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, os.path.join(root, "bench.py"), "--gpus", "2"], capture_output=True, text=True, timeout=60)
    assert r.returncode != 0
    assert "one GPU" in r.stderr and r.stdout.strip() == ""


def _kernel_metadata(path):
    """The metadata of every kernel in a library built here: its code objects are the ELF images for gfx950 in the offload bundles
    (magic, number of entries, then offset, size, length of the name and name of each), and hold a note with a msgpack map."""
    import struct

    import msgpack
    blob = open(path, "rb").read()
    magic, at, kernels = b"__CLANG_OFFLOAD_BUNDLE__", 0, []
    while (at := blob.find(magic, at)) >= 0:
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", blob, pos - 8)[0]):
            off, size, length = struct.unpack_from("<3Q", blob, pos)
            name = blob[pos + 24:pos + 24 + length]
            pos += 24 + length
            if not name.endswith(b"gfx950"):
                continue
            elf = blob[at + off:at + off + size]
            phoff, (phentsize, phnum) = struct.unpack_from("<Q", elf, 32)[0], struct.unpack_from("<2H", elf, 54)
            for i in range(phnum):
                kind, _, start, _, _, filesz = struct.unpack_from("<2I4Q", elf, phoff + i * phentsize)
                while kind == 4 and filesz > 0:              # PT_NOTE
                    n, d, note = struct.unpack_from("<3I", elf, start)
                    skip = 12 + (n + 3) // 4 * 4
                    if note == 32:                           # NT_AMDGPU_METADATA
                        kernels += msgpack.unpackb(elf[start + skip:start + skip + d])["amdhsa.kernels"]
                    start, filesz = start + skip + (d + 3) // 4 * 4, filesz - skip - (d + 3) // 4 * 4
        at = pos
    return kernels


def test_attention_kernels_keep_their_registers(lib):
    """No instantiation of the large-tile kernel has registers in memory: a load of one behind a block's loads is waited for with all of them,
    and its loop counts on some being still on their way."""
    kernels = [k for k in _kernel_metadata(sb.LIB_PATH) if "sparse_attn_v5_kernel" in k[".name"]]
    assert len(kernels) >= 30
    assert {k[".name"]: k[".private_segment_fixed_size"] for k in kernels if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]} == {}


@pytest.mark.parametrize("named", [True, False])
def test_current_stream_with_and_without_its_handle(monkeypatch, named):
    import types

    import torch
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=1000 + device))
    if named:
        monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 2000 + device, raising=False)
    else:
        monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert sb._stream() == (2003 if named else 1003)
