"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every function
the header declares, sizes workspaces, and rejects bad arguments before launching anything."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2411_05288_amd", "libvp.so")
HEADER = os.path.join(ROOT, "include", "vp.h")

VP_OK, VP_ERR_INVALID_ARG, VP_ERR_UNSUPPORTED, VP_ERR_WORKSPACE, VP_ERR_DEVICE = range(5)


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_2411_05288_amd.build import build
        build()
    import paper_2411_05288_amd as vp
    return vp.load_library()


def declared_functions():
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(vp_[a-z_]+)\s*\(", text)))


def test_exports_every_declared_symbol(lib):
    names = declared_functions()
    assert {"vp_output_fwd", "vp_combine_stats", "vp_output_bwd", "vp_embed_fwd", "vp_embed_bwd",
            "vp_workspace_bytes", "vp_version", "vp_status_string"} <= set(names)
    for n in names:
        assert getattr(lib, n) is not None


def test_version_and_status_strings(lib):
    assert lib.vp_version() >= 100
    assert lib.vp_status_string(VP_OK) == b"VP_OK"
    assert lib.vp_status_string(VP_ERR_WORKSPACE) == b"VP_ERR_WORKSPACE"
    assert lib.vp_status_string(77) == b"VP_ERR_UNKNOWN"


def test_workspace_sizes(lib):
    bad = ctypes.c_size_t(-1).value
    ws = lib.vp_workspace_bytes
    # bf16 fwd: (2 * ceil(Vs/256) + 1) * N floats
    assert ws(0, 4096, 4096, 16032, 1, 1) == (2 * 63 + 1) * 4096 * 4
    assert ws(0, 4096, 4096, 16032, 1, 0) == (2 * 63 + 1) * 4096 * 4
    # fp32 fwd: logits live in the workspace only when they are not kept
    # (plus scratch for K slices when the output has few tiles: 2 slices of [128, 4096] here)
    assert ws(0, 128, 256, 4096, 0, 1) == 2 * 128 * 4096 * 4
    assert ws(0, 128, 256, 4096, 0, 0) == 128 * 4096 * 4 + 2 * 128 * 4096 * 4
    assert ws(0, 4096, 4096, 4096, 0, 1) == 0                      # enough tiles: no slicing
    # bwd: D [N, Vs] in the storage type
    assert ws(2, 4096, 8192, 16000, 1, 0) == 4096 * 16000 * 2
    assert ws(2, 4096, 4096, 4000, 1, 1) == 4096 * 4032 * 2        # rows of D padded to 128-byte multiples
    assert ws(2, 128, 256, 4096, 0, 1) == 128 * 4096 * 4 + 32 * 128 * 256 * 4   # fp32: D, then 32 K slices of dH
    assert ws(1, 128, 256, 4096, 0, 0) == 0 and ws(3, 128, 256, 4096, 1, 0) == 0
    assert ws(4, 8192, 4096, 32000, 1, 0) == 8192 * 12 + 256   # sorted keys, run starts, run counter
    assert ws(4, 5000, 4096, 32000, 1, 0) == 8192 * 12 + 256   # padded to a power of two
    assert ws(0, 0, 256, 4096, 0, 0) == bad
    assert ws(0, 128, 256, 4096, 5, 0) == bad
    assert ws(0, 128, 256, 4096, 0, 2) == bad                       # VP_SKIP_DH belongs to the backward call only
    assert ws(2, 128, 256, 4096, 0, 2) == 128 * 4096 * 4 + 32 * 128 * 256 * 4
    # Algorithm 2 forward: partials + the padded bf16 softmax' operand; fp32: one [N, Vs] matrix
    assert ws(5, 4096, 4096, 4000, 1, 1) == (2 * 16 + 1) * 4096 * 4 + 4096 * 4032 * 2
    assert ws(5, 128, 256, 4096, 0, 0) == 128 * 4096 * 4 + 32 * 128 * 256 * 4 and ws(6, 128, 256, 4096, 0, 0) == 0
    assert ws(9, 128, 256, 4096, 0, 0) == bad
    assert ws(2, 1 << 20, 256, 1 << 20, 1, 0) == bad               # N*Vs beyond 2^31 elements
    assert ws(0, 8, 8, (1 << 20) + 8, 1, 0) == bad and ws(0, 8, 8, 1 << 20, 1, 0) != bad   # rows of at most 2^20 elements
    assert ws(2, 8, (1 << 20) + 8, 8, 1, 0) == bad


def test_group_workspace_covers_the_slices_of_fp32_products(lib):
    # outputs with few tiles are cut into K slices for a group as for a single shard: partial sums behind the D matrices
    def ws(which, N, h, rows, flags):
        return lib.vp_output_group_workspace_bytes(which, len(rows), N, h, (ctypes.c_int64 * len(rows))(*rows), 0, flags)
    one = 16 * 1000 * 4                                               # logits of a shard, a multiple of 256
    assert ws(0, 16, 2048, [1000, 1000], 0) == 2 * one + 8 * 2 * one  # 32 tiles of 64 x 64: 8 slices
    d, dw = 2048 * 128 * 4, 125 * 64 * 4                              # D with rows padded to 4; dW, 125 * 256 bytes
    assert ws(2, 2048, 64, [125] * 16, 1 | 2) == 16 * d + 8 * 16 * dw # (no dH) 32 tiles: 8 slices
    # enough tiles: no slices, and what a single shard needs for its own is more
    assert ws(2, 128, 256, [4096] * 2, 1 | 2) == lib.vp_workspace_bytes(2, 128, 256, 4096, 0, 1 | 2)


# (N, h, V, p, K slices of dH): the measured best among slices and tile heights, or within 1 % of it; where the vocabulary is long a
# choice that ignores the power limit cut K otherwise, up to 13 % slower
@pytest.mark.parametrize("N,h,V,p,slices", [(520, 4096, 128256, 8, 5), (800, 4096, 128256, 8, 4), (1300, 3072, 50000, 8, 3),
                                            (1800, 4096, 128256, 8, 2), (2300, 3072, 50000, 8, 2), (3100, 6144, 32000, 4, 4),
                                            (3100, 3072, 32000, 4, 3), (3100, 1024, 32000, 4, 4), (4096, 4096, 32000, 8, 1)])
def test_slices_of_dh(lib, N, h, V, p, slices):
    rows = [V // p] * p
    D = p * N * ((V // p + 63) // 64 * 64) * 2
    got = lib.vp_output_group_workspace_bytes(2, p, N, h, (ctypes.c_int64 * p)(*rows), 1, 1) - D
    assert got == (slices * N * h * 4 if slices > 1 else 0)


def test_group_workspace_is_bounded(lib):
    def ws(which, N, h, rows, dt, flags):
        return lib.vp_output_group_workspace_bytes(which, len(rows), N, h, (ctypes.c_int64 * len(rows))(*rows), dt, flags)
    gib = 1 << 30
    for dt, rows in ((1, 65536), (0, 32768)):                         # D of 2 GiB per shard: two shards at a time
        assert ws(2, 16384, 64, [rows] * 2, dt, 2) == 4 * gib == ws(2, 16384, 64, [rows] * 3, dt, 2)
    # 2 GiB of fp32 partial sums of dH: shard by shard, with what one shard needs
    assert ws(2, 16384, 2048, [64] * 16, 0, 0) == lib.vp_workspace_bytes(2, 16384, 2048, 64, 0, 0)
    assert ws(2, 16384, 1024, [64] * 16, 0, 0) >= gib
    bad = ctypes.c_size_t(-1).value
    assert ws(2, 64, 64, [64, 0], 1, 0) == bad and ws(1, 64, 64, [64], 1, 0) == bad and ws(2, 64, 64, [], 1, 0) == bad


def test_group_calls_validate_their_arguments(lib):
    P, arr, i64 = 0x1000, ctypes.c_void_p * 2, ctypes.c_int64 * 2
    ptrs, rows, offs = arr(P, P), i64(8, 8), i64(0, 8)
    fwd = lambda W=ptrs, r=rows, o=offs, p=2, flags=0, ws=P, wb=1 << 20: lib.vp_output_fwd_group(
        P, W, r, o, p, P, 8, 8, 1, flags, P, P, P, None, ws, wb, None)
    assert fwd(W=arr(P, None)) == VP_ERR_INVALID_ARG and fwd(W=arr(P, P + 2)) == VP_ERR_INVALID_ARG
    assert fwd(r=i64(8, 0)) == VP_ERR_INVALID_ARG and fwd(o=i64(0, -1)) == VP_ERR_INVALID_ARG and fwd(p=0) == VP_ERR_INVALID_ARG
    assert fwd(flags=1) == VP_ERR_INVALID_ARG and fwd(ws=None, wb=0) == VP_ERR_WORKSPACE and fwd(wb=16) == VP_ERR_WORKSPACE
    assert fwd(r=i64(8, (1 << 20) + 8)) == VP_ERR_UNSUPPORTED
    bwd = lambda dW=ptrs, dH=P, flags=0, wb=1 << 20: lib.vp_output_bwd_group(
        P, ptrs, rows, offs, 2, P, 8, 8, 1, flags, P, P, None, 1.0, dH, dW, P, wb, None)
    assert bwd(dW=arr(P, None)) == VP_ERR_INVALID_ARG and bwd(dW=arr(P + 4, P)) == VP_ERR_INVALID_ARG
    assert bwd(dH=None) == VP_ERR_INVALID_ARG and bwd(flags=6) == VP_ERR_INVALID_ARG and bwd(flags=1) == VP_ERR_INVALID_ARG
    assert bwd(dH=None, flags=2, wb=8) == VP_ERR_WORKSPACE and bwd(wb=8) == VP_ERR_WORKSPACE


def test_argument_validation_launches_nothing(lib):
    # every call below must be rejected on the host; fake non-null pointers are never touched
    P = 0x1000
    fwd, cmb, bwd, efw, ebw = (lib.vp_output_fwd, lib.vp_combine_stats, lib.vp_output_bwd,
                               lib.vp_embed_fwd, lib.vp_embed_bwd)
    assert fwd(None, P, P, 8, 8, 8, 0, 1, 0, P, P, P, None, P, 1 << 20, None) == VP_ERR_INVALID_ARG
    assert fwd(P, P, P, 0, 8, 8, 0, 1, 0, P, P, P, None, P, 1 << 20, None) == VP_ERR_INVALID_ARG
    assert fwd(P, P, P, 8, 8, 8, -1, 1, 0, P, P, P, None, P, 1 << 20, None) == VP_ERR_INVALID_ARG
    assert fwd(P, P, P, 8, 8, 8, 0, 3, 0, P, P, P, None, P, 1 << 20, None) == VP_ERR_INVALID_ARG
    assert fwd(P, P, P, 8, 8, 8, 0, 1, 1, P, P, P, None, P, 1 << 20, None) == VP_ERR_INVALID_ARG   # flag w/o buffer
    assert fwd(P, P, P, 8, 8, 8, 0, 1, 0, P, P, P, P, P, 1 << 20, None) == VP_ERR_INVALID_ARG      # buffer w/o flag
    assert fwd(P + 2, P, P, 8, 8, 8, 0, 1, 0, P, P, P, None, P, 1 << 20, None) == VP_ERR_INVALID_ARG  # misaligned
    assert fwd(P, P, P, 8, 8, 8, 0, 1, 0, P, P, P, None, P, 16, None) == VP_ERR_WORKSPACE
    assert fwd(P, P, P, 8, 8, 8, 0, 1, 0, P, P, P, None, None, 0, None) == VP_ERR_WORKSPACE
    assert fwd(P, P, P, 1 << 20, 8, 1 << 20, 0, 1, 0, P, P, P, None, P, 1 << 40, None) == VP_ERR_UNSUPPORTED
    assert cmb(P, P, P, 0, 8, P, P, None, P, None) == VP_ERR_INVALID_ARG
    assert cmb(P, P, P, 2, 8, P, P, None, None, None) == VP_ERR_INVALID_ARG
    assert bwd(P, P, P, 8, 8, 8, 0, 1, 0, P, P, None, 1.0, None, P, P, 1 << 20, None) == VP_ERR_INVALID_ARG
    assert bwd(P, P, P, 8, 8, 8, 0, 1, 0, P, P, None, 1.0, P, P, P, 8, None) == VP_ERR_WORKSPACE
    assert bwd(P, P, P, 8, 8, 8, 0, 1, 1, P, P, None, 1.0, P, P, P, 1 << 20, None) == VP_ERR_INVALID_ARG
    assert efw(P, None, 8, 8, 8, 0, 1, P, None) == VP_ERR_INVALID_ARG
    assert efw(P, P, 8, 8, 8, 0, 7, P, None) == VP_ERR_INVALID_ARG
    assert ebw(P, P, 8, 8, 8, 0, 1, P, None, 0, None) == VP_ERR_WORKSPACE
    assert ebw(P, P, 1 << 25, 8, 8, 0, 1, P, P, 1 << 40, None) == VP_ERR_UNSUPPORTED
    assert ebw(P, P, 8, 0, 8, 0, 1, P, P, 1 << 20, None) == VP_ERR_INVALID_ARG
    # Algorithm 2: pass S with A and B, the input-gradient term, pass T without dH
    fwd2, dx2 = lib.vp_output_fwd_alg2, lib.vp_output_dx_alg2
    assert fwd2(P, P, P, 8, 8, 8, 0, 1, 0, P, P, P, None, None, P, P, 1 << 20, None) == VP_ERR_INVALID_ARG   # no A
    assert fwd2(P, P, P, 8, 8, 8, 0, 1, 0, P, P, P, None, P, None, P, 1 << 20, None) == VP_ERR_INVALID_ARG   # no B
    assert fwd2(P, P, P, 8, 8, 8, 0, 1, 2, P, P, P, None, P, P, P, 1 << 20, None) == VP_ERR_INVALID_ARG      # bad flag
    assert fwd2(P, P, P, 8, 8, 8, 0, 1, 0, P, P, P, None, P, P, P, 64, None) == VP_ERR_WORKSPACE
    assert dx2(P, P, P, P, P, P, 8, 8, 1, 0, 1.0, None, None) == VP_ERR_INVALID_ARG
    assert dx2(P, P, P, P, P, P, 0, 8, 1, 0, 1.0, P, None) == VP_ERR_INVALID_ARG
    assert dx2(P, P + 4, P, P, P, P, 8, 8, 1, 0, 1.0, P, None) == VP_ERR_INVALID_ARG
    assert dx2(P, P, P, P, P, P, 8, 8, 1, 2, 1.0, P, None) == VP_ERR_INVALID_ARG                            # only VP_DH_OVERWRITE
    assert bwd(P, P, P, 8, 8, 8, 0, 1, 2, P, P, None, 1.0, None, P, P, 8, None) == VP_ERR_WORKSPACE          # VP_SKIP_DH: dH may be NULL
    assert bwd(P, P, P, 8, 8, 8, 0, 1, 8, P, P, None, 1.0, P, P, P, 1 << 20, None) == VP_ERR_INVALID_ARG
    assert bwd(P, P, P, 8, 8, 8, 0, 1, 6, P, P, None, 1.0, P, P, P, 1 << 20, None) == VP_ERR_INVALID_ARG      # skip + overwrite
    assert bwd(P, P, P, 8, 8, 8, 0, 1, 4, P, P, None, 1.0, P, P, P, 8, None) == VP_ERR_WORKSPACE               # VP_DH_OVERWRITE is valid


def test_binding_refuses_cpu_tensors(lib):
    import torch
    import paper_2411_05288_amd as vp
    H = torch.zeros(8, 8)
    with pytest.raises(vp.VPError):
        vp.vp_embed_fwd(H, torch.zeros(8, dtype=torch.int64), 0, torch.zeros(8, 8))


def test_bench_refuses_more_than_one_gpu():
    # the path runs on one GPU; asking for more must end with a message, before anything touches a GPU
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=120)
    assert r.returncode != 0
    assert "one GPU" in r.stderr


def test_missing_library_is_an_error_not_a_fallback(monkeypatch):
    # the product path has no CPU fallback: without libvp.so every entry point raises
    import paper_2411_05288_amd.binding as B
    monkeypatch.setattr(B, "_LIB", None)
    monkeypatch.setattr(B, "lib_path", lambda: "/nonexistent/libvp.so")
    with pytest.raises(B.VPError):
        B.load_library()
    with pytest.raises(B.VPError):
        B.vp_version()
    with pytest.raises(B.VPError):
        B.vp_workspace_bytes(B.VP_CALL_OUTPUT_FWD, 8, 8, 8, B.VP_BF16, 0)
