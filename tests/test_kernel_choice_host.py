"""Which kernels the forward calls choose, read off without a GPU: on a dry run a call checks its arguments, takes its
decisions and launches nothing.  The pointers are made up and never followed."""
import ctypes as C
import os
import threading

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2407_02031_amd", "libswiftdiff.so")
BF16, F32 = 0, 1


@pytest.fixture(scope="module")
def B():
    if not os.path.exists(LIB):
        from paper_2407_02031_amd import build
        build.build(verbose=False)
    from paper_2407_02031_amd import binding
    return binding


def linear(B, M, K, N, r=0, ln=False, geglu=False, res=False, f32=False):
    """The kernels of one projection."""
    L = B.lib()
    p = B.sd_proj(0x10000, 0x20000, 0x30000 if r else None, 0x40000 if r else None, r, 1.0)
    need = L.sd_lora_linear_workspace_bytes(M, N, K, r, int(ln))
    g = 0x50000 if ln else None
    with B.dry_run() as names:
        rc = L.sd_lora_linear_fwd(0x60000, BF16, C.byref(p), g, g, 1e-5, 0x70000 if res else None, 0x80000, F32 if f32 else BF16, int(geglu), M, N, K, 0x100000, need, None)
    assert rc == 0, L.sd_last_error()
    return names


def test_dry_run_launches_nothing_and_belongs_to_its_thread(B):
    L = B.lib()
    assert linear(B, 300, 328, 200) == ["gemm 64x128/4 waves/3 stages guard"]
    assert linear(B, 300, 328, 200, r=200) == ["clear", "gemm 64x128/4 waves/3 stages guard flags"]
    assert linear(B, 300, 328, 200, r=128) == ["gemm 64x128/4 waves/3 stages guard records"]
    assert linear(B, 300, 328, 200, r=8, ln=True)[0] == "layernorm clear"
    assert linear(B, 0, 328, 200) == []
    seen = []
    with B.dry_run() as mine:
        t = threading.Thread(target=lambda: seen.append((L.sd_dry_run(0), L.sd_dry_run_text())))
        t.start()
        t.join()
        assert L.sd_lora_patch(0x1000, 1, 10, None) == 0
    assert seen == [(0, b"")] and mine == ["patch 1 tile/3 stages"]
    with B.dry_run() as names:
        assert L.sd_attention_fwd(0x1000, 0x2000, 0x3000, 0x4000, 2, 64, 1300, 128, 2, None, 0, None) == 0
        assert L.sd_attention_fwd(0x1000, 0x2000, 0x3000, 0x4000, 2, 64, 1216, 128, 2, None, 0, None) == 0
        assert L.sd_attention_fwd(0x1000, 0x2000, 0x3000, 0x4008, 2, 64, 1216, 128, 2, None, 0, None) == -1
    assert names == ["attention try", "attention"]


@pytest.mark.parametrize("tiles,single,multi", [(1, "1 tile/3 stages", "1 tile/3 stages"), (512, "1 tile/3 stages", "1 tile/3 stages"), (513, "1 tile/2 stages", "1 tile/2 stages"),
                                                (768, "1 tile/2 stages", "1 tile/2 stages"), (769, "2 tiles/3 stages", "2 tiles/2 stages"), (100000, "2 tiles/3 stages", "2 tiles/2 stages")])
def test_patch_cuts(B, tiles, single, multi):
    L = B.lib()
    with B.dry_run() as names:
        L.sd_lora_patch(0x1000, 1, tiles, None)
        L.sd_lora_patch_multi(0x1000, 1, tiles, None)
        L.sd_lora_unpatch(0x1000, 1, tiles, None)
    assert names == ["patch " + single, "patch multi " + multi, "unpatch"]


# one round of 64-row tiles (three ring stages, two), of 128-row tiles; beyond that by estimate, against what was measured:
# the general kernel's 256x128 ahead of the wide tiles where the K loop is long and the rounds come out even for it, the wide
# ones at the feed-forward widths of 640 and 1280 channels
@pytest.mark.parametrize("M,K,F,r,kernel", [
    (256, 1280, 2560, 16, "gemm 64x128/4 waves/3 stages geglu"), (2048, 320, 1280, 0, "gemm 64x128/4 waves/2 stages geglu"),
    (3952, 320, 640, 64, "gemm 64x128/4 waves/2 stages geglu"), (988, 640, 2560, 8, "gemm 64x128/4 waves/2 stages geglu"),
    (1500, 640, 2560, 8, "gemm 128x128/4 waves/2 stages geglu"), (512, 2048, 8192, 8, "gemm 128x128/4 waves/2 stages geglu"),
    (1500, 1280, 5120, 128, "gemm 256x256/8 waves/2 stages geglu"), (7904, 2048, 4096, 64, "gemm 256x256/8 waves/2 stages geglu"),
    (8192, 2048, 4096, 0, "gemm 256x256/8 waves/2 stages geglu"), (988, 1280, 5120, 16, "geglu 128x160"),
    (2048, 1280, 5120, 64, "geglu 256x160"), (8192, 640, 2560, 64, "geglu 256x160"), (7904, 640, 2560, 0, "geglu 256x160"),
    (1000, 640, 5120, 72, "geglu 128x160"), (8192, 640, 2564, 0, "gemm 256x256/8 waves/2 stages geglu"), (8192, 648, 2560, 0, "gemm 128x128/4 waves/2 stages geglu"),
])
def test_feed_forward_in_projection(B, M, K, F, r, kernel):
    names = linear(B, M, K, F, r, ln=True, geglu=True)
    assert names[0].startswith("layernorm")
    if kernel.startswith("gemm"):
        kernel += (" guard" if K % 64 or r % 64 else "") + (" flags" if r else "")
    assert names[1:] == (["down"] if r and kernel.startswith("geglu") else []) + [kernel]


# an adapter in the tile up to rank 32, to rank 64 while K is short or N = 320; a lone projection not where the general kernel
# fits it into one round, its producers counted and dealt over the 8 XCDs
@pytest.mark.parametrize("M,K,N,r,kernel", [
    (512, 320, 320, 8, "gemm16 64x80/1"), (512, 320, 320, 64, "gemm16 64x80/4"), (154, 2048, 1280, 16, "gemm16 64x80/1"), (154, 2048, 1280, 64, "gemm 64x128/4 waves/3 stages records"),
    (8192, 640, 640, 64, "gemm16 128x160/2"), (8192, 640, 640, 72, "gemm 64x128/4 waves/2 stages guard records"), (2048, 1280, 1280, 32, "gemm16 64x160/1"), (2048, 1280, 1280, 40, "gemm 128x128/8 waves/4 stages guard records"),
    (4100, 640, 640, 0, "gemm 128x128/8 waves/4 stages"), (6500, 640, 640, 0, "gemm 128x128/8 waves/4 stages"), (6600, 640, 640, 0, "gemm16 128x160/0"), (5100, 640, 640, 16, "gemm 128x128/8 waves/4 stages guard records"),
    (5350, 640, 640, 16, "gemm16 128x160/1"), (5350, 1280, 640, 72, "gemm 256x128/8 waves/3 stages guard records"), (6144, 640, 640, 16, "gemm16 128x160/1"), (4100, 320, 320, 32, "gemm16 64x160/1"), (4100, 320, 320, 0, "gemm 64x128/4 waves/3 stages"),
    (6000, 320, 320, 0, "gemm16 64x160/0"), (2300, 640, 640, 16, "gemm16 64x160/1"), (2300, 640, 640, 64, "gemm 64x128/4 waves/3 stages records"), (2300, 1280, 640, 16, "gemm 64x128/4 waves/3 stages guard records"),
    (8192, 320, 320, 64, "gemm16 64x160/2"), (8300, 1280, 320, 64, "gemm16 128x160/2"),
])
@pytest.mark.parametrize("ln", [False, True])
def test_projection_in_tile_or_not(B, M, K, N, r, kernel, ln):
    names = linear(B, M, K, N, r, ln=ln)
    assert names[-1] == (kernel.replace("records", "flags") if ln else kernel)


# GroupNorm's second pass asks for statistics and affine ahead of its rows where a workgroup has six slabs of 16-byte pieces; without SiLU only while
# workgroups do not follow each other on a CU for long, of five samples and more not in a round that has hardly more than a workgroup a CU
@pytest.mark.parametrize("Bn,T,Cc,groups,plain,silu", [
    (2, 16384, 320, 32, True, True), (1, 43000, 320, 32, True, True), (9, 1200, 1280, 32, False, True), (4, 16384, 320, 32, False, True), (16, 1024, 1280, 32, False, True),
    (1, 12000, 100, 10, False, False), (8, 3000, 1220, 10, False, False), (2, 4096, 320, 32, False, False),
    (20, 900, 320, 32, False, False), (16, 1600, 320, 32, False, True), (90, 300, 320, 32, True, True), (4, 4610, 320, 32, True, True), (6, 1000, 960, 32, False, False),
])
def test_groupnorm_second_pass(B, Bn, T, Cc, groups, plain, silu):
    L = B.lib()
    with B.dry_run(detail=True) as names:
        for call in (L.sd_groupnorm_fwd, L.sd_groupnorm_silu_fwd):
            assert call(0x10000, 0x20000, 0x30000, 0x40000, Bn, T, Cc, groups, 1e-6, 0x100000, L.sd_groupnorm_workspace_bytes(Bn, T, Cc, groups), None) == 0
    assert names == ["groupnorm" + (", statistics first" if first else "") for first in (plain, silu)]


# Cut attention tiles have 128 queries, and their halves fit the scratch memory that the call asks for: over token and key counts, heads and samples, on its
# own and inside a block
def test_cut_attention_tiles(B):
    L = B.lib()
    p = B.sd_proj(0x10000, None, None, None, 0, 0.0)
    seen = set()
    for Tq in (64, 200, 800, 1000, 1290, 1500, 1800, 2048, 3000, 3952, 4096):
        for Tk in (77, 500, 800, 1300, 1500, 2000, 3952, 4096):
            for Bn, heads in ((1, 5), (1, 10), (2, 5), (1, 20), (2, 10), (2, 20), (4, 20), (8, 20)):
                tiles = (Tq + 127) // 128 * heads * Bn
                with B.dry_run(detail=3) as names:
                    need = L.sd_attention_workspace_bytes(Bn, Tq, Tk, heads)
                    assert L.sd_attention_fwd(0x1000, 0x2000, 0x3000, 0x4000, Bn, Tq, Tk, 64 * heads, heads, 0x100000, need, None) == 0
                    rc = L.sd_attn_block_fwd(0x1000, 0x2000, BF16, 0x3000, Tk, 128, 0x4000, 0x5000, 1e-5, C.byref(p), C.byref(p), C.byref(p), C.byref(p), Bn, Tq, 64 * heads, heads,
                                             0x100000, L.sd_attn_block_workspace_bytes(Bn, Tq, 64 * heads, Tk, 128, 0), None)
                    assert rc == 0, L.sd_last_error()
                launches = [n for n in names if n.startswith("attention")]
                assert len(launches) == 2
                for n in launches:
                    seen.add(n)
                    assert " cut" not in n or n.endswith((", 128 queries, 1 groups", ", 128 queries, 2 groups")), (n, Bn, Tq, Tk, heads)
                if " cut" in launches[0]:        # a half: 128 x 64 values, 128 maxima, 128 sums
                    assert need >= (768 - tiles) * 2 * 128 * 66 * 4
    assert {n.split(",", 1)[1] for n in seen} == {" 128 queries, 1 groups", " 128 queries, 2 groups", " 256 queries, 1 groups", " 256 queries, 2 groups"}
    assert {n.split(",")[0] for n in seen} >= {"attention try cut merge", "attention prescaled try cut", "attention prescaled try", "attention try", "attention"}
