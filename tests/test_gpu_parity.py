"""GPU parity: every C-ABI call against the CPU oracle on the same seeded inputs, element
by element, at sizes that span several tiles and ragged tails.  Tolerances are the ones the
task states: max|d|/max|ref| <= 1e-2 for bf16 paths, <= 1e-5 for fp32 patching, unpatch
bit-exact.  Each call's output is normalised by its own maximum (for residual sub-layers:
the update, not the residual stream), and negative controls show the check can fail."""
import time

import numpy as np
import pytest

from conftest import rel_err
from oracle import sdxl_block_oracle as O
from workloads import sdxl_inputs as G

pytestmark = pytest.mark.gpu

BF16_TOL = 1e-2
PATCH_TOL = 1e-5


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2407_02031_amd import binding
    return binding


def dev(a, B):
    return B.to_bf16(a)


def host(t):
    import torch
    return t.detach().to(torch.float32).cpu().numpy()


def rng(seed):
    return np.random.default_rng(seed)


def mkproj(r, N, K, rank, bias=True, scale=1.0, w_std=0.05):
    return G.make_projection(r, N, K, bias=bias, r=rank, scale=scale, w_std=w_std, a_std=0.3 if rank else 0.0, b_std=0.05)


# ------------------------------------------------------------------- lora_linear_fwd
@pytest.mark.parametrize("M,K,N,rank,scale", [
    (300, 328, 200, 8, 0.5),      # ragged in every dimension, K not a multiple of 64
    (512, 320, 320, 8, 1.0),      # the tiny config's projection
    (1000, 640, 1920, 64, 1.0),   # several 256-row tiles
    (77, 2048, 320, 16, 2.0),     # text-context projection shape
    (130, 64, 136, 0, 0.0),       # no adapter
    (1, 8, 8, 8, 1.0),            # smallest legal shape
])
def test_lora_linear_matches_oracle(B, M, K, N, rank, scale):
    r = rng(M + K + N)
    p = mkproj(r, N, K, rank, bias=True, scale=scale)
    x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
    ref = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
    y = B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p))
    assert y.shape == (M, N)
    assert rel_err(host(y), ref) <= BF16_TOL
    if rank:
        # negative control: the adapter term is well above the tolerance, so dropping it
        # (or its scale) would be seen
        base = O.linear(x, p["W"], p["b"])
        assert rel_err(base, ref) > 3 * BF16_TOL
        # merged-weight path: plain linear on W' agrees with the unmerged call
        Wm = G.bf16_round(O.merged_weight(p["W"], p["A"], p["B"], p["scale"]).astype(np.float32))
        pm = dict(p, W=Wm, A=None, B=None)
        ym = B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(pm))
        assert rel_err(host(ym), ref) <= 2 * BF16_TOL     # W' itself is rounded to bf16 here


def test_lora_linear_same_workspace_new_inputs(B):
    """The base GEMM's tiles read the down-projection that other tiles of the same launch
    wrote moments before, possibly on another XCD with its own L2.  Reusing one workspace with
    changing inputs and adapters would serve a stale down-projection (the previous call's, still
    cached) if those reads and writes were not of device scope; a tile that did not wait at all
    would read the previous call's too.  Large enough that every XCD runs tiles of both kinds."""
    import torch
    M, K, N, rank = 4096 + 37, 640, 640, 64
    r = rng(99)
    need = B.lib().sd_lora_linear_workspace_bytes(M, N, K, rank, 0)
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    for trial in range(4):
        p = mkproj(r, N, K, rank, bias=True, scale=1.0 + trial)
        x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
        ref = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
        base = O.linear(x, p["W"], p["b"])
        assert rel_err(base, ref) > 10 * BF16_TOL          # the adapter term carries most of the output
        xd, pd = dev(x, B), B.Proj.from_numpy(p)
        for rep in range(3):
            y = B.lora_linear_fwd(xd, pd, ws=ws)
            assert rel_err(host(y), ref) <= BF16_TOL, (trial, rep)
    assert B.gemm_dep_timeouts() == 0


# base tiles that read what other tiles of the same launch wrote, announced by flags and by records: one workspace, changing inputs and
# adapters, large enough that every XCD runs tiles of both kinds; and the same bits as with the two GEMMs as two launches
@pytest.mark.parametrize("M,K,N,rank,ln,kernel", [(4133, 640, 640, 72, True, "flags"), (4133, 640, 640, 72, False, "records"), (8192, 1280, 1280, 64, True, "flags"), (8192, 640, 1280, 128, False, "records"),
                                                  (4133, 640, 640, 136, False, "flags")])
def test_lora_linear_waits_inside_the_launch(B, M, K, N, rank, ln, kernel):
    import torch
    r = rng(M + K + N + rank)
    ws = torch.zeros(B.lib().sd_lora_linear_workspace_bytes(M, N, K, rank, int(ln)), dtype=torch.uint8, device="cuda")
    ones, zeros = dev(np.ones(K, np.float32), B), dev(np.zeros(K, np.float32), B)
    kw = dict(ln_gamma=ones, ln_beta=zeros) if ln else {}
    for trial in range(3):
        p = mkproj(r, N, K, rank, bias=True, scale=1.0 + trial)
        x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
        rows = np.arange(trial, M, 7)
        xr = O.layernorm(x[rows], np.ones(K, np.float32), np.zeros(K, np.float32)) if ln else x[rows]
        ref = O.lora_linear(xr, p["W"], p["b"], p["A"], p["B"], p["scale"])
        assert rel_err(O.linear(xr, p["W"], p["b"]), ref) > 10 * BF16_TOL       # the adapter term carries most of the output
        xd, pd = dev(x, B), B.Proj.from_numpy(p)
        with B.dry_run() as names:
            B.lora_linear_fwd(xd, pd, ws=ws, **kw)
        assert names[-1].startswith("gemm ") and names[-1].endswith(kernel)
        ys = [B.lora_linear_fwd(xd, pd, ws=ws, **kw) for _ in range(3)]
        assert rel_err(host(ys[0])[rows], ref) <= BF16_TOL, trial
        try:
            B.set_projection_fusion(False)
            with B.dry_run() as names:
                B.lora_linear_fwd(xd, pd, ws=ws, **kw)
            assert sum(n.startswith("gemm ") for n in names) == 2 and not names[-1].endswith(kernel)
            ys.append(B.lora_linear_fwd(xd, pd, ws=ws, **kw))
        finally:
            B.set_projection_fusion(True)
        assert all(torch.equal(ys[0], y) for y in ys[1:]), trial
    assert B.gemm_dep_timeouts() == 0


def test_stack_as_one_launch_or_two_gives_the_same_bits_where_tiles_wait(B):
    """A stack whose projections wait inside their launches (rank 72: no tile forms t by itself; the in-projection's tiles are the
    general kernel's), its cut attention merged inside the launch and by a kernel of its own."""
    import torch
    cfg = small_cfg(Bn=2, T=2560, C=1024, heads=16, depth=1, r=72, alpha=8.0)
    p = G.make_stack_inputs(cfg, seed=9)
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    outs, names = {}, {}
    try:
        for on in (True, False):
            B.set_projection_fusion(on)
            with B.dry_run() as names[on]:
                B.spatial_transformer_fwd(x, ctx, sp, cfg.heads)
            outs[on] = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads).clone()
    finally:
        B.set_projection_fusion(True)
    waits = lambda ns: sum(n.endswith(("flags", "records")) for n in ns)
    assert waits(names[True]) >= 4 and waits(names[False]) == 0
    assert "attention prescaled try cut" in names[True] and "attention prescaled try cut merge" in names[False]
    assert torch.equal(outs[True], outs[False])
    assert B.gemm_dep_timeouts() == 0


def test_lora_linear_random_shapes(B):
    """Seeded sweep over ragged shapes and ranks (rank > 64: two column tiles of down-projection
    per row block, so a base tile waits for a count of 2; rank not a multiple of 64; one-row and
    one-tile problems; more row blocks than CUs) through the single-launch projection."""
    r = rng(2024)
    shapes = [(1, 64, 8, 8), (63, 72, 40, 128), (64, 64, 64, 64), (65, 136, 264, 72), (129, 200, 136, 128),
              (700, 640, 640, 96), (2100, 320, 136, 24), (20000, 64, 136, 8), (333, 1288, 72, 200)]
    for _ in range(6):
        shapes.append((int(r.integers(1, 900)), 8 * int(r.integers(1, 60)), 8 * int(r.integers(1, 60)), 8 * int(r.integers(1, 20))))
    for (M, K, N, rank) in shapes:
        p = mkproj(r, N, K, rank, bias=True, scale=0.7)
        x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
        ref = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
        y = B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p))
        assert rel_err(host(y), ref) <= BF16_TOL, (M, K, N, rank)
    assert B.gemm_dep_timeouts() == 0


def test_lora_linear_layernorm_residual_fp32(B):
    import torch
    r = rng(7)
    M, K, N = 260, 320, 320
    p = mkproj(r, N, K, 16, bias=True, scale=0.5)
    x = (r.standard_normal((M, K)) * 2 + 0.5).astype(np.float32)
    g, b = G.bf16_round((1 + 0.1 * r.standard_normal(K)).astype(np.float32)), G.bf16_round((0.1 * r.standard_normal(K)).astype(np.float32))
    res = r.standard_normal((M, N)).astype(np.float32)
    upd = O.lora_linear(O.layernorm(x, g, b), p["W"], p["b"], p["A"], p["B"], p["scale"])
    xd, resd = torch.from_numpy(x).cuda(), torch.from_numpy(res).cuda()
    y = B.lora_linear_fwd(xd, B.Proj.from_numpy(p), ln_gamma=dev(g, B), ln_beta=dev(b, B), residual=resd, out_dtype=torch.float32)
    assert y.dtype == torch.float32
    assert rel_err(host(y) - res, upd) <= BF16_TOL
    # in place on the residual buffer
    B.lora_linear_fwd(xd, B.Proj.from_numpy(p), ln_gamma=dev(g, B), ln_beta=dev(b, B), residual=resd, out=resd)
    assert np.array_equal(host(resd), host(y))


@pytest.mark.parametrize("M,C,F,rank", [(200, 64, 96, 8), (512, 320, 1280, 0), (384, 640, 2560, 64),
                                        # narrow outputs (F <= 64: no wider than one down-projection tile)
                                        (150, 64, 32, 0), (150, 64, 32, 8), (300, 128, 64, 0), (300, 128, 64, 16), (70, 72, 8, 8)])
def test_lora_linear_geglu_epilogue(B, M, C, F, rank):
    r = rng(M + F)
    p = mkproj(r, 2 * F, C, rank, bias=True, scale=1.0, w_std=0.08)
    x = G.bf16_round(r.standard_normal((M, C)).astype(np.float32))
    ref = O.geglu(O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"]))
    y = B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p), epilogue=B.SD_EPI_GEGLU)
    assert y.shape == (M, F)
    assert rel_err(host(y), ref) <= BF16_TOL
    # negative control: value/gate halves swapped is a different function
    u = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
    assert rel_err(O.geglu(np.concatenate([u[:, F:], u[:, :F]], 1)), ref) > 10 * BF16_TOL


@pytest.mark.parametrize("M,C,F,rank", [(8192 + 77, 328, 2560 + 8, 16), (8192, 328, 2560 - 8, 16), (8192 - 100, 64, 2560, 0)])
def test_lora_linear_geglu_large_ragged(B, M, C, F, rank):
    """Enough tiles for the 256-row GEGLU tile body (two rounds of the chip or more), with ragged
    last row and column tiles and a K that is not a multiple of 64; with and without an adapter
    (without one the launch has no down-projection tiles ahead of the 256x256 ones)."""
    r = rng(M + F)
    p = mkproj(r, 2 * F, C, rank, bias=True, scale=0.5, w_std=0.08)
    x = G.bf16_round(r.standard_normal((M, C)).astype(np.float32))
    ref = O.geglu(O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"]))
    y = B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p), epilogue=B.SD_EPI_GEGLU)
    got = host(y)
    assert got.shape == (M, F)
    assert rel_err(got, ref) <= BF16_TOL
    # corners and an interior band, each on its own scale
    for rows, cols in ((slice(0, 256), slice(0, 128)), (slice(M - 77, M), slice(F - 8, F)), (slice(M - 77, M), slice(0, 128)),
                       (slice(0, M), slice(2048 - 64, 2048 + 64)), (slice(M - 130, M), slice(2048, F))):
        assert rel_err(got[rows, cols], ref[rows, cols]) <= BF16_TOL
    assert B.gemm_dep_timeouts() == 0


@pytest.mark.parametrize("M,N,K,rank", [(8192 + 77, 2048 + 8, 2048 + 8, 16), (8192, 2048, 2048, 0)])
def test_lora_linear_large_plain_projection(B, M, N, K, rank):
    """One plain projection large enough for the 256x256 tile body (two rounds of the chip or more,
    K >= 2048): ragged last row and column tiles and a ragged K with an adapter, exact tiles without."""
    r = rng(M + N + K)
    p = mkproj(r, N, K, rank, bias=True, scale=0.5, w_std=0.03)
    x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
    ref = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
    got = host(B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p)))
    assert got.shape == (M, N)
    assert rel_err(got, ref) <= BF16_TOL
    for rows, cols in ((slice(0, 256), slice(0, 256)), (slice(M - 77, M), slice(N - 8, N)), (slice(M - 77, M), slice(0, 256)),
                       (slice(0, M), slice(1024 - 64, 1024 + 64)), (slice(4096 - 3, 4096 + 3), slice(0, N))):
        assert rel_err(got[rows, cols], ref[rows, cols]) <= BF16_TOL
    assert B.gemm_dep_timeouts() == 0


# one round of 128x160, 64x160 or 64x80 tiles: K of one, two, three and many 64 deep steps (both parities, rings that never fill), ragged
# rows and columns, ranks with 1, 2 or 4 column blocks of A and none, an fp32 or bf16 residual, bias or none
@pytest.mark.parametrize("M,K,N,rank,f32", [(1, 64, 8, 8, False), (63, 128, 84, 24, True), (130, 192, 80, 64, False), (333, 320, 324, 0, True), (512, 320, 320, 8, True),
                                            (988, 1280, 1280, 16, False), (1000, 640, 1284, 0, False), (1990, 704, 1280, 64, False), (2048, 256, 1280, 0, True),
                                            (5000, 128, 640, 0, False), (8192, 640, 640, 40, True), (8190, 64, 640, 0, True), (154, 2048, 1280, 0, False)])
def test_lora_linear_one_round_of_tiles(B, M, K, N, rank, f32):
    import torch
    r = rng(M + K + N)
    p = mkproj(r, N, K, rank, bias=M % 2 == 0, scale=0.7)
    x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
    res = G.bf16_round(r.standard_normal((M, N)).astype(np.float32))
    upd = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
    resd = torch.from_numpy(res).cuda() if f32 else dev(res, B)
    y = B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p), residual=resd, out_dtype=torch.float32 if f32 else torch.bfloat16)
    # a bf16 y rounds the sum: its unit in the last place is relative to the sum, not to the update
    assert rel_err(host(y), upd + res) <= BF16_TOL
    if f32:
        assert rel_err(host(y) - res, upd) <= BF16_TOL


# one round of in-tile tiles (128x160, 64x160, 64x80) with a residual in the output's type, which is requested while the first
# stages are in flight: fewer steps than stages, as many, one more, many; ragged rows and columns, no rows of a second block
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("M,K,N,rank", [(16380, 64, 320, 0), (5000, 192, 644, 40), (8192, 256, 640, 64), (8190, 320, 636, 0), (4757, 128, 324, 24), (5900, 384, 320, 0),
                                        (1, 64, 4, 8), (65, 128, 84, 0), (777, 192, 1284, 64), (130, 256, 76, 16), (63, 1280, 164, 32)])
def test_lora_linear_one_round_of_tiles_residual(B, M, K, N, rank, f32):
    import torch
    r = rng(M + K + N + rank)
    p = mkproj(r, N, K, rank, bias=M % 2 == 0, scale=0.7)
    x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
    res = G.bf16_round(r.standard_normal((M, N)).astype(np.float32))
    rd = torch.from_numpy(res).cuda()
    call = lambda: B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p), residual=rd if f32 else rd.bfloat16(), out_dtype=torch.float32 if f32 else torch.bfloat16)
    with B.dry_run() as names:
        call()
    assert names[-1].startswith("gemm16 ")
    got = host(call())
    ref = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
    # a bf16 sum of up to |update| + |residual| is rounded once more: half a unit in the last of 8 bits of it
    allow = 0 if f32 else 2.0 ** -9 * (np.abs(ref).max() + np.abs(res).max())
    assert np.abs(got - res - ref).max() <= BF16_TOL * np.abs(ref).max() + allow
    assert np.abs(got - ref).max() > 0.3 * np.abs(res).max()         # negative control: the residual is seen


# every number of steps about the ring's depth (three and four stages of 64x80, five of 64x160, four of 128x160): loops of no step, one pair
# and more for the steps that wait for the first stages, for those behind them and for the last ones, odd and even
@pytest.mark.parametrize("M,N,rank,kernel", [(70, 84, 8, "gemm16 64x80/1"), (63, 76, 0, "gemm16 64x80/0"), (8250, 160, 8, "gemm16 64x160/1"), (16400, 160, 0, "gemm16 128x160/0")])
def test_lora_linear_in_tile_every_number_of_steps(B, M, N, rank, kernel):
    import torch
    r = rng(M + N)
    for steps in range(1, 15):
        K = 64 * steps
        p = mkproj(r, N, K, rank, bias=steps % 2 == 0, scale=0.7)
        x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
        res = r.standard_normal((M, N)).astype(np.float32)
        call = lambda: B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p), residual=torch.from_numpy(res).cuda(), out_dtype=torch.float32)
        with B.dry_run(detail=True) as names:
            call()
        stages = {"gemm16 64x80": 3 if K <= 640 else 4, "gemm16 64x160": 5, "gemm16 128x160": 4}[kernel.split("/")[0]]
        assert names[-1] == "%s, 1 problems, %d stages, fp32 residual" % (kernel, stages), K
        ref = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
        assert np.abs(host(call()) - res - ref).max() <= BF16_TOL * np.abs(ref).max(), K


# feed-forward in-projections about the sizes where the wide tiles begin and end to pay: K loops of one, two, three and more steps, ranks of
# less and more than 64 (which kernel each of them takes: test_lora_linear_geglu_every_kernel)
@pytest.mark.parametrize("M,C,F,rank", [(6300, 64, 1288, 0), (8192, 128, 2560, 8), (4000, 192, 2568, 0), (1000, 640, 5120, 72), (988, 1280, 5120, 0), (2047, 1280, 5120, 64)])
def test_lora_linear_geglu_wide_tiles(B, M, C, F, rank):
    r = rng(M + F + rank)
    p = mkproj(r, 2 * F, C, rank, bias=rank != 8, scale=0.6, w_std=0.05)
    x = G.bf16_round(r.standard_normal((M, C)).astype(np.float32))
    y = B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p), epilogue=B.SD_EPI_GEGLU)
    assert y.shape == (M, F)
    rows = np.unique(np.concatenate([np.arange(0, M, 97), np.arange(max(0, M - 40), M), np.arange(96, 160), np.arange(250, 262)]))
    ref = O.geglu(O.lora_linear(x[rows], p["W"], p["b"], p["A"], p["B"], p["scale"]))
    assert rel_err(host(y)[rows], ref) <= BF16_TOL


# the down-projection in front of the wide tiles, about the ends of its three tilings, by what depends on it alone (no base weights): ranks off
# 16, K of fewer 64 deep blocks than wavefronts, of more than they have in flight, odd numbers.  t, B's products and y are rounded to bf16
@pytest.mark.parametrize("M,K,F,rank,tile", [
    (1024, 1280, 5120, 64, "16 rows by 16"), (1540, 1280, 5120, 64, "32 rows by 16"), (2048, 1280, 5120, 64, "32 rows by 16"), (3206, 640, 2560, 64, "32 rows by 64"),
    (990, 1280, 5120, 8, "16 rows by 16"), (1000, 640, 5120, 72, "32 rows by 16"), (4096, 640, 2560, 16, "16 rows by 16"), (6531, 448, 2560, 16, "32 rows by 16"),
    (6200, 192, 1288, 16, "32 rows by 16"), (8192, 640, 2560, 16, "32 rows by 16"), (16384, 640, 2560, 16, "32 rows by 16"), (1000, 2112, 5120, 24, "16 rows by 16"), (2040, 1664, 5120, 40, "32 rows by 16"),
])
def test_down_projection_tiles(B, M, K, F, rank, tile):
    r = rng(M + K + rank)
    p = mkproj(r, 2 * F, K, rank, bias=False, scale=1.0)
    p["W"] = np.zeros_like(p["W"])
    p["A"] = G.bf16_round(r.standard_normal((rank, K)).astype(np.float32) / np.sqrt(K).astype(np.float32))
    p["B"] = G.bf16_round(r.standard_normal((2 * F, rank)).astype(np.float32) / np.sqrt(rank).astype(np.float32))
    x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
    call = lambda: B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p), epilogue=B.SD_EPI_GEGLU)
    with B.dry_run(detail=True) as names:
        call()
    assert [n for n in names if n.startswith("down")] == ["down, " + tile]
    ref = O.geglu(O.lora_linear(x, p["W"], None, p["A"], p["B"], p["scale"]))
    assert rel_err(host(call()), ref) <= BF16_TOL


# each body of the plain projection, asserted to be the one that runs: in-tile adapters with every number of A columns, the
# general kernel's tiles with dependency flags (a LayerNorm in front has cleared them), with records, and without an adapter, with an
# fp32 residual, with K or the rank off 64, two column tiles of producers, ragged rows and columns.  mode: plain, res (fp32 residual), ln
@pytest.mark.parametrize("M,K,N,rank,mode,kernel", [
    (16380, 64, 320, 0, "res", "gemm16 128x160/0"), (5000, 64, 644, 8, "plain", "gemm16 128x160/1"), (5000, 640, 644, 40, "res", "gemm16 128x160/2"), (8190, 640, 640, 64, "ln", "gemm16 128x160/2"),
    (5900, 128, 320, 0, "plain", "gemm16 64x160/0"), (4757, 1280, 324, 24, "ln", "gemm16 64x160/1"), (8190, 320, 320, 40, "res", "gemm16 64x160/2"),
    (2500, 2048, 324, 0, "res", "gemm16 64x80/0"), (63, 5120, 84, 16, "res", "gemm16 64x80/1"), (1000, 2048, 644, 32, "ln", "gemm16 64x80/2"), (777, 192, 1284, 64, "plain", "gemm16 64x80/4"),
    (4100, 640, 640, 16, "plain", "gemm 128x128/8 waves/4 stages guard records"), (2100, 1280, 1284, 0, "res", "gemm 128x128/8 waves/4 stages res32"),
    (1990, 64, 1284, 128, "ln", "gemm 128x128/8 waves/4 stages flags"), (3900, 72, 644, 0, "plain", "gemm 128x128/8 waves/4 stages guard"),
    (1990, 128, 1284, 200, "res", "gemm 128x128/8 waves/4 stages res32 guard flags"), (2500, 1280, 1284, 64, "res", "gemm 128x128/8 waves/4 stages res32 records"),
    (12000, 1280, 324, 0, "plain", "gemm 256x128/8 waves/3 stages"), (4757, 1280, 1284, 64, "plain", "gemm 256x128/8 waves/3 stages records"), (4700, 1280, 1284, 128, "ln", "gemm 256x128/8 waves/3 stages flags"),
    (4757, 1288, 1284, 24, "plain", "gemm 256x128/8 waves/3 stages guard records"), (3900, 1288, 1284, 200, "res", "gemm 256x128/8 waves/3 stages res32 guard flags"), (12000, 1280, 320, 72, "res", "gemm 256x128/8 waves/3 stages res32 guard records"),
    (12000, 128, 1284, 0, "plain", "gemm 128x128/4 waves/2 stages"), (12000, 64, 644, 0, "res", "gemm 128x128/4 waves/2 stages res32"), (8190, 64, 324, 128, "ln", "gemm 128x128/4 waves/2 stages flags"),
    (8190, 64, 324, 72, "plain", "gemm 128x128/4 waves/2 stages guard records"), (12000, 128, 1284, 128, "res", "gemm 128x128/4 waves/2 stages res32 records"), (4757, 648, 644, 200, "res", "gemm 128x128/4 waves/2 stages res32 guard flags"),
    (4757, 320, 1284, 64, "ln", "gemm 64x128/4 waves/2 stages flags"), (12000, 64, 324, 8, "plain", "gemm 64x128/4 waves/2 stages guard records"), (12000, 72, 324, 0, "res", "gemm 64x128/4 waves/2 stages res32 guard"),
    (5000, 320, 1284, 200, "res", "gemm 64x128/4 waves/2 stages res32 guard flags"),
    (4757, 1280, 324, 128, "ln", "gemm 64x128/4 waves/3 stages flags"), (1, 64, 40, 128, "plain", "gemm 64x128/4 waves/3 stages records"), (1000, 1288, 324, 24, "res", "gemm 64x128/4 waves/3 stages res32 guard records"),
    (5000, 2048, 64, 64, "ln", "gemm 64x64/4 waves/5 stages flags"), (333, 1288, 40, 24, "plain", "gemm 64x64/4 waves/5 stages guard records"), (12000, 72, 64, 0, "plain", "gemm 64x64/4 waves/5 stages guard"),
    (12000, 2048, 1284, 64, "plain", "gemm 256x256/8 waves/2 stages records"),
])
def test_lora_linear_every_kernel(B, M, K, N, rank, mode, kernel):
    import torch
    r = rng(M + K + N + rank)
    p = mkproj(r, N, K, rank, bias=M % 2 == 0, scale=0.7)
    x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
    ones, zeros = np.ones(K, np.float32), np.zeros(K, np.float32)
    kw = {}
    if mode == "ln":
        kw = dict(ln_gamma=dev(ones, B), ln_beta=dev(zeros, B))
    if mode == "res":
        res = r.standard_normal((M, N)).astype(np.float32)
        kw = dict(residual=torch.from_numpy(res).cuda(), out_dtype=torch.float32)
    xd, pd = dev(x, B), B.Proj.from_numpy(p)
    call = lambda: B.lora_linear_fwd(xd, pd, **kw)
    with B.dry_run() as names:
        call()
    assert names[-1] == kernel
    got = host(call())
    rows = np.unique(np.concatenate([np.arange(0, M, 61), np.arange(max(0, M - 140), M), np.arange(min(M, 300))]))
    xr = O.layernorm(x[rows], ones, zeros) if mode == "ln" else x[rows]
    ref = O.lora_linear(xr, p["W"], p["b"], p["A"], p["B"], p["scale"])
    upd = got[rows] - (res[rows] if mode == "res" else 0)
    assert rel_err(upd, ref) <= BF16_TOL
    # every tile by itself: a wrong one must not hide behind the largest value of the whole
    assert np.isfinite(got).all() and np.abs(got - (res if mode == "res" else 0)).max() <= 2 * np.abs(ref).max()
    if rank:
        assert rel_err(O.linear(xr, p["W"], p["b"]), ref) > 3 * BF16_TOL
    assert B.gemm_dep_timeouts() == 0


# each body of the in-projection, asserted to be the one that runs: the general kernel's four, with and without an adapter and
# K or rank off 64, and the wide tiles of 256 and 128 rows with ragged rows and columns, one, two and more steps, an adapter
# segment of less than 64 columns, of exactly 64 and of more, its down-projection with one and two column tiles and a last stage of
# 320 that is full, partly filled and the only one
@pytest.mark.parametrize("M,C,F,rank,kernel", [
    (250, 1280, 2560, 24, "gemm 64x128/4 waves/3 stages geglu guard flags"), (130, 640, 1284, 0, "gemm 64x128/4 waves/3 stages geglu"),
    (2000, 320, 1284, 64, "gemm 64x128/4 waves/2 stages geglu flags"), (1001, 328, 2564, 8, "gemm 64x128/4 waves/2 stages geglu guard flags"),
    (1500, 640, 2564, 72, "gemm 128x128/4 waves/2 stages geglu guard flags"), (1500, 640, 2564, 0, "gemm 128x128/4 waves/2 stages geglu"),
    (1490, 1280, 5124, 128, "gemm 256x256/8 waves/2 stages geglu flags"), (1490, 1288, 5124, 16, "gemm 256x256/8 waves/2 stages geglu guard flags"),
    (3900, 64, 2552, 0, "geglu 256x160"), (7900, 128, 1272, 0, "geglu 256x160"), (2047, 128, 5112, 72, "geglu 256x160"), (3900, 192, 2552, 8, "geglu 256x160"),
    (3900, 384, 2560, 64, "geglu 256x160"), (2047, 1280, 5120, 128, "geglu 256x160"),
    (3900, 64, 1272, 0, "geglu 128x160"), (988, 192, 5112, 24, "geglu 128x160"), (3900, 320, 1272, 72, "geglu 128x160"), (988, 1280, 5120, 16, "geglu 128x160"),
    (1000, 640, 5120, 72, "geglu 128x160"), (988, 1344, 5112, 64, "geglu 128x160"), (1003, 960, 5112, 128, "geglu 128x160"),
])
def test_lora_linear_geglu_every_kernel(B, M, C, F, rank, kernel):
    r = rng(M + C + F + rank)
    p = mkproj(r, 2 * F, C, rank, bias=rank != 64, scale=0.6, w_std=0.05)
    x = G.bf16_round(r.standard_normal((M, C)).astype(np.float32))
    xd, pd, ones, zeros = dev(x, B), B.Proj.from_numpy(p), dev(np.ones(C, np.float32), B), dev(np.zeros(C, np.float32), B)
    call = lambda: B.lora_linear_fwd(xd, pd, ln_gamma=ones, ln_beta=zeros, epilogue=B.SD_EPI_GEGLU)
    with B.dry_run() as names:
        call()
    assert names[-1] == kernel
    y = call()
    rows = np.unique(np.concatenate([np.arange(0, M, 97), np.arange(max(0, M - 40), M), np.arange(96, min(160, M)), np.arange(min(250, M - 1), min(262, M))]))
    n = O.layernorm(x[rows], np.ones(C, np.float32), np.zeros(C, np.float32))
    ref = O.geglu(O.lora_linear(n, p["W"], p["b"], p["A"], p["B"], p["scale"]))
    assert rel_err(host(y)[rows], ref) <= BF16_TOL
    if rank:        # the adapter would be missed
        assert rel_err(O.geglu(O.linear(n, p["W"], p["b"])), ref) > 3 * BF16_TOL
    assert B.gemm_dep_timeouts() == 0


# ---------------------------------------------------------------------- attention_fwd
def vt_layout(v, B):
    """[Bn, Tk, C] -> the transposed, per-sample padded layout [C, Bn * Tkp]."""
    Bn, Tk, C = v.shape
    Tkp = (Tk + 7) // 8 * 8
    vt = np.full((C, Bn * Tkp), np.nan, np.float32)      # padding is garbage on purpose
    for b in range(Bn):
        vt[:, b * Tkp:b * Tkp + Tk] = v[b].T
    return dev(vt, B)


@pytest.mark.parametrize("Bn,Tq,Tk,heads,qscale", [
    (2, 300, 300, 2, 1.0),      # ragged self-attention, several key tiles
    (2, 256, 77, 5, 1.0),       # cross-attention shape, Tk = 77
    (1, 2048, 640, 1, 3.0),     # the 256-query kernel, peaky softmax
    (2, 130, 1, 1, 1.0),        # single key
    (1, 64, 200, 3, 8.0),       # scores with std ~ 8: online-softmax rescaling exercised
])
def test_attention_matches_oracle(B, Bn, Tq, Tk, heads, qscale):
    r = rng(Tq + Tk)
    C = heads * 64
    q = G.bf16_round((qscale * r.standard_normal((Bn, Tq, C))).astype(np.float32))
    k = G.bf16_round(r.standard_normal((Bn, Tk, C)).astype(np.float32))
    v = G.bf16_round(r.standard_normal((Bn, Tk, C)).astype(np.float32))
    if Tk > 100:
        k[:, Tk - 3] *= 8.0      # a planted large-score key in the last tile (x8 keeps bf16 values exact)
    ref = O.attention(q, k, v, heads)
    out = B.attention_fwd(dev(q, B), dev(k, B), vt_layout(v, B), heads)
    got = host(out)
    assert np.isfinite(got).all()
    assert rel_err(got, ref) <= BF16_TOL
    if Tk > 1:
        # negative control: values paired with the wrong keys move the result far beyond tolerance
        assert rel_err(O.attention(q, k, np.roll(v, 1, axis=1), heads), ref) > 10 * BF16_TOL


def test_attention_cut_tiles(B):
    """640 query tiles on a 256-CU part: the launch cuts the key range of 128 tiles in half and
    merges the halves afterwards (odd number of key tiles, ragged last one, peaky scores so the
    two halves of a tile end with different running maxima)."""
    Bn, Tq, Tk, heads = 1, 4096, 520, 20
    r = rng(4096 + 520)
    C = heads * 64
    q = G.bf16_round((2.0 * r.standard_normal((Bn, Tq, C))).astype(np.float32))
    k = G.bf16_round(r.standard_normal((Bn, Tk, C)).astype(np.float32))
    v = G.bf16_round(r.standard_normal((Bn, Tk, C)).astype(np.float32))
    k[:, 100] *= 4.0
    k[:, Tk - 2] *= 4.0
    assert B.lib().sd_attention_workspace_bytes(Bn, Tq, Tk, heads) > 256   # this shape does take the cut path
    ref = O.attention(q, k, v, heads)
    got = host(B.attention_fwd(dev(q, B), dev(k, B), vt_layout(v, B), heads))
    assert np.isfinite(got).all()
    assert rel_err(got, ref) <= BF16_TOL
    # per query tile too: a wrong merge of one cut tile must not hide behind the global maximum
    per_tile = np.abs(got - ref).reshape(Bn, Tq // 128, 128, C).max(axis=(2, 3)) / np.abs(ref).max()
    assert per_tile.max() <= BF16_TOL


def test_attention_large_scores_in_alternate_key_octets(B):
    """Keys whose index has bit 3 set score ~+770, the others ~-770: a running maximum taken
    over only part of a tile's keys would overflow the exponentials (the kernel holds the two
    octets of every 16 keys in different half-wavefronts and must exchange their maxima)."""
    Bn, Tq, Tk, heads = 1, 96, 160, 1
    r = rng(77)
    q = G.bf16_round((1.0 + 0.0625 * r.integers(-2, 3, size=(Bn, Tq, 64))).astype(np.float32))
    sign = np.where((np.arange(Tk) & 8) != 0, 1.0, -1.0).astype(np.float32)
    k = G.bf16_round((12.0 * sign)[None, :, None] * np.ones((Bn, Tk, 64), np.float32))
    v = G.bf16_round(r.standard_normal((Bn, Tk, 64)).astype(np.float32))
    ref = O.attention(q, k, v, heads)
    got = host(B.attention_fwd(dev(q, B), dev(k, B), vt_layout(v, B), heads))
    assert np.isfinite(got).all()
    assert rel_err(got, ref) <= BF16_TOL
    # and the mirrored pattern
    k2 = -k
    ref2 = O.attention(q, k2, v, heads)
    got2 = host(B.attention_fwd(dev(q, B), dev(k2, B), vt_layout(v, B), heads))
    assert np.isfinite(got2).all()
    assert rel_err(got2, ref2) <= BF16_TOL


# Plain keys of 1217 and more try without measuring the key tiles between the first and the last: ordinary scores, ragged and whole
# last tiles, key ranges cut in half; shorter ones measure every tile
@pytest.mark.parametrize("Bn,Tq,Tk,heads,qscale,kernel", [(2, 150, 1217, 2, 1.0, "attention try"), (1, 300, 1344, 1, 3.0, "attention try"), (1, 77, 1999, 3, 6.0, "attention try"),
                                                          (1, 4096, 1285, 20, 1.0, "attention try cut merge"), (2, 150, 1216, 2, 1.0, "attention")])
def test_attention_long_plain_keys(B, Bn, Tq, Tk, heads, qscale, kernel):
    r = rng(Tq + Tk)
    C = heads * 64
    q = G.bf16_round((qscale * r.standard_normal((Bn, Tq, C))).astype(np.float32))
    k = G.bf16_round(r.standard_normal((Bn, Tk, C)).astype(np.float32))
    v = G.bf16_round(r.standard_normal((Bn, Tk, C)).astype(np.float32))
    args = (dev(q, B), dev(k, B), vt_layout(v, B), heads)
    with B.dry_run() as names:
        B.attention_fwd(*args)
    assert names[0] == kernel
    got = host(B.attention_fwd(*args))
    h = np.arange(heads) if Tq * Tk < 10 ** 6 else np.array([0, 7, heads - 1])       # (of many heads, three: the last query tiles are the cut ones)
    cols = (h[:, None] * 64 + np.arange(64)).ravel()
    ref = O.attention(q[..., cols], k[..., cols], v[..., cols], len(h), dtype=np.float32 if Tq > 1000 else np.float64)
    assert np.isfinite(got).all()
    per_tile = [rel_err(got[:, i:i + 128][..., cols], ref[:, i:i + 128]) for i in range(0, Tq, 128)]
    assert max(per_tile) <= BF16_TOL
    assert rel_err(O.attention(q[:, :8][..., cols], k[..., cols], np.roll(v[..., cols], 1, axis=1), len(h)), ref[:, :8]) > 10 * BF16_TOL


# ... scores that climb from key tile to key tile, by less than 2^100 (the attempt stands) and by more than 2^128 in a middle tile
# and in the last (it overflows, and the measured form takes over), falling for half of the queries; whole and cut key ranges
@pytest.mark.parametrize("boost", [1.0, 3.2])
@pytest.mark.parametrize("Tq,Tk,heads", [(200, 64 * 20 + 23, 2), (4096, 64 * 21, 20)])
def test_attention_plain_scores_that_climb(B, boost, Tq, Tk, heads):
    r = rng(Tq + Tk)
    C = heads * 64
    nt = (Tk + 63) // 64
    level = np.zeros(nt, np.float32)                     # natural-log score of a key tile for the climbing queries
    level[3], level[nt // 2:], level[nt // 2 + 1], level[nt - 1] = 14.0, 30.0, 47.0, 40.0
    n0 = r.choice([-1.0, 1.0], 64).astype(np.float32)
    sign = np.where(r.random((1, Tq, heads, 1)) < 0.5, 1.0, -1.0)
    q = G.bf16_round((sign * n0 + 0.1 * r.standard_normal((1, Tq, heads, 64))).astype(np.float32))
    k = G.bf16_round((boost * level[np.arange(Tk) // 64][None, :, None, None] * n0 / 8.0 + 0.3 * r.standard_normal((1, Tk, heads, 64))).astype(np.float32))
    v = G.bf16_round(r.standard_normal((1, Tk, C)).astype(np.float32))
    q, k = q.reshape(1, Tq, C), k.reshape(1, Tk, C)
    up = int(np.argmax(sign[0, :, 0, 0] > 0))
    s = (q[0, up, :64].astype(np.float64) @ k[0, :, :64].T.astype(np.float64)) / 8.0 * 1.4426950408889634
    climb = max(s[64 * (nt // 2 + 1):64 * (nt // 2 + 2)].max(), 0) - s[:64].max()
    assert (40 < climb < 95) if boost == 1.0 else climb > 140
    args = (dev(q, B), dev(k, B), vt_layout(v, B), heads)
    with B.dry_run() as names:
        B.attention_fwd(*args)
    assert names[0] == ("attention try cut merge" if Tq == 4096 else "attention try")
    got = host(B.attention_fwd(*args))
    assert np.isfinite(got).all()
    h = np.array([0, 1]) if heads == 2 else np.array([0, 11, 19])
    cols = (h[:, None] * 64 + np.arange(64)).ravel()
    ref = O.attention(q[..., cols], k[..., cols], v[..., cols], len(h), dtype=np.float32 if Tq > 1000 else np.float64)
    per_tile = [rel_err(got[:, i:i + 128][..., cols], ref[:, i:i + 128]) for i in range(0, Tq, 128)]
    assert max(per_tile) <= BF16_TOL


# The kernels that a launch's tile count chooses (queries of a workgroup, groups of wavefronts that share its key range), each with a key range of an odd number
# of tiles and a ragged last one: ordinary scores, and scores that climb by more than 2^128 in a middle tile (where the first attempt, if
# any, overflows).
@pytest.mark.parametrize("climb", [False, True])
@pytest.mark.parametrize("Bn,Tq,Tk,heads,queries,groups", [(1, 130, 64 * 8 + 3, 3, 128, 2), (1, 200, 64 * 20 + 9, 2, 128, 2), (1, 1100, 64 * 24 + 61, 30, 256, 2),
                                                           (1, 1000, 64 * 20 + 10, 100, 256, 1), (1, 300, 64 * 6 + 40, 2, 128, 1)])
def test_attention_kernels_by_tile_count(B, Bn, Tq, Tk, heads, queries, groups, climb):
    r = rng(Tq + Tk)
    C = heads * 64
    nt = (Tk + 63) // 64
    level = np.zeros(nt, np.float32)
    level[nt // 2], level[nt - 1] = 150.0, 60.0
    n0 = r.choice([-1.0, 1.0], 64).astype(np.float32)
    sign = np.where(r.random((Bn, Tq, heads, 1)) < 0.5, 1.0, -1.0).astype(np.float32)
    q = (0.3 * r.standard_normal((Bn, Tq, heads, 64), dtype=np.float32) + (sign * n0 if climb else 0)).astype(np.float32)
    k = r.standard_normal((Bn, Tk, heads, 64), dtype=np.float32) * (0.3 if climb else 3.0) + (level[np.arange(Tk) // 64][None, :, None, None] * n0 / 8.0 if climb else 0)
    q, k = G.bf16_round(q).reshape(Bn, Tq, C), G.bf16_round(k.astype(np.float32)).reshape(Bn, Tk, C)
    v = G.bf16_round(r.standard_normal((Bn, Tk, C), dtype=np.float32))
    args = (dev(q, B), dev(k, B), vt_layout(v, B), heads)
    with B.dry_run(detail=3) as names:
        B.attention_fwd(*args)
    assert names[0] == "attention%s, %d queries, %d groups" % (" try" if nt >= 20 else "", queries, groups)
    got = host(B.attention_fwd(*args))
    assert np.isfinite(got).all()
    h = np.array(sorted({0, heads // 2, heads - 1}))
    cols = (h[:, None] * 64 + np.arange(64)).ravel()
    ref = O.attention(q[..., cols], k[..., cols], v[..., cols], len(h), dtype=np.float32 if Tq >= 1000 else np.float64)
    per_tile = [rel_err(got[:, i:i + 128][..., cols], ref[:, i:i + 128]) for i in range(0, Tq, 128)]
    assert max(per_tile) <= BF16_TOL


# ... and inside a block, with prescaled keys: 256 queries and one group
def test_attn_block_of_many_tiles(B):
    import torch
    Bn, T, C = 8, 1290, 640
    r = rng(T)
    ps = [mkproj(r, C, C, 0, bias=i == 3, scale=1.0) for i in range(4)]
    g, b = G.bf16_round((1 + 0.02 * r.standard_normal(C)).astype(np.float32)), G.bf16_round((0.02 * r.standard_normal(C)).astype(np.float32))
    x = r.standard_normal((Bn, T, C), dtype=np.float32)
    args = (torch.from_numpy(x).cuda(), None, dev(g, B), dev(b, B), *[B.Proj.from_numpy(p) for p in ps], C // 64)
    with B.dry_run(detail=3) as names:
        B.attn_block_fwd(*args)
    assert "attention prescaled try, 256 queries, 1 groups" in names
    y = host(B.attn_block_fwd(*args))
    for s in (0, Bn - 1):        # (samples do not meet)
        ref = O.attn_sublayer(x[s:s + 1], None, g, b, *ps, C // 64)
        assert rel_err(y[s:s + 1] - x[s:s + 1], ref - x[s:s + 1]) <= BF16_TOL


# Row sums just under the top of the fp32 range: one key of each half-wavefront's octets scores 2^127.3 above the first key
# tile, so either half's sum is finite and their sum is not.  (1217 keys and more take the attempt without maxima; the values
# are small, so that the accumulators stay in range.)  Whole tiles, and tiles whose halves are merged.
@pytest.mark.parametrize("Bn,Tq,Tk,heads", [(1, 200, 1300, 1), (1, 200, 400, 1), (1, 4096, 1220, 20)])
def test_attention_row_sums_at_the_top_of_the_range(B, Bn, Tq, Tk, heads):
    r = rng(Tk)
    C = heads * 64
    q = np.full((Bn, Tq, C), 4.0, np.float32)
    k = np.zeros((Bn, Tk, C), np.float32)
    k[:, [300, 308]] = np.tile(np.repeat(np.array([2.75, 2.765625], np.float32), 32), heads)
    score = float(q[0, 0, :64] @ k[0, 300, :64]) / 8.0 * 1.4426950408889634
    assert 127.0 < score < 127.6 and 2.0 * 2.0 ** score > 3.41e38
    v = G.bf16_round((1e-3 * r.standard_normal((Bn, Tk, C))).astype(np.float32))
    got = host(B.attention_fwd(dev(q, B), dev(k, B), vt_layout(v, B), heads))
    ref = (v[:, 300:301].astype(np.float64) + v[:, 308:309]) / 2 + np.zeros_like(q)     # every other key weighs 2^-127
    assert np.abs(O.attention(q[:, :1], k, v, heads) - ref[:, :1]).max() <= 1e-9
    assert rel_err(got, ref) <= BF16_TOL


# ------------------------------------------------------- attn_block_fwd / ff_block_fwd
def small_cfg(**kw):
    base = dict(name="t", Bn=2, T=200, C=128, heads=2, depth=1, r=8, alpha=4.0, lora_ff=True, Tc=77, Dc=256,
                w_std=0.08, ctx_std=1.0, a_std=0.3, b_std=0.08)
    base.update(kw)
    return G.StackConfig(**base)


@pytest.mark.parametrize("cross", [False, True])
@pytest.mark.parametrize("io", ["f32", "bf16"])
def test_attn_block_matches_oracle(B, cross, io):
    import torch
    cfg = small_cfg()
    p = G.make_stack_inputs(cfg, seed=3)
    blk = p["blocks"][0]
    names = ("q2", "k2", "v2", "o2", "ln2_g", "ln2_b") if cross else ("q1", "k1", "v1", "o1", "ln1_g", "ln1_b")
    pq, pk, pv, po, g, b = (blk[n] for n in names)
    h = p["x"] if io == "bf16" else rng(5).standard_normal(p["x"].shape).astype(np.float32)
    ctx = p["ctx"] if cross else None
    ref = O.attn_sublayer(h, ctx, g, b, pq, pk, pv, po, cfg.heads)
    hd = dev(h, B) if io == "bf16" else torch.from_numpy(h).cuda()
    y = B.attn_block_fwd(hd, dev(ctx, B) if cross else None, dev(g, B), dev(b, B), B.Proj.from_numpy(pq), B.Proj.from_numpy(pk),
                         B.Proj.from_numpy(pv), B.Proj.from_numpy(po), cfg.heads)
    got = host(y)
    if io == "f32":
        # the update alone, normalised by its own maximum
        assert rel_err(got - h, ref - h) <= BF16_TOL
        # negative controls on the update: no adapter, or a zeroed context, is visible
        nol = [dict(q, A=None, B=None) for q in (pq, pk, pv, po)]
        assert rel_err(O.attn_sublayer(h, ctx, g, b, *nol, cfg.heads) - h, ref - h) > 3 * BF16_TOL
        if cross:
            assert rel_err(O.attn_sublayer(h, np.zeros_like(ctx), g, b, pq, pk, pv, po, cfg.heads) - h, ref - h) > 3 * BF16_TOL
    else:
        assert rel_err(got, ref) <= BF16_TOL


@pytest.mark.parametrize("Bn,T,Tc,C,heads,rank", [(1, 1, 1, 64, 1, 8), (3, 70, 5, 64, 1, 16), (2, 129, 100, 128, 2, 72),
                                                   (1, 600, 77, 192, 3, 128), (2, 257, 130, 128, 2, 8)])
def test_attn_block_ragged_sizes(B, Bn, T, Tc, C, heads, rank):
    """Self- and cross-attention sub-layers at ragged token counts, including ranks above 64 and
    context lengths that are not multiples of 8: the v^T projection is a transposed problem whose
    tiles wait for the down-projection row blocks that cover their token columns."""
    import torch
    # alpha fixed: the adapter's share of q and k, and with it the score scale, does not grow with the rank
    cfg = small_cfg(Bn=Bn, T=T, Tc=Tc, C=C, heads=heads, r=rank, alpha=8.0, Dc=72)
    p = G.make_stack_inputs(cfg, seed=T + Tc)
    blk = p["blocks"][0]
    h = rng(T).standard_normal(p["x"].shape).astype(np.float32)
    for cross in (False, True):
        names = ("q2", "k2", "v2", "o2", "ln2_g", "ln2_b") if cross else ("q1", "k1", "v1", "o1", "ln1_g", "ln1_b")
        pq, pk, pv, po, g, b = (blk[n] for n in names)
        ctx = p["ctx"] if cross else None
        ref = O.attn_sublayer(h, ctx, g, b, pq, pk, pv, po, cfg.heads)
        args = (torch.from_numpy(h).cuda(), dev(ctx, B) if cross else None, dev(g, B), dev(b, B), B.Proj.from_numpy(pq),
                B.Proj.from_numpy(pk), B.Proj.from_numpy(pv), B.Proj.from_numpy(po), cfg.heads)
        y = B.attn_block_fwd(*args)
        assert rel_err(host(y) - h, ref - h) <= BF16_TOL, (cross,)
        try:        # the same call as two launches per projection: same bits
            B.set_projection_fusion(False)
            y2 = B.attn_block_fwd(*args)
        finally:
            B.set_projection_fusion(True)
        assert torch.equal(y, y2), (cross,)
    assert B.gemm_dep_timeouts() == 0


# q, k and v transposed sharing a launch of more than one round (eight wavefronts): adapters of whole and partial k-steps, none,
# and two column tiles of them; row, column and token remainders
@pytest.mark.parametrize("rank,flags", [(64, " flags"), (8, " guard flags"), (0, ""), (72, " guard flags")])
def test_attn_block_projections_in_several_rounds(B, rank, flags):
    import torch
    # Weights that hold the scores near 1.  q and k are each rounded to bf16, so a score of size s is off by up to s 2^-8 and its
    # probability by that fraction; with small_cfg's own the scores of 320 channels and rank 8 reach 17 (17 2^-8 = 0.066 of a
    # probability that may be most of its row), here 6, of which the row's mean over 3101 keys leaves a tenth.
    cfg = small_cfg(Bn=3, T=3101, Tc=5, C=320, heads=5, r=max(rank, 8), alpha=8.0, Dc=72, w_std=0.05, a_std=0.15)
    p = G.make_stack_inputs(cfg, seed=rank)
    blk = p["blocks"][0]
    h = rng(rank).standard_normal(p["x"].shape).astype(np.float32)
    projs = [dict(blk[n], A=None, B=None) if rank == 0 else blk[n] for n in ("q1", "k1", "v1", "o1")]
    ref = O.attn_sublayer(h, None, blk["ln1_g"], blk["ln1_b"], *projs, cfg.heads)
    args = (torch.from_numpy(h).cuda(), None, dev(blk["ln1_g"], B), dev(blk["ln1_b"], B), *[B.Proj.from_numpy(q) for q in projs], cfg.heads)
    with B.dry_run() as names:
        B.attn_block_fwd(*args)
    assert "gemm 128x128/8 waves/2 stages" + flags in names
    y = B.attn_block_fwd(*args)
    assert rel_err(host(y) - h, ref - h) <= BF16_TOL
    try:        # the same call as two launches per projection: same bits
        B.set_projection_fusion(False)
        y2 = B.attn_block_fwd(*args)
    finally:
        B.set_projection_fusion(True)
    assert torch.equal(y, y2)
    assert B.gemm_dep_timeouts() == 0


# every tile cut in half along the keys: from 24 key tiles and up to two tiles per CU, where that takes work off the most loaded CU, from
# 48 also at one tile per CU; tile counts that are a multiple of 4 and not,
# odd and ragged key tiles.  Bits do not depend on which half arrives last nor on where the halves are merged; a workspace without
# room for them still does.
@pytest.mark.parametrize("Bn,T,heads,cut", [(1, 1472, 2, ""), (1, 1473, 2, " cut"), (3, 1601, 1, " cut"), (1, 2050, 5, " cut"), (2, 1536, 13, " cut"), (2, 1536, 20, ""), (8, 1473, 8, ""), (1, 4096, 5, " cut")])
def test_attn_block_every_tile_cut(B, Bn, T, heads, cut):
    import torch
    C = 64 * heads
    cfg = small_cfg(Bn=Bn, T=T, Tc=5, C=C, heads=heads, r=8, alpha=8.0, Dc=72, w_std=0.05 * (320 / C) ** 0.5, a_std=0.15)
    p = G.make_stack_inputs(cfg, seed=T)
    blk = p["blocks"][0]
    h = rng(T).standard_normal(p["x"].shape).astype(np.float32)
    projs = [dict(blk[n], A=None, B=None) for n in ("q1", "k1", "v1", "o1")]
    args = (torch.from_numpy(h).cuda(), None, dev(blk["ln1_g"], B), dev(blk["ln1_b"], B), *[B.Proj.from_numpy(q) for q in projs], heads)
    need = B.lib().sd_attn_block_workspace_bytes(Bn, T, C, 0, 0, 0)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    with B.dry_run() as names:
        B.attn_block_fwd(*args, ws=ws)
    assert "attention prescaled try" + cut in names
    y = B.attn_block_fwd(*args, ws=ws)
    ref = O.attn_sublayer(h, None, blk["ln1_g"], blk["ln1_b"], *projs, heads)
    assert rel_err(host(y) - h, ref - h) <= BF16_TOL
    for _ in range(3):
        assert torch.equal(B.attn_block_fwd(*args, ws=ws), y)
    try:
        B.set_projection_fusion(False)
        assert torch.equal(B.attn_block_fwd(*args, ws=ws), y)
    finally:
        B.set_projection_fusion(True)
    if cut:
        tiles = (T + 127) // 128 * heads * Bn
        little = ws[:need - tiles * 2 * 34 * 256 * 4]
        with B.dry_run() as names:
            B.attn_block_fwd(*args, ws=little)
        assert "attention prescaled try" in names
        assert rel_err(host(B.attn_block_fwd(*args, ws=little)) - h, ref - h) <= BF16_TOL
        with pytest.raises(Exception):
            B.attn_block_fwd(*args, ws=little[:-256])


# self-attention whose q, k and transposed v are one round of 128x160 tiles (token counts off every tile, adapters or none) or of 64x80
@pytest.mark.parametrize("Bn,T,C,rank", [(2, 700, 640, 16), (1, 1003, 640, 0), (2, 261, 320, 24)])
def test_attn_block_projections_in_one_round(B, Bn, T, C, rank):
    import torch
    r = rng(T + C)
    ps = [mkproj(r, C, C, rank, bias=i == 3, scale=0.5) for i in range(4)]
    g, b = G.bf16_round((1 + 0.02 * r.standard_normal(C)).astype(np.float32)), G.bf16_round((0.02 * r.standard_normal(C)).astype(np.float32))
    x = r.standard_normal((Bn, T, C)).astype(np.float32)
    y = B.attn_block_fwd(torch.from_numpy(x).cuda(), None, dev(g, B), dev(b, B), *[B.Proj.from_numpy(p) for p in ps], C // 64)
    ref = O.attn_sublayer(x, None, g, b, *ps, C // 64)
    assert rel_err(host(y) - x, ref - x) <= BF16_TOL


@pytest.mark.parametrize("T,Tc", [(256, 128), (200, 77)])
def test_attn_block_with_biased_q_k_v(B, T, Tc):
    """A projection record may carry a bias whatever its role.  With one on k the keys cannot leave
    their projection pre-multiplied by the softmax scale (the attention kernel scales the scores
    itself), and one on v is a per-row bias of the transposed v^T problem; T = 256 gives tiles that
    lie inside the output, T = 200 ragged ones."""
    import torch
    cfg = small_cfg(Bn=2, T=T, Tc=Tc, C=128, heads=2, r=16)
    p = G.make_stack_inputs(cfg, seed=11)
    blk = p["blocks"][0]
    r = rng(T + 1)
    h = r.standard_normal(p["x"].shape).astype(np.float32)
    for cross in (False, True):
        names = ("q2", "k2", "v2", "o2", "ln2_g", "ln2_b") if cross else ("q1", "k1", "v1", "o1", "ln1_g", "ln1_b")
        pq, pk, pv, po, g, b = (blk[n] for n in names)
        pq, pk, pv = (dict(q, b=G.bf16_round((0.5 * r.standard_normal(q["W"].shape[0])).astype(np.float32))) for q in (pq, pk, pv))
        ctx = p["ctx"] if cross else None
        ref = O.attn_sublayer(h, ctx, g, b, pq, pk, pv, po, cfg.heads)
        y = B.attn_block_fwd(torch.from_numpy(h).cuda(), dev(ctx, B) if cross else None, dev(g, B), dev(b, B), B.Proj.from_numpy(pq),
                             B.Proj.from_numpy(pk), B.Proj.from_numpy(pv), B.Proj.from_numpy(po), cfg.heads)
        assert rel_err(host(y) - h, ref - h) <= BF16_TOL, (cross,)
        # the q and v biases matter at this tolerance; a k bias shifts every score of a query by
        # the same amount, which softmax removes (so the GPU's scaling of biased keys is what is tested)
        for drop in range(3):
            qs = [pq, pk, pv]
            qs[drop] = dict(qs[drop], b=None)
            e = rel_err(O.attn_sublayer(h, ctx, g, b, *qs, po, cfg.heads) - h, ref - h)
            assert (e < 1e-9) if drop == 1 else (e > 3 * BF16_TOL), (cross, drop, e)


def test_attn_block_long_keys_with_a_k_bias(B):
    """A k bias keeps the keys from being prescaled: in a self-attention of 1300 tokens the attention kernel tries on plain keys."""
    import torch
    T, C = 1300, 128
    r = rng(T)
    ps = [mkproj(r, C, C, 16, bias=True, scale=0.5) for _ in range(4)]
    g, b = np.ones(C, np.float32), np.zeros(C, np.float32)
    x = r.standard_normal((1, T, C)).astype(np.float32)
    args = (torch.from_numpy(x).cuda(), None, dev(g, B), dev(b, B), *[B.Proj.from_numpy(p) for p in ps], 2)
    with B.dry_run() as names:
        B.attn_block_fwd(*args)
    assert "attention try" in names
    y = B.attn_block_fwd(*args)
    ref = O.attn_sublayer(x, None, g, b, *ps, 2)
    assert rel_err(host(y) - x, ref - x) <= BF16_TOL


def test_ff_block_matches_oracle(B):
    import torch
    cfg = small_cfg(T=150, C=192, heads=3)
    p = G.make_stack_inputs(cfg, seed=4)
    blk = p["blocks"][0]
    h = rng(6).standard_normal((cfg.M, cfg.C)).astype(np.float32)
    ref = O.ff_sublayer(h, blk["ln3_g"], blk["ln3_b"], blk["ff1"], blk["ff2"])
    y = B.ff_block_fwd(torch.from_numpy(h).cuda(), dev(blk["ln3_g"], B), dev(blk["ln3_b"], B),
                       B.Proj.from_numpy(blk["ff1"]), B.Proj.from_numpy(blk["ff2"]))
    assert rel_err(host(y) - h, ref - h) <= BF16_TOL


# ---------------------------------------------------------------------- groupnorm_fwd
@pytest.mark.parametrize("Bn,T,C", [(2, 256, 320), (1, 70, 64), (2, 1000, 640), (1, 33, 1280)])
def test_groupnorm_matches_oracle(B, Bn, T, C):
    r = rng(T + C)
    x = G.bf16_round((r.standard_normal((Bn, T, C)) * 1.5 + r.standard_normal((Bn, 1, C)) * 2).astype(np.float32))
    g = G.bf16_round((1 + 0.1 * r.standard_normal(C)).astype(np.float32))
    b = G.bf16_round((0.1 * r.standard_normal(C)).astype(np.float32))
    ref = O.groupnorm(x, g, b)
    y = B.groupnorm_fwd(dev(x, B), dev(g, B), dev(b, B))
    assert rel_err(host(y), ref) <= BF16_TOL
    # the fused GroupNorm + SiLU operator of the ResNet blocks
    ref_s = O.groupnorm_silu(x, g, b)
    ys = B.groupnorm_silu_fwd(dev(x, B), dev(g, B), dev(b, B))
    assert rel_err(host(ys), ref_s) <= BF16_TOL
    assert rel_err(ref, ref_s) > 10 * BF16_TOL          # the activation is visible at this tolerance


# slabs of whole rows: more rows than threads, several slabs a workgroup, a last one that is partly empty; channel counts that
# are no multiple of 8 (2-channel accesses); more groups than threads of a row; the largest row
@pytest.mark.parametrize("Bn,T,C,groups", [(1, 1, 64, 32), (3, 27, 320, 32), (1, 5000, 320, 32), (2, 1537, 960, 32), (1, 300, 36, 3), (2, 130, 100, 50),
                                           (1, 40, 2048, 1024), (1, 2100, 2046, 33)])
def test_groupnorm_slabs_match_oracle(B, Bn, T, C, groups):
    r = rng(T + C + groups)
    x = G.bf16_round((r.standard_normal((Bn, T, C)) * 1.5 + r.standard_normal((Bn, 1, C)) * 2).astype(np.float32))
    g = G.bf16_round((1 + 0.1 * r.standard_normal(C)).astype(np.float32))
    b = G.bf16_round((0.1 * r.standard_normal(C)).astype(np.float32))
    y = B.groupnorm_fwd(dev(x, B), dev(g, B), dev(b, B), groups=groups)
    assert rel_err(host(y), O.groupnorm(x, g, b, groups=groups)) <= BF16_TOL


# partials per thread in one batch, in several and in a last one that is partly empty; chunks whose last slab is; three and more
# partial workgroups whose count is not a multiple of anything
@pytest.mark.parametrize("Bn,T,C,groups", [(1, 400, 2048, 1024), (2, 700, 1000, 250), (1, 1023, 1280, 32), (3, 49, 320, 32), (2, 8191, 640, 16), (70, 33, 64, 2)])
def test_groupnorm_partial_batches_match_oracle(B, Bn, T, C, groups):
    r = rng(T + C + groups)
    x = G.bf16_round((r.standard_normal((Bn, T, C)) * 1.5 + r.standard_normal((Bn, 1, C)) * 2).astype(np.float32))
    g = G.bf16_round((1 + 0.1 * r.standard_normal(C)).astype(np.float32))
    b = G.bf16_round((0.1 * r.standard_normal(C)).astype(np.float32))
    ref = O.groupnorm(x, g, b, groups=groups)
    got = host(B.groupnorm_fwd(dev(x, B), dev(g, B), dev(b, B), groups=groups))
    assert rel_err(got, ref) <= BF16_TOL
    assert np.abs(got - ref).mean() <= 2e-3 * np.abs(ref).mean() * 2       # bf16 rounds by 2^-9 at most, a wrong statistic moves everything


# inputs of as many slabs as take all six to a workgroup, where the statistics and the affine are requested ahead of the rows (with SiLU; without, in as many
# workgroups as a round and less): more groups than threads, less than a 16-byte piece to a group, the last slab cut off, one row short of that many slabs; and
# channels off eight, where they are not
@pytest.mark.parametrize("Bn,T,C,groups", [(1, 2043, 2048, 1024), (2, 1201, 1280, 32), (1, 12000, 100, 10), (4, 3100, 320, 32), (2, 12239, 320, 160), (1, 12228, 320, 32)])
def test_groupnorm_large_matches_oracle(B, Bn, T, C, groups):
    r = rng(T + C)
    x = G.bf16_round((r.standard_normal((Bn, T, C)) + 3.0 * r.standard_normal((Bn, 1, C))).astype(np.float32))
    g, b = G.bf16_round((1 + 0.1 * r.standard_normal(C)).astype(np.float32)), G.bf16_round((0.1 * r.standard_normal(C)).astype(np.float32))
    for call, ref in ((B.groupnorm_fwd, O.groupnorm), (B.groupnorm_silu_fwd, O.groupnorm_silu)):
        assert rel_err(host(call(dev(x, B), dev(g, B), dev(b, B), groups=groups)), ref(x, g, b, groups=groups)) <= BF16_TOL


# samples of one launch: a thread holds one row, two, three, four and, one token later, two launches; units of one group, two and
# four; pieces of a row of 64 bytes and of a whole row; a batch just too large
@pytest.mark.parametrize("Bn,T,C,groups,unit", [(1, 1, 320, 32, 1), (2, 204, 320, 32, 1), (2, 205, 640, 32, 1), (1, 408, 1280, 32, 1), (3, 409, 320, 32, 1), (1, 816, 640, 32, 1),
                                                (1, 817, 640, 32, 0), (2, 100, 960, 32, 1), (1, 4, 2048, 1, 1), (1, 5, 2048, 1, 1), (2, 17, 2048, 1, 0), (2, 300, 64, 2, 1),
                                                (2, 300, 96, 4, 0), (1, 777, 48, 2, 0), (8, 409, 1280, 32, 1), (8, 410, 1280, 32, 0)])
def test_groupnorm_one_launch_matches_oracle(B, Bn, T, C, groups, unit):
    r = rng(T + C + groups)
    x = G.bf16_round((r.standard_normal((Bn, T, C)) * 1.5 + r.standard_normal((Bn, 1, C)) * 2).astype(np.float32))
    g = G.bf16_round((1 + 0.1 * r.standard_normal(C)).astype(np.float32))
    b = G.bf16_round((0.1 * r.standard_normal(C)).astype(np.float32))
    xd, gd, bd = dev(x, B), dev(g, B), dev(b, B)
    with B.dry_run() as names:
        B.groupnorm_fwd(xd, gd, bd, groups=groups)
    assert names == ["groupnorm unit" if unit else "groupnorm"]
    for call, ref in ((B.groupnorm_fwd, O.groupnorm), (B.groupnorm_silu_fwd, O.groupnorm_silu)):
        want = ref(x, g, b, groups=groups)
        got = host(call(xd, gd, bd, groups=groups))
        assert rel_err(got, want) <= BF16_TOL
        assert np.abs(got - want).mean() <= 2e-3 * np.abs(want).mean() * 2     # bf16 rounds by 2^-9 at most


# ------------------------------------------------------------ spatial_transformer_fwd
def run_stack(B, cfg, seed=0):
    p = G.make_stack_inputs(cfg, seed)
    sp = B.StackParams(p)
    y = B.spatial_transformer_fwd(dev(p["x"], B), dev(p["ctx"], B), sp, cfg.heads)
    return p, host(y)


def test_stack_small_ragged(B):
    cfg = small_cfg(T=200, depth=2)
    p, got = run_stack(B, cfg, seed=1)
    ref = O.spatial_transformer(p["x"], p["ctx"], p, cfg.heads)
    assert rel_err(got, ref) <= BF16_TOL
    assert rel_err(got - p["x"], ref - p["x"]) <= 2 * BF16_TOL     # what the stack adds, bf16 output rounding included


# text keys / values of the second block in the first one's ff2 launch (128x128 tiles in one round, 256x128 tiles) or, where ff2 takes its
# adapter into the tile, in the block's own q, k, v launch; of three samples, where ff2 takes 256x128 tiles for them, too; as two launches per
# projection they are in the latter: same bits
@pytest.mark.parametrize("Bn,T,Tc,rank,ff2,alone", [(1, 3300, 77, 64, "gemm 128x128/8 waves/4 stages res32 flags", ""), (3, 1800, 131, 64, "gemm 256x128/8 waves/3 stages res32 flags", ""),
                                                    (3, 1600, 131, 64, "gemm 256x128/8 waves/3 stages res32 flags", "gemm 128x128/8 waves/4 stages res32 flags"), (1, 3300, 77, 16, "gemm16 64x160/1", "")])
def test_stack_text_keys_in_the_ff2_launch(B, Bn, T, Tc, rank, ff2, alone):
    import torch
    # adapter scale 1/8 at either rank.  (At 1/2, rank 16, q and k have a deviation of 1.4 and scores reach 10: rounded to bf16, q and k
    # put such a score off by 10 2^-8 = 0.04, and with it a probability that is most of its row.)
    cfg = small_cfg(Bn=Bn, T=T, Tc=Tc, C=640, heads=10, r=rank, alpha=rank / 8, depth=2, w_std=0.03)
    p = G.make_stack_inputs(cfg, seed=T)
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    with B.dry_run(detail=True) as names:
        B.spatial_transformer_fwd(x, ctx, sp, cfg.heads)
    norms = [i for i, n in enumerate(names) if n.startswith("layernorm")]
    kernel, problems = zip(*(n.split(", ")[:2] for n in (names[norms[3] - 1], names[-2])))       # ff2 of both blocks, the last launches of theirs
    assert kernel == (ff2, alone or ff2)
    text = 0 if ff2.startswith("gemm16") else 2 + 2 * Bn
    assert [int(p.split()[0]) for p in problems] == [text + (1 if ff2.startswith("gemm16") else 2), 1 if ff2.startswith("gemm16") else 2]
    y = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads).clone()
    ref = O.spatial_transformer(p["x"], p["ctx"], p, cfg.heads)
    assert rel_err(host(y), ref) <= BF16_TOL
    try:
        B.set_projection_fusion(False)
        assert torch.equal(B.spatial_transformer_fwd(x, ctx, sp, cfg.heads), y)
    finally:
        B.set_projection_fusion(True)
    assert B.gemm_dep_timeouts() == 0


# a stack in a workspace that lacks the room for the halves of cut attention tiles, and what lies behind that room moves up
@pytest.mark.parametrize("Bn,T,C", [(1, 4096, 320), (1, 1500, 640)])
def test_stack_in_a_workspace_without_room_for_cut_tiles(B, Bn, T, C):
    import torch
    cfg = small_cfg(Bn=Bn, T=T, Tc=77, C=C, heads=C // 64, r=16, alpha=2.0, depth=1, w_std=0.03)
    p = G.make_stack_inputs(cfg, seed=T)
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    need = B.spatial_transformer_workspace_bytes(Bn, T, C, 77, cfg.Dc, sp.r_max)
    least = need - (T + 127) // 128 * cfg.heads * Bn * 2 * 34 * 256 * 4
    ref = O.spatial_transformer(p["x"], p["ctx"], p, cfg.heads)
    for size, cut in ((need, " cut"), (least, "")):
        ws = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")       # and what lies behind it stays as it is
        with B.dry_run() as names:
            B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws[:size])
        assert "attention prescaled try" + cut in names
        y = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws[:size])
        assert rel_err(host(y), ref) <= BF16_TOL
        assert bool((ws[size:] == 0x5A).all())
    with pytest.raises(B.SwiftDiffError) as e:
        B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws[:least - 256])
    assert e.value.code == -3


# deep stacks, whose attention (tiles cut in half; whole ones to the text) and LayerNorm launches (rows of 640 and of 1280 channels) read
# weights ahead
@pytest.mark.parametrize("Bn,T,C,depth", [(1, 1500, 640, 11), (1, 2100, 1280, 3)])
def test_deep_stack_reads_weights_ahead(B, Bn, T, C, depth):
    import torch
    cfg = small_cfg(Bn=Bn, T=T, Tc=77, C=C, heads=C // 64, Dc=2048, r=16, alpha=2.0, depth=depth, w_std=0.02)
    p = G.make_stack_inputs(cfg, seed=T)
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    with B.dry_run(detail=True) as names:
        B.spatial_transformer_fwd(x, ctx, sp, cfg.heads)
    for what in ("attention prescaled try cut, ahead", "attention prescaled try, ahead", "layernorm, ahead"):
        assert any(n.startswith(what) for n in names), what
    y = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads).clone()
    ref = O.spatial_transformer(p["x"], p["ctx"], p, cfg.heads)
    assert rel_err(host(y), ref) <= BF16_TOL
    for _ in range(3):
        assert torch.equal(B.spatial_transformer_fwd(x, ctx, sp, cfg.heads), y)


# several blocks of one launch each from self-attention to the feed-forward, one after the other in the same buffers; and stacks whose weights it reads ahead too
@pytest.mark.parametrize("Bn,T,C,depth,ahead", [(10, 300, 640, 3, 0), (40, 100, 320, 2, 0), (10, 300, 640, 11, 10), (46, 350, 320, 18, 10)])
def test_deep_stack_chain(B, Bn, T, C, depth, ahead):
    import torch
    cfg = small_cfg(Bn=Bn, T=T, Tc=77, C=C, heads=C // 64, Dc=2048, r=16, alpha=2.0, depth=depth, w_std=0.02)
    p = G.make_stack_inputs(cfg, seed=T + depth)
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    with B.dry_run(detail=True) as names:
        B.spatial_transformer_fwd(x, ctx, sp, cfg.heads)
    assert sum(n.startswith("attention of the chain") for n in names) == depth
    assert sum(n.startswith("layernorm of the chain, ahead") for n in names) >= ahead and ("ahead" in " ".join(names)) == (ahead > 0)
    ws = torch.full((B.spatial_transformer_workspace_bytes(Bn, T, C, 77, cfg.Dc, sp.r_max),), 0xFF, dtype=torch.uint8, device="cuda")   # (what no launch wrote is NaN)
    y = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws).clone()
    some = [0, Bn - 1]
    ref = O.spatial_transformer(p["x"][some], p["ctx"][some], p, cfg.heads)
    assert rel_err(host(y)[some], ref) <= BF16_TOL
    for _ in range(3):
        assert torch.equal(B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws), y)


# few rows: K split over eight wavefronts (fewer slices than wavefronts, uneven shares, one and two stages in flight), tiles of 32x32, 32x64, 64x64
# and 64x32, rows cut off, ranks that fill one block of A, two, four and none whole; no bias, or one with a residual
@pytest.mark.parametrize("M,K,N,rank,res,kernel", [
    (1, 320, 64, 8, "", "thin 32x32/1"), (33, 384, 320, 0, "f32", "thin 32x32/0"), (154, 2048, 1280, 64, "", "thin 32x32/4"), (250, 1088, 640, 40, "bf16", "thin 32x32/4"), (77, 576, 128, 32, "f32", "thin 32x32/2"),
    (300, 1280, 1280, 16, "", "thin 32x64/1"), (1000, 320, 320, 24, "bf16", "thin 32x64/2"), (309, 1024, 1280, 0, "", "thin 32x64/0"),
    (1000, 2560, 640, 16, "f32", "thin 64x64/1"), (499, 1280, 1280, 32, "", "thin 64x64/2"), (1990, 1088, 320, 0, "f32", "thin 64x64/0"), (305, 640, 1280, 64, "f32", "thin 64x32/4"),
])
def test_lora_linear_few_rows(B, M, K, N, rank, res, kernel):
    import torch
    r = rng(M + K + N + rank)
    p = mkproj(r, N, K, rank, bias=bool(res), scale=0.7)
    x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
    rs = G.bf16_round(r.standard_normal((M, N)).astype(np.float32))
    rd = None if not res else torch.from_numpy(rs).cuda() if res == "f32" else torch.from_numpy(rs).cuda().bfloat16()
    call = lambda: B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(p), residual=rd, out_dtype=torch.float32 if res == "f32" else torch.bfloat16)
    with B.dry_run() as names:
        call()
    assert names[-1] == kernel
    ref = O.lora_linear(x, p["W"], p["b"], p["A"], p["B"], p["scale"])
    got = host(call()) - (rs if res else 0)
    # (a bf16 sum is rounded once more: half a unit in the last of 8 bits of it)
    allow = 2.0 ** -9 * (np.abs(ref).max() + np.abs(rs).max()) if res == "bf16" else 0
    assert np.abs(got - ref).max() <= BF16_TOL * np.abs(ref).max() + allow


def test_attn_block_few_rows(B):
    """q, keys and values (stored transposed) of one group, cut-off rows, an adapter on the keys only."""
    import torch
    r = rng(77)
    Bn, T, C, Tc, Dc = 2, 77, 128, 21, 320
    h = r.standard_normal((Bn, T, C)).astype(np.float32)
    ctx = G.bf16_round(r.standard_normal((Bn, Tc, Dc)).astype(np.float32))
    g, b = np.ones(C, np.float32), np.zeros(C, np.float32)
    projs = [mkproj(r, C, C, 0, bias=False), mkproj(r, C, Dc, 40, bias=False, scale=0.1), mkproj(r, C, Dc, 0, bias=False), mkproj(r, C, C, 8, scale=0.5)]
    args = (torch.from_numpy(h).cuda(), dev(ctx, B), dev(g, B), dev(b, B), *[B.Proj.from_numpy(p) for p in projs], C // 64)
    with B.dry_run() as names:
        B.attn_block_fwd(*args)
    assert "thin 32x32/4" in names
    got = host(B.attn_block_fwd(*args))
    assert rel_err(got - h, O.attn_sublayer(h, ctx, g, b, *projs, C // 64) - h) <= BF16_TOL


# from self-attention's output to the feed-forward's input in one launch: blocks of 32 rows cut off at each row count, text keys about the ends
# of the 64 and 16 that are fetched together and of groups of eight, ranks about those of the tiles of A and of the steps of B (none, less than a
# tile, beside each other), biased projections (keys that are not scaled ahead).  Of 320 channels in
# one workgroup a CU, two, and a second round; of 640 in one round and in two.
@pytest.mark.parametrize("Bn,T,C,Tc,rank,bias", [(38, 1, 320, 1, 0, False), (40, 31, 320, 7, 8, False), (39, 32, 320, 64, 40, True), (20, 33, 320, 65, 128, False), (13, 70, 320, 80, 72, False),
                                                 (41, 71, 640, 77, 64, False), (45, 65, 640, 63, 16, True), (31, 95, 640, 72, 128, False), (167, 95, 640, 77, 0, False), (150, 95, 320, 16, 24, False),
                                                 (208, 95, 320, 7, 8, False)])
def test_stack_chain(B, Bn, T, C, Tc, rank, bias):
    import torch
    cfg = small_cfg(Bn=Bn, T=T, Tc=Tc, C=C, heads=C // 64, r=rank, alpha=rank / 8, depth=1, w_std=0.03, ctx_std=1.0)
    p = G.make_stack_inputs(cfg, seed=T + Tc)
    r = rng(C + Tc)
    if bias:
        for n in ("q2", "k2", "v2"):
            p["blocks"][0][n]["b"] = G.bf16_round((0.1 * r.standard_normal(C)).astype(np.float32))
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    with B.dry_run() as names:
        B.spatial_transformer_fwd(x, ctx, sp, cfg.heads)
    assert names.count("attention of the chain") == 1
    ws = torch.full((B.spatial_transformer_workspace_bytes(Bn, T, C, Tc, cfg.Dc, sp.r_max),), 0xFF, dtype=torch.uint8, device="cuda")   # (what no launch wrote is NaN)
    y = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws).clone()
    some = slice(0, 4)
    q = dict(p, x=p["x"][some], ctx=p["ctx"][some])
    ref = O.spatial_transformer(q["x"], q["ctx"], p, cfg.heads)
    got = host(y)[some]
    assert rel_err(got, ref) <= BF16_TOL
    assert rel_err(got - q["x"], ref - q["x"]) <= 2 * BF16_TOL
    assert torch.equal(B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws), y)
    # and the samples that the oracle was not asked for, by themselves
    last = B.spatial_transformer_fwd(x[-1:].repeat(Bn, 1, 1), ctx[-1:].repeat(Bn, 1, 1), sp, cfg.heads)
    assert torch.equal(last[0], y[-1]) and torch.equal(last[-1], y[-1])


# scores beside which any finite mask is lost in rounding (6e37), equal for all text tokens: keys that are no tokens must not count.  The keys' scale
# applied ahead, or to the scores (keys with a bias)
@pytest.mark.parametrize("Tc", [1, 9])
@pytest.mark.parametrize("bias", [False, True])
def test_stack_chain_large_scores(B, Tc, bias):
    Bn, T, C = 39, 32, 320
    cfg = small_cfg(Bn=Bn, T=T, Tc=Tc, C=C, heads=C // 64, r=0, depth=1, w_std=0.03, ctx_std=1.0)
    p = G.make_stack_inputs(cfg, seed=Tc)
    q2, k2 = p["blocks"][0]["q2"], p["blocks"][0]["k2"]
    q2["W"][:] = 0
    q2["b"] = G.bf16_round(np.full(C, 1e18, np.float32))
    k2["W"][:] = 0
    if bias:
        k2["b"] = q2["b"].copy()
    else:
        k2["W"][:, 0] = G.bf16_round(np.full(C, 5e18, np.float32))
        p["ctx"][:, :, 0] = 1
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    with B.dry_run() as names:
        B.spatial_transformer_fwd(x, ctx, sp, cfg.heads)
    assert "attention of the chain" in names
    got = host(B.spatial_transformer_fwd(x, ctx, sp, cfg.heads))[:4]
    ref = O.spatial_transformer(p["x"][:4], p["ctx"][:4], p, cfg.heads)
    assert rel_err(got - p["x"][:4], ref - p["x"][:4]) <= 2 * BF16_TOL


def test_stack_with_biased_q_k_v(B):
    """SDXL's q, k, v carry no bias, but a projection record may: the stack takes them too (the
    text keys / values projected ahead inside the self-attention launches included)."""
    cfg = small_cfg(T=200, depth=2)
    p = G.make_stack_inputs(cfg, seed=4)
    r = rng(40)
    for blk in p["blocks"]:
        for name in ("q1", "k1", "v1", "q2", "k2", "v2"):
            blk[name] = dict(blk[name], b=G.bf16_round((0.5 * r.standard_normal(blk[name]["W"].shape[0])).astype(np.float32)))
    got = host(B.spatial_transformer_fwd(dev(p["x"], B), dev(p["ctx"], B), B.StackParams(p), cfg.heads))
    ref = O.spatial_transformer(p["x"], p["ctx"], p, cfg.heads)
    assert rel_err(got - p["x"], ref - p["x"]) <= 2 * BF16_TOL
    # without the value biases the oracle's result is far away
    for blk in p["blocks"]:
        blk["v1"] = dict(blk["v1"], b=None)
        blk["v2"] = dict(blk["v2"], b=None)
    e = rel_err(O.spatial_transformer(p["x"], p["ctx"], p, cfg.heads) - p["x"], ref - p["x"])
    assert e > 6 * BF16_TOL, e


def test_stack_tiny_config(B):
    # configs[0]: batch 2, 16x16 latent, C = 320, rank 8 on the attention projections
    p, got = run_stack(B, G.TINY, seed=0)
    ref = O.spatial_transformer(p["x"], p["ctx"], p, G.TINY.heads)
    assert rel_err(got, ref) <= BF16_TOL
    # batch independence (Section 3.3): sample b alone gives the same bits
    import torch
    sp = B.StackParams(p)
    for b in range(2):
        yb = B.spatial_transformer_fwd(dev(p["x"][b:b + 1], B), dev(p["ctx"][b:b + 1], B), sp, G.TINY.heads)
        assert rel_err(host(yb), ref[b:b + 1]) <= BF16_TOL
    # run-to-run determinism
    y1 = B.spatial_transformer_fwd(dev(p["x"], B), dev(p["ctx"], B), sp, G.TINY.heads)
    y2 = B.spatial_transformer_fwd(dev(p["x"], B), dev(p["ctx"], B), sp, G.TINY.heads)
    assert torch.equal(y1, y2)


# --------------------------------------------------------------- multi_lora_linear_fwd
def test_multi_lora_small(B):
    cfg = G.MultiLoraConfig(name="s", requests=5, T=150, C=128, ranks=(8, 16, 32), request_adapter=(2, 0, 1, 0, 2), std=0.08, x_std=1.0)
    p = G.make_multi_lora_inputs(cfg, seed=2, n_proj=1, bias=True)
    pr = p["projs"][0]
    offs = [0, 150, 150, 290, 450, 601, 750]           # ragged, one empty segment
    adp = [2, 1, 0, -1, 1, 2]
    ref = O.multi_lora_linear(p["x"], pr["W"], pr["b"], pr["A"], pr["B"], [0.5, 1.0, 2.0], offs, adp)
    y = B.multi_lora_linear_fwd(dev(p["x"], B), dev(pr["W"], B), dev(pr["b"], B), [dev(a, B) for a in pr["A"]],
                                [dev(b, B) for b in pr["B"]], [0.5, 1.0, 2.0], offs, adp)
    assert rel_err(host(y), ref) <= BF16_TOL
    wrong = O.multi_lora_linear(p["x"], pr["W"], pr["b"], pr["A"], pr["B"], [0.5, 1.0, 2.0], offs, [0, 1, 0, -1, 1, 2])
    assert rel_err(wrong, ref) > 3 * BF16_TOL


# several problems of one launch on more than one round of 128x128 tiles: whole and partial k-steps of
# the adapters, segments without one, column and row remainders, flags of several column tiles of producers
@pytest.mark.parametrize("lengths,ranks,kernel", [([3001, 900, 2690], [64, 128, 64], "records"), ([2999, 129, 3500], [8, 72, 0], "guard records"),
                                                  ([130, 6400, 60], [200, 64, 16], "guard flags"), ([3300, 3300], [0, 0], "")])
def test_multi_lora_many_tiles(B, lengths, ranks, kernel):
    r = rng(sum(lengths))
    K, N, M = 64, 1284, sum(lengths)
    draw = lambda *shape, s: G.bf16_round((s * r.standard_normal(shape)).astype(np.float32))
    x, W, bias = draw(M, K, s=1.0), draw(N, K, s=0.1), draw(N, s=0.5)
    A, Bm = [draw(k, K, s=0.3) for k in ranks if k], [draw(N, k, s=0.1) for k in ranks if k]
    offsets = [sum(lengths[:i]) for i in range(len(lengths) + 1)]
    have = [k > 0 for k in ranks]
    adapters = [sum(have[:i]) if h else -1 for i, h in enumerate(have)]
    args = (dev(x, B), dev(W, B), dev(bias, B), [dev(a, B) for a in A], [dev(b, B) for b in Bm], [0.5] * len(A), offsets, adapters)
    with B.dry_run() as names:
        B.multi_lora_linear_fwd(*args)
    assert names[-1] == ("gemm 128x128/4 waves/2 stages " + kernel).strip()
    ref = O.multi_lora_linear(x, W, bias, A, Bm, [0.5] * len(A), offsets, adapters)
    assert rel_err(host(B.multi_lora_linear_fwd(*args)), ref) <= BF16_TOL
    if A:
        assert rel_err(O.linear(x, W, bias), ref) > 3 * BF16_TOL


# ------------------------------------------------------------- lora_patch / lora_unpatch
def patch_roundtrip(B, mats):
    import torch
    dm = []
    for m in mats:
        W = torch.from_numpy(m["W"]).cuda()
        dm.append((W, torch.from_numpy(m["A"]).cuda(), torch.from_numpy(m["B"]).cuda(), torch.zeros_like(W), m["scale"]))
    plan = B.PatchPlan(dm)
    B.lora_patch(plan)
    patched = [t[0].cpu().numpy().copy() for t in dm]
    B.lora_unpatch(plan)
    restored = [t[0].cpu().numpy() for t in dm]
    return patched, restored


# dependency records that the launch finds as it may: all ones, what another call left, what the launch's own replay left.  One and two
# column tiles of producers, several launches' worth of segments, row blocks that are not full
@pytest.mark.parametrize("lengths,ranks", [((4096, 2100, 2990), (16, 128, 72)), ((700,) * 12, (64, 8, 128, 24) * 3), ((9000,), (64,))])
def test_multi_lora_workspace_contents_do_not_matter(B, lengths, ranks):
    import torch
    r = rng(sum(lengths))
    K, N, M = 128, 640, sum(lengths)
    W = G.bf16_round((0.05 * r.standard_normal((N, K))).astype(np.float32))
    offsets = [sum(lengths[:i]) for i in range(len(lengths) + 1)]
    ws = torch.full((B.lib().sd_multi_lora_linear_workspace_bytes(M, max(ranks)),), 255, dtype=torch.uint8, device="cuda")
    x = torch.empty((M, K), dtype=torch.bfloat16, device="cuda")
    A = [torch.empty((k, K), dtype=torch.bfloat16, device="cuda") for k in ranks]
    Bm = [torch.empty((N, k), dtype=torch.bfloat16, device="cuda") for k in ranks]
    out = torch.empty((M, N), dtype=torch.bfloat16, device="cuda")

    def draw():
        arrays = [G.bf16_round((s * r.standard_normal(t.shape)).astype(np.float32)) for t, s in [(x, 1.0)] + [(t, 0.3) for t in A] + [(t, 0.1) for t in Bm]]
        for t, a in zip([x] + A + Bm, arrays):
            t.copy_(dev(a, B))
        return arrays[0], arrays[1:1 + len(ranks)], arrays[1 + len(ranks):]

    def call():
        B.multi_lora_linear_fwd(x, dev_W, None, A, Bm, [0.5] * len(ranks), offsets, list(range(len(ranks))), out=out, ws=ws)

    def check(arrays):
        xs, As, Bs = arrays
        got = host(out)
        for i, (a, b) in enumerate(zip(As, Bs)):
            rows = slice(offsets[i], offsets[i + 1])
            ref = O.lora_linear(xs[rows], W, None, a, b, 0.5)
            assert rel_err(got[rows], ref) <= BF16_TOL
            assert rel_err(O.linear(xs[rows], W, None), ref) > 3 * BF16_TOL     # a stale or missing adapter term would be seen

    dev_W = dev(W, B)
    arrays = draw()
    call()
    check(arrays)
    arrays = draw()
    call()
    check(arrays)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        call()
    for _ in range(3):
        arrays = draw()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        check(arrays)
    assert B.gemm_dep_timeouts() == 0


def test_patch_small_ragged_and_roundtrip(B):
    groups = ((2, 300, 200), (1, 128, 128), (1, 33, 1027), (3, 640, 640), (1, 1, 4))
    mats = G.make_patch_inputs(groups, r=32, alpha=16.0, seed=5)
    mats += G.make_patch_inputs(((1, 70, 72),), r=5, alpha=5.0, seed=6)       # odd rank
    patched, restored = patch_roundtrip(B, mats)
    for m, Wp, Wr in zip(mats, patched, restored):
        ref, _ = O.lora_patch(m["W"], m["A"], m["B"], m["scale"])
        assert rel_err(Wp, ref) <= PATCH_TOL
        assert not np.array_equal(Wp, m["W"])
        assert Wr.tobytes() == m["W"].tobytes()                                  # bit-exact
        # the arithmetic inverse would not have restored the bits
    sub = O.lora_unpatch_by_subtraction(patched[3], mats[3]["A"], mats[3]["B"], mats[3]["scale"])
    assert sub.tobytes() != mats[3]["W"].tobytes()


# one, two, three and more chunks of 16 ranks, chunks that are partly past the rank; tiles of 64 x 256 with rows, columns or
# whole wavefronts outside the matrix
@pytest.mark.parametrize("out,in_", [(64, 256), (65, 260), (31, 132), (128, 508)])
@pytest.mark.parametrize("ranks", [(4,), (12,), (16,), (20,), (36,), (64,), (128,), (4, 52), (64, 16), (48, 8, 32)])
def test_patch_rank_chunks(B, out, in_, ranks):
    import torch
    r = rng(out + in_ + sum(ranks))
    W = (0.02 * r.standard_normal((out, in_))).astype(np.float32)
    ads = [((0.02 * r.standard_normal((rk, in_))).astype(np.float32), (0.02 * r.standard_normal((out, rk))).astype(np.float32), sc)
           for rk, sc in zip(ranks, (1.0, 0.5, -2.0))]
    ref = O.lora_patch_multi(W, ads)[0]
    d = [(torch.from_numpy(A).cuda(), torch.from_numpy(Bm).cuda(), sc) for A, Bm, sc in ads]
    Wm, Ws = torch.from_numpy(W).cuda(), torch.from_numpy(W).cuda()
    undo = torch.empty_like(Wm)
    plan = B.PatchMultiPlan([(Wm, undo, torch.empty(Wm.shape, dtype=torch.bfloat16, device="cuda"), d)])
    B.lora_patch_multi(plan)
    for A, Bm, sc in d:
        B.lora_patch(B.PatchPlan([(Ws, A, Bm, torch.empty_like(Ws), sc)]))
    assert rel_err(Wm.cpu().numpy(), ref) <= PATCH_TOL
    assert torch.equal(Wm, Ws) and undo.cpu().numpy().tobytes() == W.tobytes()
    B.lora_unpatch_multi(plan)
    assert Wm.cpu().numpy().tobytes() == W.tobytes()


def patch_pair(B, W, ads, serving=True):
    """The adapters in one multi pass and one after the other in single passes: (multi, single, undo, serving, plan)."""
    import torch
    d = [(torch.from_numpy(A).cuda(), torch.from_numpy(Bm).cuda(), sc) for A, Bm, sc in ads]
    Wm, Ws = torch.from_numpy(W).cuda(), torch.from_numpy(W).cuda()
    undo, S = torch.empty_like(Wm), torch.empty(Wm.shape, dtype=torch.bfloat16, device="cuda")
    plan = B.PatchMultiPlan([(Wm, undo, S, d)])
    B.lora_patch_multi(plan)
    for A, Bm, sc in d:
        B.lora_patch(B.PatchPlan([(Ws, A, Bm, torch.empty_like(Ws), sc)]))
    return Wm, Ws, undo, S, plan


# ranks that are no multiple of 4 (B rows at any 4-byte address), next to ones that are; rows of W that are 16-byte aligned and
# rows that are not; tiles inside the matrix, ragged ones, an odd number of 32-row tiles
@pytest.mark.parametrize("out,in_", [(64, 256), (96, 516), (65, 254), (33, 1027), (130, 1278)])
@pytest.mark.parametrize("ranks", [(1,), (6,), (33,), (7, 30), (64, 3), (5, 16, 2, 17)])
def test_patch_any_rank_any_row_length(B, out, in_, ranks):
    import torch
    r = rng(out * in_ + sum(ranks))
    W = (0.02 * r.standard_normal((out, in_))).astype(np.float32)
    ads = [((0.02 * r.standard_normal((rk, in_))).astype(np.float32), (0.02 * r.standard_normal((out, rk))).astype(np.float32), sc)
           for rk, sc in zip(ranks, (1.0, 0.5, -2.0, 3.0))]
    ref = O.lora_patch_multi(W, ads)[0]
    Wm, Ws, undo, S, plan = patch_pair(B, W, ads)
    assert rel_err(Wm.cpu().numpy(), ref) <= PATCH_TOL
    assert rel_err(W, ref) > 10 * PATCH_TOL
    assert torch.equal(Wm, Ws) and torch.equal(S, Wm.to(torch.bfloat16)) and undo.cpu().numpy().tobytes() == W.tobytes()
    B.lora_unpatch_multi(plan)
    assert Wm.cpu().numpy().tobytes() == W.tobytes()


# the number of tiles decides how a pass is cut into workgroups (up to 512, up to 768, more): each cut under ranks of half a
# chunk, one, several, and a B at 4-byte addresses; matrices with an odd and an even number of 32-row tiles, columns off the tile
@pytest.mark.parametrize("tiles", [500, 760, 1000])
@pytest.mark.parametrize("ranks", [(8,), (20,), (64,), (33,), (8, 40), (32, 8, 7)])
def test_patch_every_cut_into_workgroups(B, tiles, ranks):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(tiles + sum(ranks))
    normal = lambda *shape: torch.empty(shape, device="cuda").normal_(0.0, 0.02, generator=g)
    mats, left = [], tiles
    for out, in_ in [(96, 516), (64, 256), (33, 1024), (70, 260), (96, 1030)] * 100:
        left -= ((out + 31) // 32) * ((in_ + 255) // 256)
        if left < 0:
            break
        mats.append((normal(out, in_), [(normal(rk, in_), normal(out, rk), sc) for rk, sc in zip(ranks, (1.0, -0.5, 2.0))]))
    first = [W.clone() for W, _ in mats]
    undo = [torch.zeros_like(W) for W, _ in mats]
    S = [torch.zeros(W.shape, dtype=torch.bfloat16, device="cuda") for W, _ in mats]
    plan = B.PatchMultiPlan([(W, u, s, ads) for (W, ads), u, s in zip(mats, undo, S)])
    assert tiles - 20 < plan.total_tiles <= tiles
    B.lora_patch_multi(plan)
    single = [W.clone() for W in first]
    for a in range(len(ranks)):
        B.lora_patch(B.PatchPlan([(W, *ads[a][:2], torch.empty_like(W), ads[a][2]) for W, (_, ads) in zip(single, mats)]))
    for (W, ads), W0, Ws, u, s in zip(mats, first, single, undo, S):
        ref = W0.double()
        for A, Bm, sc in ads:
            ref += sc * (Bm.double() @ A.double())
        assert float((W.double() - ref).abs().max() / ref.abs().max()) <= PATCH_TOL
        assert float((W0.double() - ref).abs().max() / ref.abs().max()) > 10 * PATCH_TOL
        assert torch.equal(W, Ws) and torch.equal(u, W0) and torch.equal(s, W.to(torch.bfloat16))
    B.lora_unpatch_multi(plan)
    for (W, _), W0, s in zip(mats, first, S):
        assert torch.equal(W, W0) and torch.equal(s, W0.to(torch.bfloat16))


def test_patch_matrix_of_more_than_2_to_the_30_elements(B):
    """Byte offsets past 2^32: the first, middle and last rows against float64 sums."""
    import torch
    out, in_, r = 8200, 131076, 6
    assert out * in_ > 2 ** 30
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    normal = lambda *shape: torch.empty(shape, device="cuda").normal_(0.0, 0.02, generator=g)
    W, A, Bm = normal(out, in_), normal(r, in_), normal(out, r)
    undo = torch.empty_like(W)
    rows = torch.tensor([0, 1, 31, 32, 63, 64, 4095, 4096, 8160, 8191, 8192, 8199], device="cuda")
    before, first_sum = W[rows].clone(), W.double().sum()
    plan = B.PatchPlan([(W, A, Bm, undo, 0.5)])
    B.lora_patch(plan)
    ref = before.double() + 0.5 * (Bm[rows].double() @ A.double())
    assert float((W[rows].double() - ref).abs().max() / ref.abs().max()) <= PATCH_TOL
    assert float((before.double() - ref).abs().max() / ref.abs().max()) > 10 * PATCH_TOL
    assert torch.equal(undo[rows], before) and bool(undo.double().sum() == first_sum)
    B.lora_unpatch(plan)
    assert torch.equal(W, undo)


def test_patch_exact_integers(B):
    r = rng(9)
    W = r.integers(-8, 9, (256, 384)).astype(np.float32)
    A = r.integers(-3, 4, (32, 384)).astype(np.float32)
    Bm = r.integers(-3, 4, (256, 32)).astype(np.float32)
    patched, restored = patch_roundtrip(B, [{"W": W, "A": A, "B": Bm, "scale": 2.0}])
    ref, _ = O.lora_patch(W, A, Bm, 2.0)
    assert np.array_equal(patched[0], ref)           # exactly representable -> identical bits
    assert np.array_equal(restored[0], W)


def test_patch_several_adapters_one_pass(B):
    """Two and three adapters per matrix in one pass: the oracle's successive-patch chain, the
    bits of successive single-adapter launches, the bf16 serving copy, and the exact restore."""
    import torch
    # (rank 32 throughout on tiles that lie inside the matrix takes a pipelined path of its own for
    # one and for two adapters: 96 x 512 and 300 x 200 / 160 x 768 reach it)
    shapes = ((300, 200), (128, 128), (33, 1027), (640, 640), (64, 256), (96, 512), (160, 768))
    ranks = ((32, 32), (32, 8, 5), (32,), (16, 32), (32, 32, 32, 32), (32,), (32, 32))
    r = rng(21)
    host, devm, single = [], [], []
    for (o, i), rks in zip(shapes, ranks):
        W = (0.02 * r.standard_normal((o, i))).astype(np.float32)
        ads = [((0.02 * r.standard_normal((rk, i))).astype(np.float32), (0.02 * r.standard_normal((o, rk))).astype(np.float32), sc)
               for rk, sc in zip(rks, (1.0, 0.5, 2.0, -1.0))]
        host.append((W, ads))
        Wd = torch.from_numpy(W).cuda()
        devm.append((Wd, torch.empty_like(Wd), torch.empty(Wd.shape, dtype=torch.bfloat16, device="cuda"),
                     [(torch.from_numpy(A).cuda(), torch.from_numpy(Bm).cuda(), sc) for A, Bm, sc in ads]))
    plan = B.PatchMultiPlan(devm)
    B.lora_patch_multi(plan)
    torch.cuda.synchronize()
    for (W, ads), (Wd, undo, serving, dads) in zip(host, devm):
        ref, ref_undo, ref_serving = O.lora_patch_multi(W, ads, serving=True)
        got = Wd.cpu().numpy()
        assert rel_err(got, ref) <= PATCH_TOL
        assert undo.cpu().numpy().tobytes() == W.tobytes()
        # the serving copy is the rounding of what the GPU itself stored, bit for bit
        assert serving.float().cpu().numpy().tobytes() == O.bf16_rne(got).tobytes()
        assert rel_err(serving.float().cpu().numpy(), ref_serving) <= 2.0 ** -7
        # dropping the last adapter is visible at this tolerance (the check is not vacuous)
        if len(ads) > 1:
            assert rel_err(O.lora_patch_multi(W, ads[:-1])[0], ref) > 100 * PATCH_TOL
        # successive single-adapter launches on a fresh copy give the same bits
        Ws = torch.from_numpy(W).cuda()
        for A, Bm, sc in dads:
            one = B.PatchPlan([(Ws, A, Bm, torch.empty_like(Ws), sc)])
            B.lora_patch(one)
        torch.cuda.synchronize()
        assert Ws.cpu().numpy().tobytes() == got.tobytes()
    B.lora_unpatch_multi(plan)
    torch.cuda.synchronize()
    for (W, ads), (Wd, undo, serving, dads) in zip(host, devm):
        assert Wd.cpu().numpy().tobytes() == W.tobytes()
        assert serving.float().cpu().numpy().tobytes() == O.bf16_rne(W).tobytes()


def test_cfg_combine_bit_exact(B):
    import torch
    r = rng(31)
    for n, g in ((1, 7.5), (7, 1.0), (4096, 7.5), (2 * 4 * 128 * 128 + 3, 5.0), (65536, 0.0)):
        eu = G.bf16_round(r.standard_normal(n).astype(np.float32))
        ec = G.bf16_round(r.standard_normal(n).astype(np.float32))
        got = B.cfg_combine(dev(eu, B), dev(ec, B), g)
        assert host(got).tobytes() == O.cfg_combine(eu, ec, g).tobytes()
    # batch-of-two layout: the two halves of one buffer, unaligned second half, in place
    n = 1001
    x = G.bf16_round(r.standard_normal(2 * n).astype(np.float32))
    xd = dev(x, B)
    out = B.cfg_combine(xd[:n], xd[n:], 3.0, out=xd[:n])
    assert host(out).tobytes() == O.cfg_combine(x[:n], x[n:], 3.0).tobytes()


def test_controlnet_residual_add_bit_exact(B):
    """Section 2, "ControlNet": the summed ControlNet outputs added to a skip-connection tensor."""
    import torch
    r = rng(37)
    for n, nres in ((1, 1), (7, 3), (4096, 2), (2 * 320 * 64 * 64 + 5, 3), (65536, 8), (2049, 0)):
        h = G.bf16_round(r.standard_normal(n).astype(np.float32))
        rs = [G.bf16_round(r.standard_normal(n).astype(np.float32)) for _ in range(nres)]
        got = B.controlnet_residual_add(dev(h, B), [dev(x, B) for x in rs])
        assert host(got).tobytes() == O.controlnet_residual_add(h, rs).tobytes(), (n, nres)
    # in place on the backbone tensor, residuals at unaligned offsets of one buffer
    n = 1001
    x = G.bf16_round(r.standard_normal(3 * n).astype(np.float32))
    xd = dev(x, B)
    out = B.controlnet_residual_add(xd[:n], [xd[n:2 * n], xd[2 * n:]], out=xd[:n])
    assert host(out).tobytes() == O.controlnet_residual_add(x[:n], [x[n:2 * n], x[2 * n:]]).tobytes()
    # more ControlNets than the entry point takes
    with pytest.raises(B.SwiftDiffError):
        B.controlnet_residual_add(xd[:n], [xd[n:2 * n]] * 9)


def test_empty_inputs_are_no_ops(B):
    """Zero rows, zero tokens, zero samples: every forward call returns without touching its
    outputs (which are empty) and without an error; a later ordinary call still works."""
    import torch
    r = rng(7)
    p = B.Proj.from_numpy(mkproj(r, 64, 32, 8, bias=True, scale=1.0))
    e = torch.empty((0, 32), dtype=torch.bfloat16, device="cuda")
    assert B.lora_linear_fwd(e, p).shape == (0, 64)
    g = torch.ones(32, dtype=torch.bfloat16, device="cuda")
    assert B.lora_linear_fwd(e, p, ln_gamma=g, ln_beta=g).shape == (0, 64)
    C_, heads = 128, 2
    pq, pk, pv, po = (B.Proj.from_numpy(mkproj(r, C_, C_, 8, bias=False, scale=1.0)) for _ in range(4))
    gc = torch.ones(C_, dtype=torch.bfloat16, device="cuda")
    for shape in ((0, 64, C_), (2, 0, C_)):
        xe = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
        assert B.attn_block_fwd(xe, None, gc, gc, pq, pk, pv, po, heads).shape == shape
        assert B.groupnorm_fwd(xe, gc, gc, 32).shape == shape
    qe = torch.empty((2, 0, C_), dtype=torch.bfloat16, device="cuda")      # no queries against eight keys
    k8 = torch.zeros((2, 8, C_), dtype=torch.bfloat16, device="cuda")
    assert B.attention_fwd(qe, k8, torch.zeros((C_, 16), dtype=torch.bfloat16, device="cuda"), heads).shape == (2, 0, C_)
    f1 = B.Proj.from_numpy(mkproj(r, 2 * 4 * C_, C_, 8, bias=True, scale=1.0))
    f2 = B.Proj.from_numpy(mkproj(r, C_, 4 * C_, 8, bias=True, scale=1.0))
    xe = torch.empty((0, C_), dtype=torch.bfloat16, device="cuda")
    assert B.ff_block_fwd(xe, gc, gc, f1, f2).shape == (0, C_)
    W = torch.zeros((64, 32), dtype=torch.bfloat16, device="cuda")
    A = torch.zeros((8, 32), dtype=torch.bfloat16, device="cuda")
    Bm = torch.zeros((64, 8), dtype=torch.bfloat16, device="cuda")
    assert B.multi_lora_linear_fwd(e, W, None, [A], [Bm], [1.0], [0], [], out=None).shape == (0, 64)
    torch.cuda.synchronize()
    # and the library is in working order afterwards
    x = G.bf16_round(r.standard_normal((40, 32)).astype(np.float32))
    pn = mkproj(r, 64, 32, 8, bias=True, scale=1.0)
    ref = O.lora_linear(x, pn["W"], pn["b"], pn["A"], pn["B"], pn["scale"])
    assert rel_err(host(B.lora_linear_fwd(dev(x, B), B.Proj.from_numpy(pn))), ref) <= BF16_TOL


def test_ceiling_copies_copy(B):
    """The streaming-ceiling kernels of the benchmark are plain copies: every byte arrives, sizes
    that are not a multiple of the grid's stride included."""
    import torch
    for n in (4, 1028, 128 * 4 * 131072 + 4 * 77):
        src = torch.arange(n, device="cuda", dtype=torch.float32)
        d0, d1, d2 = (torch.full((n,), -1.0, device="cuda") for _ in range(3))
        B.ceiling_copy_f32(src, d0)
        B.ceiling_copy_1r2w_f32(src, d1, d2)
        assert torch.equal(d0, src) and torch.equal(d1, src) and torch.equal(d2, src), n


def test_ceiling_valu_loop_runs_and_counts(B):
    """The vector-ALU ceiling loop: instruction counts as documented, and a finite result in every
    lane (2^-|a| chains stay in (0, 1], the FMA chains converge to 1)."""
    import torch
    out = torch.full((8 * 256,), float("nan"), device="cuda")
    for mode, (e, f) in enumerate(((1, 0), (0, 4), (1, 4), (2, 0))):
        exps, fmas = B.ceiling_valu(out, 8, 100, mode)
        assert exps == e * 8 * 4 * 100 * 8 and fmas == f * 8 * 4 * 100 * 8
        torch.cuda.synchronize()
        assert bool(torch.isfinite(out).all())
    with pytest.raises(Exception):
        B.ceiling_valu(out, 8, 100, 4)


def test_bal_orders_the_patch_inside_a_denoising_loop(B):
    """The serving loop of Section 4.2 in miniature: a projection reads the bf16 serving copy of an
    fp32 master weight; two adapters load in the background (gated so that they arrive during
    step 3 of 8); the loop early-starts unpatched, patches when the scheduler says so, and patches
    off after the request.  Steps before the order equal the base projection, steps after it the
    patched one, and the master weight ends with its original bits."""
    import threading
    import torch
    r = rng(41)
    M, K, N, k_bound, n_steps = 192, 256, 320, 6, 8
    W = (0.05 * r.standard_normal((N, K))).astype(np.float32)
    ads_h = [((0.3 * r.standard_normal((rk, K))).astype(np.float32), (0.05 * r.standard_normal((N, rk))).astype(np.float32), sc)
             for rk, sc in ((32, 1.0), (16, 0.5))]
    x = G.bf16_round(r.standard_normal((M, K)).astype(np.float32))
    Wd = torch.from_numpy(W).cuda()
    undo = torch.empty_like(Wd)
    serving = Wd.to(torch.bfloat16)
    stage = [(torch.empty(A.shape, dtype=torch.float32).pin_memory(), torch.empty(Bm.shape, dtype=torch.float32).pin_memory()) for A, Bm, _ in ads_h]
    dev_ads = [(torch.empty(A.shape, dtype=torch.float32, device="cuda"), torch.empty(Bm.shape, dtype=torch.float32, device="cuda"), sc) for A, Bm, sc in ads_h]
    plan = B.PatchMultiPlan([(Wd, undo, serving, dev_ads)])
    gate = threading.Event()

    def load(i):                      # loader thread: "disk" -> pinned host memory
        if not gate.wait(10.0):
            return 1
        stage[i][0].copy_(torch.from_numpy(ads_h[i][0]))
        stage[i][1].copy_(torch.from_numpy(ads_h[i][1]))
        return 0

    bal = B.Bal(len(ads_h), load)
    bal.start()
    xd = dev(x, B)
    outs, ordered = [], None
    for step in range(1, n_steps + 1):
        if step == 4:                 # the adapters arrived during step 3
            gate.set()
            t0 = time.time()
            while not bal.loaded():
                assert time.time() - t0 < 5.0
                time.sleep(0.001)
        if bal.before_step(step, k_bound):
            ordered = step
            for (hA, hB), (dA, dB, _) in zip(stage, dev_ads):
                dA.copy_(hA, non_blocking=True)
                dB.copy_(hB, non_blocking=True)
            B.lora_patch_multi(plan)
        outs.append(host(B.lora_linear_fwd(xd, B.Proj(serving))))
    assert ordered == 4 and bal.stats()["stall_s"] == 0.0
    base = O.linear(x, O.bf16_rne(W), None)
    Wp, _, Wserv = O.lora_patch_multi(W, ads_h, serving=True)
    patched = O.linear(x, Wserv, None)
    assert rel_err(patched, base) > 10 * BF16_TOL            # the adapters matter at this tolerance
    for step, y in enumerate(outs, start=1):
        assert rel_err(y, base if step < ordered else patched) <= BF16_TOL
    assert rel_err(Wd.cpu().numpy(), Wp) <= PATCH_TOL
    assert bal.finish() is True
    B.lora_unpatch_multi(plan)
    torch.cuda.synchronize()
    assert Wd.cpu().numpy().tobytes() == W.tobytes()
    assert rel_err(host(B.lora_linear_fwd(xd, B.Proj(serving))), base) <= BF16_TOL
    bal.close()


# ------------------------------------------------------------------ HIP graph replay
def test_stack_graph_replay_matches_eager(B):
    """The stack call only enqueues kernels, so it can be captured into a HIP graph.  Every
    replay, with eager work and synchronisations in between, must give the eager bits."""
    import torch
    cfg = small_cfg(T=200, depth=1)
    p = G.make_stack_inputs(cfg, seed=2)
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    ws = torch.empty(B.spatial_transformer_workspace_bytes(cfg.Bn, cfg.T, cfg.C, cfg.Tc, cfg.Dc, sp.r_max), dtype=torch.uint8, device="cuda")
    y_eager = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws).clone()
    y = torch.empty_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, out=y, ws=ws)
    for i in range(4):
        y.zero_()
        ws.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, y_eager), f"replay {i} differs from the eager result"
        # eager work between replays
        again = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads, ws=ws)
        assert torch.equal(again, y_eager)


def test_projections_as_one_launch_or_two_give_the_same_bits(B):
    """A projection runs as one launch (base-GEMM tiles wait for the down-projection tiles of the
    same grid) or, with the diagnostic switch off, as two; the arithmetic is the same, so the
    whole stack and a many-segment multi-LoRA batch must agree bit for bit."""
    import torch
    cfg = small_cfg(T=200, depth=2)
    p = G.make_stack_inputs(cfg, seed=5)
    sp = B.StackParams(p)
    x, ctx = dev(p["x"], B), dev(p["ctx"], B)
    # 20 segments of 3 adapters: more projections than one launch's group holds
    mcfg = G.MultiLoraConfig(name="m", requests=20, T=70, C=128, ranks=(8, 16, 32), request_adapter=tuple(i % 3 for i in range(20)),
                             std=0.08, x_std=1.0)
    mp = G.make_multi_lora_inputs(mcfg, seed=3, n_proj=1, bias=True)
    pr = mp["projs"][0]
    offs = [70 * i for i in range(21)]
    adp = [(-1 if i % 7 == 6 else i % 3) for i in range(20)]
    margs = (dev(mp["x"], B), dev(pr["W"], B), dev(pr["b"], B), [dev(a, B) for a in pr["A"]], [dev(b, B) for b in pr["B"]],
             [0.5, 1.0, 2.0], offs, adp)
    mref = O.multi_lora_linear(mp["x"], pr["W"], pr["b"], pr["A"], pr["B"], [0.5, 1.0, 2.0], offs, adp)
    outs = {}
    try:
        for on in (False, True):
            B.set_projection_fusion(on)
            y = B.spatial_transformer_fwd(x, ctx, sp, cfg.heads)
            my = B.multi_lora_linear_fwd(*margs)
            torch.cuda.synchronize()
            outs[on] = (y.clone(), my.clone())
    finally:
        B.set_projection_fusion(True)
    assert torch.equal(outs[False][0], outs[True][0])
    assert torch.equal(outs[False][1], outs[True][1])
    assert rel_err(host(outs[True][1]), mref) <= BF16_TOL
    assert B.gemm_dep_timeouts() == 0


def test_zz_no_tile_gave_up_waiting(B):
    """Runs last in this file: across everything above, no base-GEMM tile ran out of spins
    while waiting for a down-projection tile of its own launch."""
    assert B.gemm_dep_timeouts() == 0


@pytest.mark.parametrize("boost", [1.0, 4.0])
def test_attn_block_scores_that_climb_from_key_tile_to_key_tile(B, boost):
    """Inside the block the attention kernel first tries without measuring the maximum of the
    key tiles between a segment's first and last: the exponentials are formed against the first
    tile's maximum, which is exact as long as nothing overflows, and a workgroup whose row sums
    or accumulators end up non-finite runs again in the measured form.  Cross-attention with keys
    under the caller's control (W_k picks the context's leading channels): the scores of
    successive 64-key tiles step up, fall back, stay level and step up again.  boost = 1: the
    steps (up to 2^68 above the first tile) stay in range, the first attempt stands.  boost = 4:
    they reach 2^270, the first attempt overflows and the measured form must take over.  Half of
    the queries see the mirrored, falling sequence, so both kinds share wavefronts.  Ragged last
    tile."""
    import torch
    Bn, T, Tc, C, Dc = 2, 200, 64 * 6 + 23, 64, 64
    r = rng(4242)
    n0 = r.standard_normal(C).astype(np.float32)
    n0 = (n0 - n0.mean()) / n0.std()                       # what LayerNorm makes of a row along n0
    sign = np.where(r.random((Bn, T, 1)) < 0.5, 1.0, -1.0).astype(np.float32)
    h = (sign * n0 * (1.0 + 0.05 * r.standard_normal((Bn, T, 1))) + 0.15 * r.standard_normal((Bn, T, C))).astype(np.float32)
    # natural-log score of key j for a query along +n0: level[j // 64] (+ noise); the head-room is 8 in log2 = 5.5
    level = boost * np.array([0.0, 14.0, 3.0, 3.5, 30.0, 29.0, 47.0], np.float32)
    a = level[np.arange(Tc) // 64] + 0.5 * r.standard_normal(Tc).astype(np.float32)
    ctx = np.zeros((Bn, Tc, Dc), np.float32)
    ctx[:, :, :C] = (a[None, :, None] * n0[None, None, :] / C * 8.0)
    ctx += 0.05 * r.standard_normal(ctx.shape).astype(np.float32)
    ctx = G.bf16_round(ctx)
    eye = np.eye(C, dtype=np.float32)
    mk = lambda W, bias: {"W": G.bf16_round(W), "b": bias, "A": G.bf16_round(0.05 * r.standard_normal((8, W.shape[1])).astype(np.float32)),
                          "B": G.bf16_round(0.02 * r.standard_normal((W.shape[0], 8)).astype(np.float32)), "scale": 0.5}
    pq, pk = mk(eye, None), mk(eye, None)
    pv = mk(0.3 * r.standard_normal((C, Dc)).astype(np.float32), None)
    po = mk(0.3 * r.standard_normal((C, C)).astype(np.float32), G.bf16_round(0.1 * r.standard_normal(C).astype(np.float32)))
    g, b = np.ones(C, np.float32), np.zeros(C, np.float32)
    ref = O.attn_sublayer(h, ctx, g, b, pq, pk, pv, po, 1)
    # the test is what it says: scores (in powers of two) of a +n0 query climb from tile to tile, past 2^100 with the boost
    qn = O.proj(O.layernorm(h, g, b), pq)
    kn = O.proj(ctx, pk)
    i_pos = int(np.argmax(sign[0, :, 0] > 0))
    s_row = (qn[0, i_pos] @ kn[0].T) / 8.0 * 1.4426950408889634
    tile_max = [s_row[i:i + 64].max() for i in range(0, Tc, 64)]
    assert tile_max[1] - tile_max[0] > 8 and tile_max[2] < tile_max[1] and tile_max[4] - tile_max[3] > 8 and tile_max[6] - tile_max[5] > 8
    assert (tile_max[6] - tile_max[0] > 140) == (boost > 1) and tile_max[6] - tile_max[0] < (300 if boost > 1 else 100)
    y = B.attn_block_fwd(torch.from_numpy(h).cuda(), dev(ctx, B), dev(g, B), dev(b, B), B.Proj.from_numpy(pq), B.Proj.from_numpy(pk),
                         B.Proj.from_numpy(pv), B.Proj.from_numpy(po), 1)
    got = host(y)
    assert np.isfinite(got).all()
    assert rel_err(got - h, ref - h) <= BF16_TOL
    # negative control: the output depends on which keys win (attention to the first tile only is far away)
    ref_first = O.attn_sublayer(h, ctx[:, :64], g, b, pq, pk, pv, po, 1)
    assert rel_err(ref_first - h, ref - h) > 10 * BF16_TOL


# Prescaled keys (inside a block) through every kernel that a launch's tile count chooses, with scores that climb to 2^150 above the first tile
# inside each range that keeps a reference of its own (the first attempt overflows, the measured form takes over), and with first tiles of
# those ranges 2^150 below the others (the reference starts there; nothing has been summed up that it could rescale).
# Half of the queries see the mirrored scores, so both kinds share wavefronts.
@pytest.mark.parametrize("where", ["climb", "low"])
@pytest.mark.parametrize("Bn,T,Tc,heads,cut,queries,groups", [
    (2, 200, 64 * 6 + 23, 1, False, 128, 1), (2, 200, 64 * 7 + 23, 2, False, 128, 2), (2, 200, 64 * 8 + 23, 2, False, 128, 2), (2, 200, 64 * 26 + 23, 2, True, 128, 2),
    (4, 1800, 64 * 24 + 5, 5, True, 128, 1), (4, 1200, 64 * 24 + 9, 10, False, 256, 2), (8, 1290, 64 * 20 + 10, 10, False, 256, 1),
])
def test_attn_block_references_of_every_kernel(B, Bn, T, Tc, heads, cut, queries, groups, where):
    import torch
    C = heads * 64
    r = rng(T + Tc)
    n0 = r.standard_normal((heads, 64)).astype(np.float32)
    n0 = ((n0 - n0.mean(1, keepdims=True)) / n0.std(1, keepdims=True)).reshape(C)       # what LayerNorm makes of a row along n0
    sign = np.where(r.random((Bn, T, 1)) < 0.5, 1.0, -1.0).astype(np.float32)
    h = (sign * n0 * (1.0 + 0.05 * r.standard_normal((Bn, T, 1))) + 0.15 * r.standard_normal((Bn, T, C))).astype(np.float32)
    # the key tiles [lo, hi) of each range with a reference of its own: halves of a cut tile, and in them (or in the whole) groups of wavefronts
    nt = (Tc + 63) // 64
    ranges = [(0, (nt + 1) // 2), ((nt + 1) // 2, nt)] if cut else [(0, nt)]
    if groups == 2:
        ranges = [s for lo, hi in ranges for s in ((lo, lo + (hi - lo) // 2), (hi - (hi - lo + 1) // 2, hi))]
    level = np.zeros(nt, np.float32)                     # natural-log score of a key tile for a query along +n0
    for lo, hi in ranges:
        level[(lo + hi) // 2 if where == "climb" else lo] = 105.0
    a = level[np.arange(Tc) // 64] + 0.5 * r.standard_normal(Tc).astype(np.float32)
    ctx = G.bf16_round((a[None, :, None] * n0[None, None, :] / 8.0 + 0.05 * r.standard_normal((Bn, Tc, C))).astype(np.float32))
    eye = {"W": np.eye(C, dtype=np.float32), "b": None, "A": None, "B": None, "scale": 0.0}
    pv = mkproj(r, C, C, 0, bias=False)
    po = mkproj(r, C, C, 0, bias=True)
    g, b = np.ones(C, np.float32), np.zeros(C, np.float32)
    # the test is what it says
    q0 = O.layernorm(h[0], g, b)[:, :64]
    scores = {up: (q0[int(np.argmax(sign[0, :, 0] == up))] @ ctx[0, :, :64].T.astype(np.float64)) / 8.0 * 1.4426950408889634 for up in (1.0, -1.0)}
    for lo, hi in ranges:
        first, rest = slice(64 * lo, 64 * lo + 64), slice(64 * lo + 64, 64 * hi)
        if where == "climb":
            assert scores[1.0][rest].max() - scores[1.0][first].max() > 135
        else:
            assert scores[-1.0][first].max() < -135 and scores[-1.0][rest].max() > -30 and scores[1.0][first].max() > 135
    args = (torch.from_numpy(h).cuda(), dev(ctx, B), dev(g, B), dev(b, B), B.Proj.from_numpy(eye), B.Proj.from_numpy(eye), B.Proj.from_numpy(pv), B.Proj.from_numpy(po), heads)
    with B.dry_run(detail=3) as names:
        B.attn_block_fwd(*args)
    assert "attention prescaled try%s, %d queries, %d groups" % (" cut" if cut else "", queries, groups) in names
    got = host(B.attn_block_fwd(*args))
    assert np.isfinite(got).all()
    for s in (0, Bn - 1):        # (samples do not meet)
        ref = O.attn_sublayer(h[s:s + 1], ctx[s:s + 1], g, b, eye, eye, pv, po, heads)
        assert rel_err(got[s:s + 1] - h[s:s + 1], ref - h[s:s + 1]) <= BF16_TOL


# Whole key tiles with scores of -inf (weights of exactly zero): where a range of keys with a reference of its own begins, and the whole of the last
# such range.  Plain keys, and keys of a block whose projection overflows there
@pytest.mark.parametrize("where", ["first", "all"])
@pytest.mark.parametrize("block,Bn,Tq,Tk,heads,kernel", [
    (False, 1, 130, 64 * 8 + 3, 3, ", 128 queries, 2 groups"), (False, 1, 200, 64 * 20 + 9, 2, " try, 128 queries, 2 groups"), (False, 1, 1100, 64 * 24 + 61, 30, " try, 256 queries, 2 groups"),
    (False, 1, 4096, 64 * 21, 20, " try cut merge, 128 queries, 1 groups"), (True, 2, 200, 64 * 8 + 23, 2, " prescaled try, 128 queries, 2 groups"),
    (True, 2, 200, 64 * 26 + 23, 2, " prescaled try cut, 128 queries, 2 groups"), (True, 4, 1200, 64 * 24 + 9, 10, " prescaled try, 256 queries, 2 groups"),
])
def test_attention_key_tiles_at_minus_infinity(B, block, Bn, Tq, Tk, heads, kernel, where):
    import torch
    C = heads * 64
    r = rng(Tq + Tk + heads)
    nt = (Tk + 63) // 64
    ranges = [(0, (nt + 1) // 2), ((nt + 1) // 2, nt)] if " cut" in kernel else [(0, nt)]
    if kernel.endswith("2 groups"):
        ranges = [s for lo, hi in ranges for s in ((lo, lo + (hi - lo) // 2), (hi - (hi - lo + 1) // 2, hi))]
    out = np.zeros(nt, bool)
    for lo, hi in ranges if where == "first" else ranges[-1:]:
        out[lo:hi if where == "all" else lo + 1] = True
    out = out[np.arange(Tk) // 64]
    q = r.standard_normal((Bn, Tq, heads, 64), dtype=np.float32)
    q[..., 0] = 2.0 + np.abs(q[..., 0])                  # (positive after LayerNorm, too)
    q = G.bf16_round(q).reshape(Bn, Tq, C)
    k = r.standard_normal((Bn, Tk, heads, 64), dtype=np.float32)
    k[..., 0] = 0.0
    k = G.bf16_round(k).reshape(Bn, Tk, C)
    if block:
        eye, pk, pv, po = (mkproj(r, C, C, 0, bias=i == 3) for i in range(4))
        eye["W"] = np.eye(C, dtype=np.float32)
        pk["W"] = np.diag(np.where(np.arange(C) % 64 == 0, 64.0, 1.0)).astype(np.float32)
        pv["W"][:, ::64] = 0.0
        k[:, out, ::64] = -2.0 ** 127
        g, b = np.ones(C, np.float32), np.zeros(C, np.float32)
        args = (torch.from_numpy(q).cuda(), dev(k, B), dev(g, B), dev(b, B), *[B.Proj.from_numpy(p) for p in (eye, pk, pv, po)], heads)
        call = lambda: B.attn_block_fwd(*args)
        want = lambda s: O.attn_sublayer(q[s:s + 1], k[s:s + 1][:, ~out], g, b, eye, pk, pv, po, heads) - q[s:s + 1]
        got_of = lambda y, s: y[s:s + 1] - q[s:s + 1]
    else:
        k[:, out, ::64] = -np.inf
        v = G.bf16_round(r.standard_normal((Bn, Tk, C), dtype=np.float32))
        args = (dev(q, B), dev(k, B), vt_layout(v, B), heads)
        call = lambda: B.attention_fwd(*args)
        h = np.array(sorted({0, heads // 2, heads - 1}))
        cols = (h[:, None] * 64 + np.arange(64)).ravel()
        want = lambda s: O.attention(q[..., cols], k[..., cols][:, ~out], v[..., cols][:, ~out], len(h), dtype=np.float32 if Tq > 1000 else np.float64)
        got_of = lambda y, s: y[..., cols]
    with B.dry_run(detail=3) as names:
        call()
    assert "attention" + kernel in names
    y = host(call())
    assert np.isfinite(y).all()
    for s in sorted({0, Bn - 1}):
        assert rel_err(got_of(y, s), want(s)) <= BF16_TOL


# ... and what lies behind such a tile far below 0, but above everything before it: it has all the weight.  (A range of prescaled keys that begins with
# -inf starts from the reference 0, to which these scores, 2^-200 and less, are nothing.)
@pytest.mark.parametrize("Bn,T,Tc,heads,cut,queries,groups", [
    (2, 200, 64 * 8 + 23, 2, False, 128, 2), (2, 200, 64 * 26 + 23, 2, True, 128, 2), (4, 1200, 64 * 24 + 9, 10, False, 256, 2),
])
def test_attn_block_low_scores_behind_a_tile_at_minus_infinity(B, Bn, T, Tc, heads, cut, queries, groups):
    import torch
    C = heads * 64
    r = rng(T + Tc + heads)
    nt = (Tc + 63) // 64
    lo, hi = ((nt + 1) // 2, nt) if cut else (0, nt)
    begin = hi - (hi - lo + 1) // 2                      # first tile of the last group's keys (an odd tile count: the shared one)
    tile = np.arange(Tc) // 64
    out = tile == begin
    q = r.standard_normal((Bn, T, heads, 64), dtype=np.float32)
    q[..., 0] = 4.0 + np.abs(q[..., 0])                  # (2.4 to 5 after LayerNorm)
    q = q.reshape(Bn, T, C)
    k = r.standard_normal((Bn, Tc, heads, 64), dtype=np.float32)
    k[..., 0] = np.where(tile > begin, -8.0, -10.0)[None, :, None]
    k[:, out, :, 0] = -2.0 ** 127                        # times 64: -inf
    k = G.bf16_round(k).reshape(Bn, Tc, C)
    eye, pk, pv, po = (mkproj(r, C, C, 0, bias=i == 3) for i in range(4))
    eye["W"] = np.eye(C, dtype=np.float32)
    pk["W"] = np.diag(np.where(np.arange(C) % 64 == 0, 64.0, 1.0)).astype(np.float32)
    pv["W"][:, ::64] = 0.0
    g, b = np.ones(C, np.float32), np.zeros(C, np.float32)
    # the test is what it says (scores as exponents of 2)
    q0 = O.layernorm(q, g, b).reshape(Bn, T, heads, 64)[..., 0]
    assert q0.min() * 8.0 * 8.0 * 1.44 > 150 and q0.min() * 2.0 * 8.0 * 1.44 > 30 and q0.max() * 10.0 * 8.0 * 1.45 < 4000
    args = (torch.from_numpy(q).cuda(), dev(k, B), dev(g, B), dev(b, B), *[B.Proj.from_numpy(p) for p in (eye, pk, pv, po)], heads)
    with B.dry_run(detail=3) as names:
        B.attn_block_fwd(*args)
    assert "attention prescaled try%s, %d queries, %d groups" % (" cut" if cut else "", queries, groups) in names
    y = host(B.attn_block_fwd(*args))
    assert np.isfinite(y).all()
    for s in (0, Bn - 1):
        want = O.attn_sublayer(q[s:s + 1], k[s:s + 1][:, ~out], g, b, eye, pk, pv, po, heads) - q[s:s + 1]
        assert rel_err(y[s:s + 1] - q[s:s + 1], want) <= BF16_TOL
