"""The launches of a whole stack, read off without a GPU (dry runs; the pointers are made up and never followed): where the text keys and
values of a block ride, that they leave ff2 its kernel, and which weights are read ahead by which launch."""
import ctypes as C
import re

import pytest

from test_kernel_choice_host import B  # noqa: F401

PROJS = ("q1", "k1", "v1", "o1", "q2", "k2", "v2", "o2", "ff1", "ff2")
Tc, Dc = 77, 2048


class Stack:
    """A stack's launches by block and place, and where its weights are."""

    def __init__(self, B, Bn, T, Cc, depth, r=0, rf=0, text_r=None, ws=None, expect=0):
        L = B.lib()
        self.weights = {}          # address -> (bytes, (block, launch of the block))
        at = [1 << 32]

        def take(nbytes, use):
            p = at[0]
            self.weights[p] = (nbytes, use)
            at[0] += (nbytes + 4095) // 4096 * 4096 + 4096
            return p

        def proj(n, k, rank, use):
            W = take(n * k * 2, use)
            return B.sd_proj(W, None, take(rank * k * 2, use) if rank else None, take(n * rank * 2, use) if rank else None, rank, 1.0)

        blocks = (B.sd_block_params * depth)()
        text_r = r if text_r is None else text_r
        for i, b in enumerate(blocks):
            for n in ("ln1_g", "ln1_b", "ln2_g", "ln2_b", "ln3_g", "ln3_b"):
                setattr(b, n, 0x10000)
            for n in PROJS:
                rank = rf if n in ("ff1", "ff2") else text_r if n in ("k2", "v2") else r
                k = Dc if n in ("k2", "v2") else 4 * Cc if n == "ff2" else Cc
                setattr(b, n, proj(8 * Cc if n == "ff1" else Cc, k, rank, (i, {"q1": "qkv", "k1": "qkv", "v1": "qkv", "k2": "text", "v2": "text"}.get(n, n))))
        p = B.sd_stack_params(0x10000, 0x10000, proj(Cc, Cc, 0, (-1, "in")), proj(Cc, Cc, 0, (depth, "out")), C.cast(blocks, C.POINTER(B.sd_block_params)), depth)
        rmax = max(r, rf, text_r)
        need = L.sd_spatial_transformer_workspace_bytes(Bn, T, Cc, Tc, Dc, rmax)
        with B.dry_run(detail=True) as names:
            rc = L.sd_spatial_transformer_fwd(0x100000, 0x200000, C.byref(p), 0x300000, Bn, T, Cc, Cc // 64, Tc, Dc, 0x10000000, need if ws is None else ws, None)
        assert rc == expect, L.sd_last_error()
        if expect:
            return
        self.names = names
        # a block: LayerNorm, q k v, attention, out | LayerNorm, query, attention, out | LayerNorm, (down,) ff1, ff2
        starts = [i for i, n in enumerate(names) if n.startswith("layernorm")]
        assert len(starts) == 3 * depth and "clear" not in names[starts[-1]]
        self.at = {}               # (block, launch) -> index into names
        for b in range(depth):
            s = starts[3 * b:3 * b + 3]
            self.at[b, "qkv"], self.at[b, "o1"] = s[0] + 1, s[1] - 1
            self.at[b, "q2"], self.at[b, "o2"] = s[1] + 1, s[2] - 1
            last = starts[3 * b + 3] - 1 if b + 1 < depth else len(names) - 2
            self.at[b, "ff1"], self.at[b, "ff2"] = last - 1, last
        self.at[depth, "out"] = len(names) - 1
        for b in range(depth):
            self.at[b, "text"] = self.at[b - 1, "ff2"] if b and self.rides(b) else self.at[b, "qkv"]

    def launch(self, block, which):
        """(kernel, problems); q, k, v of many samples are two launches, whose problems are added"""
        at = end = self.at[block, which]
        while which == "qkv" and not self.names[end + 1].startswith("attention"):
            end += 1
        got = [re.match(r"(.*?), (\d+) problems", n) for n in self.names[at:end + 1]]
        return got[0].group(1), sum(int(m.group(2)) for m in got)

    def rides(self, b):
        """Whether block b's text keys / values are in the ff2 launch of the block before.  They are in one of the two."""
        in_ff2 = self.launch(b - 1, "ff2")[1] - self.alone
        in_qkv = self.launch(0, "qkv")[1] - self.launch(b, "qkv")[1]
        assert in_ff2 == in_qkv
        return in_ff2 > 0

    @property
    def alone(self):               # problems of an ff2 launch without riders: the last block's has none
        return self.launch(max(b for b, n in self.at if n == "ff2"), "ff2")[1]


# ---- text keys and values: in the ff2 launch of the block before, or in the block's q, k, v launch
@pytest.mark.parametrize("Bn,T,Cc,r,rf,ff2", [
    (2, 1024, 1280, 64, 64, "gemm 128x128/8 waves/4 stages res32 flags"), (2, 4096, 640, 64, 64, "gemm 256x128/8 waves/3 stages res32 flags"),
    (1, 3300, 640, 64, 64, "gemm 128x128/8 waves/4 stages res32 flags"), (2, 1100, 1280, 0, 0, "gemm 128x128/8 waves/4 stages res32"),
])
def test_text_keys_ride_in_the_ff2_launch(B, Bn, T, Cc, r, rf, ff2):  # noqa: F811
    s = Stack(B, Bn, T, Cc, 2, r, rf)
    assert s.rides(1) and s.launch(0, "ff2")[0] == s.launch(1, "ff2")[0] == ff2


@pytest.mark.parametrize("Bn,T,Cc,r,rf", [(1, 3300, 640, 16, 16), (2, 256, 320, 8, 0), (1, 988, 1280, 16, 0), (2, 4200, 1280, 64, 64)])
def test_text_keys_stay_with_the_queries(B, Bn, T, Cc, r, rf):  # noqa: F811
    assert not Stack(B, Bn, T, Cc, 2, r, rf).rides(1)     # ff2 in its in-tile kernel, or in several rounds


# One rule for ff2's tiles, with riders and without: ranges of token counts about the ends of a round of 128x128 tiles (where the text keys'
# tiles would push ff2 out of it into 256x128 tiles on half the CUs) and of 256x128 tiles; adapters everywhere, on attention only, on nothing.
# Where q, k, v with them would be two launches (more than 16 problems: three samples and more with adapters), any one round will do.
@pytest.mark.parametrize("Bn,Cc,r,rf,lo,hi", [
    (2, 1280, 64, 64, 1000, 1700), (2, 1280, 32, 32, 1000, 1700), (2, 1280, 16, 0, 1000, 1700), (2, 1280, 0, 0, 1000, 1700), (1, 1280, 64, 64, 2500, 3100), (4, 1280, 0, 0, 500, 800),
    (2, 640, 64, 64, 2100, 4400), (2, 640, 16, 0, 2500, 4400), (4, 640, 0, 0, 1000, 1400), (1, 640, 8, 0, 3000, 4400), (2, 320, 64, 64, 3500, 4400),
    (3, 1280, 64, 64, 600, 1100), (4, 1280, 64, 64, 450, 850), (4, 640, 64, 64, 1000, 1400), (3, 640, 32, 0, 1300, 1800),
])
def test_riders_leave_ff2_its_tiles(B, Bn, Cc, r, rf, lo, hi):  # noqa: F811
    tiles = lambda name: re.match(r"(.*) stages", name).group(1) if name.startswith("gemm ") else name
    one_round = ("gemm 128x128/8 waves/4", "gemm 256x128/8 waves/3")
    two_launches = r > 0 and 4 + 2 * Bn + 2 + 2 * Bn > 16
    for T in sorted({*range(lo, hi, 53), *(t for e in range(lo // 128, hi // 128) for t in (128 * e, 128 * e + 4))}):
        s = Stack(B, Bn, T, Cc, 2, r, rf)
        with_text, alone = tiles(s.launch(0, "ff2")[0]), tiles(s.launch(1, "ff2")[0])
        if s.rides(1):
            assert with_text in one_round and alone in one_round and (with_text == alone or two_launches), T
        else:
            assert with_text == alone and not (two_launches and alone == one_round[0]), T


@pytest.mark.parametrize("Bn,T,Cc,r,rf", [(2, 1296, 1280, 64, 64), (2, 1440, 1280, 64, 64), (1, 2800, 1280, 64, 64), (4, 640, 1280, 0, 0), (2, 2500, 640, 64, 64), (2, 1400, 1280, 16, 0)])
def test_text_keys_that_do_not_fit_stay_with_the_queries(B, Bn, T, Cc, r, rf):  # noqa: F811
    assert not Stack(B, Bn, T, Cc, 2, r, rf).rides(1)


# ---- workspaces without room for the halves of cut attention tiles
@pytest.mark.parametrize("Bn,T,Cc", [(1, 4096, 320), (2, 3100, 320), (1, 1500, 640)])
def test_workspace_without_room_for_cut_tiles(B, Bn, T, Cc):  # noqa: F811
    L = B.lib()
    need = L.sd_spatial_transformer_workspace_bytes(Bn, T, Cc, Tc, Dc, 8)
    least = need - (T + 127) // 128 * (Cc // 64) * Bn * 2 * 34 * 256 * 4
    assert "attention prescaled try cut" in Stack(B, Bn, T, Cc, 2, 8).names
    for ws in (need - 256, least):
        names = Stack(B, Bn, T, Cc, 2, 8, ws=ws).names
        assert "attention prescaled try cut" not in names and names.count("attention prescaled try") == 4
    Stack(B, Bn, T, Cc, 2, 8, ws=least - 256, expect=-3)
    assert ("need %d (%d at the least" % (need, least)) in L.sd_last_error().decode()


# ---- from self-attention's output to the feed-forward's input in one launch, or not (chain_takes)
def chain(B, Bn, T, Cc, r):  # noqa: F811
    return "attention of the chain" in Stack(B, Bn, T, Cc, 1, r).names


# 320 channels, two workgroups a CU: from 38 blocks of 32 rows on; in a second and third round with small adapters only, or where the second is well filled; nowhere
# that the launches need a round less (rows up to a multiple of 8192)
@pytest.mark.parametrize("Bn,T,none,r40,r64,r128", [
    (1, 1184, 0, 0, 0, 0), (1, 1216, 1, 1, 1, 1), (2, 4096, 1, 1, 1, 1), (2, 4125, 1, 1, 1, 1), (86, 95, 0, 0, 0, 0), (4, 3517, 1, 1, 1, 1), (8, 2048, 1, 1, 1, 1), (4, 4100, 1, 1, 0, 0),
    (6, 2730, 0, 0, 0, 0), (6, 3200, 1, 1, 1, 0), (8, 4096, 1, 1, 1, 0), (12, 2730, 0, 0, 0, 0), (10, 3280, 1, 1, 0, 0),
])
def test_chain_of_320_channels_by_rounds(B, Bn, T, none, r40, r64, r128):  # noqa: F811
    assert [chain(B, Bn, T, 320, r) for r in (0, 40, 64, 128)] == [bool(none), bool(r40), bool(r64), bool(r128)]


# samples whose last blocks are partly empty: by their rows, except where 320 channels have a CU to a workgroup
@pytest.mark.parametrize("Bn,T,Cc,taken", [
    (90, 31, 640, 0), (91, 32, 640, 1), (45, 33, 640, 0), (60, 33, 640, 0), (41, 71, 640, 1), (88, 33, 640, 1), (245, 33, 640, 0), (250, 40, 640, 0), (167, 95, 640, 1), (244, 64, 640, 1),
    (256, 1, 320, 1), (128, 33, 320, 1), (300, 1, 320, 0), (240, 33, 320, 0), (150, 95, 320, 1), (300, 75, 320, 0), (208, 95, 320, 1),
])
def test_chain_by_rows(B, Bn, T, Cc, taken):  # noqa: F811
    assert chain(B, Bn, T, Cc, 16) == bool(taken)


# 640 channels: from 2880 rows on with adapters on any of the three projections, without from 3264
@pytest.mark.parametrize("Bn,T,r,taken", [(1, 2879, 8, 0), (1, 2880, 8, 1), (1, 2880, 0, 0), (30, 97, 0, 0), (60, 48, 0, 0), (1, 3263, 0, 0), (1, 3264, 0, 1), (2, 3952, 0, 1)])
def test_chain_of_640_channels_from(B, Bn, T, r, taken):  # noqa: F811
    assert chain(B, Bn, T, 640, r) == bool(taken)


# ---- weights read ahead
def ranges(name):
    return [(int(p, 16), int(n)) for p, n in re.findall(r" ([0-9a-f]+)\+(\d+)", name.split("ahead", 1)[1])] if ", ahead" in name else []


@pytest.mark.parametrize("Bn,T,Cc,depth,r,rf", [(2, 1024, 1280, 4, 64, 64), (1, 988, 1280, 6, 16, 0), (2, 4096, 640, 8, 64, 64), (2, 4096, 640, 8, 0, 0), (1, 1500, 1280, 5, 32, 32)])
def test_weights_are_read_ahead_of_their_launches(B, Bn, T, Cc, depth, r, rf):  # noqa: F811
    """Every part lies in one weight, no byte is read twice, none after the launch that uses it, and most of the weights behind the first
    block are read."""
    s = Stack(B, Bn, T, Cc, depth, r, rf)
    assert "ahead" in " ".join(s.names)
    read = {}
    for i, name in enumerate(s.names):
        for p, n in ranges(name):
            base = max(w for w in s.weights if w <= p)
            nbytes, use = s.weights[base]
            assert n > 0 and p - base + n <= nbytes
            assert s.at[use] > i, (use, name)
            for q, m in read.get(base, []):
                assert p >= q + m or q >= p + n
            read.setdefault(base, []).append((p, n))
    later = [w for w, (_, use) in s.weights.items() if 0 < use[0] < depth]
    got = sum(n for w in later for _, n in read.get(w, []))
    assert got > 0.5 * sum(s.weights[w][0] for w in later)


# what the last-level cache holds is not read ahead
@pytest.mark.parametrize("Bn,T,Cc,depth,r,rf", [(2, 256, 320, 1, 8, 0), (2, 4096, 640, 2, 64, 64), (2, 1024, 1280, 2, 64, 64)])
def test_small_stacks_read_nothing_ahead(B, Bn, T, Cc, depth, r, rf):  # noqa: F811
    assert "ahead" not in " ".join(Stack(B, Bn, T, Cc, depth, r, rf).names)
