"""GPU parity of KIVI-style keys with one range per channel over the whole
supplied sequence, text included (kivi_group = 0; §4 Quantization setup),
against the oracle: codes, metadata, side store and reconstruction
bit-exact for quantize / dequantize and for the one-pass simulated
quantization; every slice of the full LLaVA-NeXT-7B-shaped cache.

Slices of up to 32 workgroups' capacity (24 slots of 8192/D rows: 3072,
1536 and 768 rows at head_dim 64, 128 and 256) go through the partitioned
resident kernel: P workgroups each hold a run of a slice's rows on chip and
combine their partial ranges through the call's workspace (past 8, P is
rounded up to 16 or 32); longer slices, up to 256 workgroups' capacity, go
through spread groups of 64, 128 or 256 workgroups if a roll call finds the
whole grid on the chip, and else, like still longer ones, through the split kernels (a
range launch over chunks of every slice merging per-channel ranges into the
workspace, then a code launch), and a slice one workgroup holds, on a device
too small for a group, through the two-pass kernel (no workspace).
Covered: one to eight, 16 and 32 workgroups per slice and the capacity
boundaries, several slices per group (with the grid shrunk through the
HG_TEST_CUS hook), identical bytes for different grid sizes, no exchange
wait running out of polls, and groups some of whose partners do not run or
come late (HG_TEST_ABSENT, HG_TEST_POLLS), whose slices the others then take
one workgroup a slice."""
import numpy as np
import pytest
import torch

import synthkv
import wholecache
from hgtest import GROUPS, compare_full, kivi_plan
from test_gpu_fakequant import check as check_fake
from test_gpu_parity import _assert_exact, small

pytestmark = pytest.mark.gpu

CASES = [small("kivi", D, bits, ko).with_(kivi_group=0, name=f"kiviseq-D{D}-b{bits}-ko{ko}")
         for D in (64, 128, 256) for bits in (2, 3, 4) for ko in (0, 1)]


@pytest.mark.parametrize("w", CASES, ids=lambda w: w.name)
def test_small(w):
    K, V = synthkv.gen_kv(w)
    _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w)), w.name)


@pytest.mark.parametrize("w", CASES[:6], ids=lambda w: w.name)
@pytest.mark.parametrize("inplace", [False, True])
def test_fake(w, inplace):
    K, V = synthkv.gen_kv(w)
    check_fake(w, K, V, synthkv.protect_mask(w), inplace)


@pytest.mark.parametrize("img_len,img_start,text", [(1, 0, 0), (5, 3, 40), (130, 0, 7), (64, 64, 0)])
def test_spans(img_len, img_start, text):
    w = small("kivi", img_len=img_len, img_start=img_start, text=text, L=1, B=2, H=2,
              n_protected=1).with_(kivi_group=0)
    K, V = synthkv.gen_kv(w)
    K[0, 0, 0, 0, 3] = 3000.0  # a large value in the first row (text when img_start > 0)
    _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w)), f"span{img_len}")


def test_full_size_llava():
    """The LLaVA-NeXT-7B-shaped cache with one key range per channel over the
    whole sequence: every slice against the oracle."""
    w = synthkv.WORKLOADS["llava-next-7b"].with_(kivi_group=0)
    wholecache.assert_whole(wholecache.quantize_dequantize(w), w)


@pytest.mark.parametrize("inplace", [False, True])
def test_full_size_llava_one_pass(inplace):
    w = synthkv.WORKLOADS["llava-next-7b"].with_(kivi_group=0)
    wholecache.assert_whole(wholecache.fake_quantize(w, inplace=inplace), w)


def test_long_single_slice():
    """One key slice of 2^21 + 5 tokens at head_dim 128 (512 MiB, text rows at
    both ends): far past 32 workgroups' capacity, so the split kernels range
    and code it in 1025 and 1024 chunks; every byte against the oracle."""
    T = (1 << 21) + 5
    w = synthkv.Workload("kiviseq-long-slice", L=1, B=1, H=1, T=T, D=128, img_start=1000, img_len=T - 1777,
                         bits=2, base="kivi", keys_only=0, n_protected=0, k_outliers=4, k_outlier_scale=10.0,
                         kivi_group=0, seed=21)
    assert T > 8 * capacity(128)
    wholecache.assert_whole(wholecache.quantize_dequantize(w), w)


@pytest.mark.parametrize("fake", [False, True])
def test_two_pass_without_workspace(fake, monkeypatch):
    """Slices one workgroup holds need no workspace; on a device with fewer
    than 8 compute units (the grid hook) there is no group of 8 to run them, so
    the two-pass kernel takes them."""
    monkeypatch.setenv("HG_TEST_CUS", "4")
    w = small("kivi", 128, 3, 0, img_len=1000, img_start=9, text=20, L=2, B=3, H=2,
              n_protected=1).with_(kivi_group=0, name="kiviseq-two-pass")
    assert w.T <= capacity(128)
    K, V = synthkv.gen_kv(w)
    mask = synthkv.protect_mask(w)
    if fake:
        check_fake(w, K, V, mask, False)
    else:
        _assert_exact(compare_full(w, K, V, mask), w.name)


def test_split_batches(monkeypatch):
    """More quantized key slices than the workspace holds range words for
    (2048), through the split kernels (forced by the grid hook: 4 compute
    units cannot hold a group of 8): the slices are taken in two batches, the
    second batch's words cleared by a kernel of their own."""
    monkeypatch.setenv("HG_TEST_CUS", "4")
    w = small("kivi", 64, 2, 1, img_len=50, img_start=3000, text=23, L=8, B=3, H=128,
              n_protected=24).with_(kivi_group=0, name="kiviseq-split-batches")
    assert w.T > capacity(64) and (w.L * w.H - w.n_protected) * w.B > 2048
    K, V = synthkv.gen_kv(w)
    _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w)), w.name)


def capacity(D):
    """Rows one workgroup of the partitioned kernel holds."""
    return 24 * 8192 // D


# Enough (head, row) items that every group takes several slices once the
# grid is shrunk to 32 compute units' worth (32 workgroups: 32, 16 and 8
# groups of 1, 2 and 4 workgroups), so each slot's refill with the next
# slice and the alternation of the exchange buffers are exercised.
STREAM_CASES = [small("kivi", D, bits, ko, img_len=T - 50, img_start=20, text=30, L=2, B=6, H=8,
                      n_protected=2).with_(kivi_group=0, name=f"kiviseq-streams-D{D}-T{T}-b{bits}-ko{ko}")
                for D in (64, 128, 256) for T in (200, capacity(D) + 300, 3 * capacity(D) + 7)
                for bits in (2, 3) for ko in (0, 1)]


@pytest.mark.parametrize("w", STREAM_CASES, ids=lambda w: w.name)
def test_resident_streams(w, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", "32")
    K, V = synthkv.gen_kv(w)
    _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w)), w.name)


@pytest.mark.parametrize("w", STREAM_CASES[2:4] + STREAM_CASES[8:10], ids=lambda w: w.name)
@pytest.mark.parametrize("inplace", [False, True])
def test_resident_streams_fake(w, inplace, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", "32")
    K, V = synthkv.gen_kv(w)
    check_fake(w, K, V, synthkv.protect_mask(w), inplace)


@pytest.mark.parametrize("cus", ["", "256", "64", "24", "16", "8", "1"])
def test_grid_size_does_not_change_the_bytes(cus, monkeypatch):
    """The same cache (two workgroups per slice) under persistent grids sized
    for 256 down to 1 compute units (fewer than 16 are too few workgroups for
    a multiple of 8 groups: the split kernels take over), and once more with
    the full grid: every run equals the oracle."""
    w = small("kivi", 128, 2, 0, img_len=3000, img_start=5, text=3, L=2, B=6, H=5,
              n_protected=2).with_(kivi_group=0)
    monkeypatch.setenv("HG_TEST_CUS", cus)
    K, V = synthkv.gen_kv(w)
    _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w)), f"cus{cus or 'all'}")


# Slices at each workgroup count's capacity and one row past it (one to eight
# workgroups per slice, then 16 and 32; past 32 workgroups' capacity, the
# split kernels), spans at the start, in the middle and at the end of the
# slice (the middle only for the longest slices).
def _boundary_cases():
    out = []
    for D in (64, 128, 256):
        c = capacity(D)
        for T in (c, c + 1, 2 * c + 1, 3 * c - 5, 8 * c, 8 * c + 1):
            for img_start, img_len in ((0, T), (T // 3, T // 2), (T - 40, 40)):
                out.append((D, T, img_len, img_start))
        for T in (16 * c, 16 * c + 1, 32 * c, 32 * c + 1):
            out.append((D, T, T // 2, T // 3))
    return out


@pytest.mark.parametrize("D,T,img_len,img_start", _boundary_cases(), ids=lambda v: str(v))
def test_capacity_boundary(D, T, img_len, img_start):
    w = small("kivi", D, 3, 0, img_len=img_len, img_start=img_start, text=T - img_len - img_start,
              L=1, B=2, H=2, n_protected=1).with_(kivi_group=0)
    assert w.T == T
    K, V = synthkv.gen_kv(w)
    K[0, :, :, T - 1, 5] = -4000.0  # an extreme in the last row of every slice
    K[0, :, :, 0, 9] = 5000.0       # and in the first
    _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w)), f"D{D}-T{T}-n{img_len}-s{img_start}")


# The resident kernel's forms (24, 15 and 8 slots of 8192/D rows) at their
# capacities, one row past them and just below: one round of a short form over
# more workgroups than the slice needs, the longest form at the capacity of 8
# workgroups on a grid that holds no more, and several rounds on a small grid.
def _form_cases():
    out = []
    for D in (64, 128, 256):
        r = 8192 // D
        for cus, P, slots in (("256", 6, 8), ("256", 4, 15), ("256", 32, 15), ("64", 8, 24), ("48", 2, 24)):
            out += [(D, cus, P * slots * r + d) for d in (-3, 0, 1) if P * slots * r + d > 24 * r]
    return out


@pytest.mark.parametrize("D,cus,T", _form_cases(), ids=lambda v: str(v))
def test_form_boundary(D, cus, T, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", cus)
    w = small("kivi", D, 2, 1, img_len=T - 9, img_start=4, text=5, L=2, B=3, H=5,
              n_protected=2).with_(kivi_group=0)
    K, V = synthkv.gen_kv(w)
    K[0, :, :, T - 1, 5] = -4000.0  # extremes in the last and first rows
    K[0, :, :, 0, 9] = 5000.0
    _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w)), f"D{D}-T{T}-cus{cus}")


# Each form filled to the last row slot, with the partners and slots that the plan
# takes there: one workgroup, groups of up to 8 and wide groups (24 slices).
FORM_CAPACITY = [("", 1, 8), ("", 1, 15), ("", 8, 8), ("", 6, 15), ("", 8, 15), ("", 8, 24), ("", 16, 15), ("", 16, 24),
                 ("64", 2, 15), ("64", 2, 24)]


@pytest.mark.parametrize("D,inplace", [(64, None), (128, None), (256, None), (128, True)])
@pytest.mark.parametrize("cus,P,slots", FORM_CAPACITY, ids=lambda v: str(v) or "all")
def test_form_capacity(D, cus, P, slots, inplace, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", cus)
    T = P * slots * 8192 // D
    w = small("kivi", D, 2, 1, img_len=T - 9, img_start=4, text=5, L=2, B=3, H=5,
              n_protected=2).with_(kivi_group=0, name=f"kiviseq-form-D{D}-P{P}-{slots}")
    assert kivi_plan(w.T, D, 24, w.img_len, int(cus or 256))[:3] == (GROUPS, P, slots)
    K, V = synthkv.gen_kv(w)
    K[0, :, :, T - 1, 5] = -4000.0  # extremes in the last and first rows
    K[0, :, :, 0, 9] = 5000.0
    if inplace is None:
        _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w)), w.name)
    else:
        check_fake(w, K, V, synthkv.protect_mask(w), inplace)


@pytest.mark.parametrize("T", [1536, 1537, 3008, 12288, 12289, 24577, 49152, 49153])
@pytest.mark.parametrize("inplace", [False, True])
def test_capacity_boundary_fake(T, inplace):
    w = small("kivi", 128, 2, 1, img_len=T - 60, img_start=20, text=40,
              L=1, B=2, H=2, n_protected=1).with_(kivi_group=0)
    K, V = synthkv.gen_kv(w)
    check_fake(w, K, V, synthkv.protect_mask(w), inplace)


# Spread groups: slices past 32 workgroups' capacity, at the capacities of 64,
# 128 and 256 workgroups of 8, 16 and 24 slots and one row past them, one round
# and several (the grid hook: 64 and 128 compute units hold one group of 64, one
# of 128).  `outcome` is what the roll call decides: every workgroup is here, or
# (HG_TEST_ABSENT waits for one that does not exist) the split kernels do the
# work, or no roll call (past the capacity).
def _spread_cases():
    out = []
    for D in (64, 128, 256):
        r = 8192 // D
        few = 9 if D == 64 else 4  # (few slices at head_dim 64 go to the split kernels)
        out += [(D, "", 32 * 24 * r + 1, few), (D, "", 64 * 16 * r, few), (D, "128", 64 * 16 * r + 1, 5),
                (D, "64", 64 * 24 * r, 4), (D, "", 64 * 24 * r + 1, 4), (D, "", 128 * 8 * r + 1, 1)]
    out += [(256, "128", 128 * 16 * 32, 4), (256, "", 128 * 16 * 32 + 1, 4), (256, "", 256 * 8 * 32, 1),
            (256, "", 256 * 24 * 32, 1), (256, "", 256 * 24 * 32 + 1, 1)]
    return out


def _spread_workload(D, T, H, bits=2):
    w = small("kivi", D, bits, 1, img_len=T - 700, img_start=300, text=400, L=1, B=1, H=H,
              n_protected=1 if H > 1 else 0).with_(kivi_group=0, name=f"kiviseq-spread-D{D}-T{T}")
    assert w.T == T
    K, V = synthkv.gen_kv(w)
    K[0, :, :, T - 1, 5] = -4000.0  # extremes in the last and first rows
    K[0, :, :, 0, 9] = 5000.0
    return w, K, V, synthkv.protect_mask(w)


@pytest.mark.parametrize("D,cus,T,H", _spread_cases(), ids=lambda v: str(v) or "all")
@pytest.mark.parametrize("absent", ["", "1"])
def test_spread_groups(D, cus, T, H, absent, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", cus)
    monkeypatch.setenv("HG_TEST_ABSENT", absent)
    w, K, V, mask = _spread_workload(D, T, H, bits=3 if D == 64 else 2)
    ws = []

    def prefill(pk):
        _stale_words(pk["workspace"])
        ws.append(pk["workspace"])
    _assert_exact(compare_full(w, K, V, mask, prefill=prefill), w.name)
    outcome = int(ws[0][16:24].cpu().numpy().view(np.uint64)[0])
    assert outcome == (0 if T > 256 * capacity(D) else 2 if absent else 1)


@pytest.mark.parametrize("T,H", [(65536, 4), (98305, 3), (131072, 1)])
@pytest.mark.parametrize("inplace", [False, True])
@pytest.mark.parametrize("absent", ["", "1"])
def test_spread_groups_fake(T, H, inplace, absent, monkeypatch):
    monkeypatch.setenv("HG_TEST_ABSENT", absent)
    w, K, V, mask = _spread_workload(128, T, H)
    check_fake(w, K, V, mask, inplace, prefill_ws=_stale_words)


def test_spread_groups_share_the_chip():
    """Two calls whose grids each want every compute unit, on two streams: the
    roll call of either may find workgroups missing and leave its work to the
    split kernels; the packed bytes are those of a call alone."""
    import paper_2609_35800_amd as hg
    w, K, V, mask = _spread_workload(128, 65536, 4)
    cfg = hg.make_config(**w.config_fields())
    Kg, Vg = K.cuda(), V.cuda()
    want = hg.alloc_packed(cfg, mask)
    hg.hg_quantize(cfg, Kg, Vg, mask, want)
    packed = [hg.alloc_packed(cfg, mask) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(4):
        for s, pk in zip(streams, packed):
            hg.hg_quantize(cfg, Kg, Vg, mask, pk, stream=s)
    torch.cuda.synchronize()
    for pk in packed:
        assert int(pk["workspace"][:8].view(torch.int64)[0]) == 0
        assert all(torch.equal(pk[n], want[n]) for n in hg.BUFFERS)


# Groups whose partners are not all on the chip: the ones that are close the
# group and take its slices one workgroup a slice.  HG_TEST_ABSENT leaves the last
# partners of the last eight groups out of the launch (several slices a group on
# the small grids); the workspace's fourth word counts the partners closed.
def _group_workload(D, T, H=11, B=2, bits=2):
    w = small("kivi", D, bits, 1, img_len=T - 90, img_start=30, text=60, L=1, B=B, H=H,
              n_protected=1).with_(kivi_group=0, name=f"kiviseq-groups-D{D}-T{T}")
    K, V = synthkv.gen_kv(w)
    K[0, :, :, T - 1, 5] = -4000.0  # extremes in the last and first rows
    K[0, :, :, 0, 9] = 5000.0
    return w, K, V, synthkv.protect_mask(w)


ABSENT_CASES = [(128, "", 1600, "1"), (128, "32", 1700, "1"), (128, "32", 4000, "2"), (128, "", 3008, "7"),
                (64, "16", 4000, "1"), (64, "128", 30000, "15"), (256, "", 1000, "3"), (256, "128", 7000, "1"),
                (256, "", 20000, "31")]


@pytest.mark.parametrize("D,cus,T,absent", ABSENT_CASES, ids=lambda v: str(v) or "all")
def test_absent_partners(D, cus, T, absent, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", cus)
    monkeypatch.setenv("HG_TEST_ABSENT", absent)
    w, K, V, mask = _group_workload(D, T, bits=3 if D == 64 else 2)
    ws = []

    def prefill(pk):
        _stale_words(pk["workspace"])
        ws.append(pk["workspace"])
    _assert_exact(compare_full(w, K, V, mask, prefill=prefill), w.name)
    assert int(ws[0][24:32].view(torch.int64)[0]) > 0


@pytest.mark.parametrize("D,cus,T,absent", ABSENT_CASES[:4] + ABSENT_CASES[7:], ids=lambda v: str(v) or "all")
@pytest.mark.parametrize("inplace", [False, True])
def test_absent_partners_fake(D, cus, T, absent, inplace, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", cus)
    monkeypatch.setenv("HG_TEST_ABSENT", absent)
    w, K, V, mask = _group_workload(D, T)
    check_fake(w, K, V, mask, inplace, prefill_ws=_stale_words)


@pytest.mark.parametrize("T,cus", [(1600, "32"), (3008, ""), (13000, ""), (40000, "")])
def test_closing_beside_arrivals(T, cus, monkeypatch):
    """Groups closed by the first partner that would have to wait, others still
    arriving: whichever come first, in place and packed, the bytes are those of
    a call alone."""
    import paper_2609_35800_amd as hg
    w, K, V, mask = _group_workload(128, T)
    monkeypatch.setenv("HG_TEST_CUS", cus)
    cfg = hg.make_config(**w.config_fields())
    Kg, Vg = K.cuda(), V.cuda()
    want, got = hg.alloc_packed(cfg, mask), hg.alloc_packed(cfg, mask)
    ws = hg.alloc_fake_workspace(cfg, mask)
    hg.hg_quantize(cfg, Kg, Vg, mask, want)
    Kw, Vw = torch.clone(Kg), torch.clone(Vg)
    hg.hg_fake_quantize(cfg, Kg, Vg, mask, Kw, Vw, ws)
    monkeypatch.setenv("HG_TEST_POLLS", "0")
    for _ in range(6):
        hg.hg_quantize(cfg, Kg, Vg, mask, got)
        assert all(torch.equal(got[n], want[n]) for n in hg.BUFFERS)
        Ki, Vi = torch.clone(Kg), torch.clone(Vg)
        hg.hg_fake_quantize(cfg, Ki, Vi, mask, Ki, Vi, ws)
        assert torch.equal(Ki, Kw) and torch.equal(Vi, Vw)


@pytest.mark.parametrize("T,H", [(3008, 29), (13000, 13), (40000, 9)])
def test_groups_share_the_chip(T, H):
    """Calls with groups of 8, 16 and 32 workgroups, each wanting every compute
    unit, on four streams at once: the bytes are those of a call alone and no
    wait runs out."""
    import paper_2609_35800_amd as hg
    w, K, V, mask = _group_workload(128, T, H=H, B=1)
    cfg = hg.make_config(**w.config_fields())
    Kg, Vg = K.cuda(), V.cuda()
    want = hg.alloc_packed(cfg, mask)
    hg.hg_quantize(cfg, Kg, Vg, mask, want)
    packed = [hg.alloc_packed(cfg, mask) for _ in range(4)]
    streams = [torch.cuda.Stream() for _ in packed]
    torch.cuda.synchronize()
    for _ in range(4):
        for s, pk in zip(streams, packed):
            hg.hg_quantize(cfg, Kg, Vg, mask, pk, stream=s)
    torch.cuda.synchronize()
    for pk in packed:
        assert int(pk["workspace"][:8].view(torch.int64)[0]) == 0
        assert all(torch.equal(pk[n], want[n]) for n in hg.BUFFERS)


@pytest.mark.parametrize("which", ["none", "all", "last"])
@pytest.mark.parametrize("keys_only", [0, 1])
def test_degenerate_masks(which, keys_only):
    """No key head protected, every one (no work item for the key kernel),
    and only the last head quantized (the rank search lands in the last word)."""
    w = small("kivi", 128, 2, keys_only, img_len=90, img_start=5, text=9, L=3, B=2, H=12,
              n_protected=0).with_(kivi_group=0)
    K, V = synthkv.gen_kv(w)
    mask = np.full(w.L * w.H, 1 if which != "none" else 0, np.uint8)
    if which == "last":
        mask[-1] = 0
    _assert_exact(compare_full(w, K, V, mask), f"mask-{which}-ko{keys_only}")


def _stale_words(ws):
    """Every 64-bit word of an exchange workspace set to what a partner would
    fold in if the words were not cleared before the key kernel: a small
    sequence tag (1 to 8, the first slices' tags) above the BF16 bits of the
    range [-1000, 1000]."""
    n = ws.numel() // 8
    tags = (np.arange(n, dtype=np.uint64) % np.uint64(8)) + np.uint64(1)
    words = (tags << np.uint64(32)) | (np.uint64(0x447A) << np.uint64(16)) | np.uint64(0xC47A)
    ws[: n * 8].copy_(torch.from_numpy(words.view(np.uint8)).to(ws.device))


# Two workgroups per slice (head_dim 128), 2-bit, keys and values quantized.
STALE_CASE = next(w for w in STREAM_CASES
                  if w.D == 128 and w.T == capacity(128) + 300 and w.bits == 2 and not w.keys_only)


# Resident kernel with several slices per group (32 and 256 compute units'
# grids) and the split kernels (8), every call on a workspace holding
# stale tagged words: the call must clear them before the key kernel reads.
@pytest.mark.parametrize("cus", ["32", "", "8"])
def test_stale_exchange_words(cus, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", cus)
    w = STALE_CASE
    K, V = synthkv.gen_kv(w)
    prefill = lambda pk: _stale_words(pk["workspace"])  # noqa: E731
    _assert_exact(compare_full(w, K, V, synthkv.protect_mask(w), prefill=prefill), f"stale-cus{cus or 'all'}")


@pytest.mark.parametrize("inplace", [False, True])
def test_stale_exchange_words_fake(inplace, monkeypatch):
    monkeypatch.setenv("HG_TEST_CUS", "32")
    w = STALE_CASE
    K, V = synthkv.gen_kv(w)
    check_fake(w, K, V, synthkv.protect_mask(w), inplace, prefill_ws=_stale_words)
