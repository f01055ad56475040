"""The mask routes' kernels at the sizes where their rules change: contexts
around and past one workgroup's panel (131,072 positions), rows off the
16-byte grid, bins narrower than a thread's 16 positions, and packed lengths
at the edges of the copy's 8 KiB chunks.  Whole numbers and bytes: exact."""

import numpy as np
import pytest
import torch

import oracle as o

pytestmark = pytest.mark.gpu

DEV = "cuda"


@pytest.fixture(scope="module")
def d():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2609_32663_amd as lib
    return lib


def _mask(nseg, T, seed):
    """Long runs and scattered positions, an empty and a full row among them."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    runs = (torch.rand((nseg, (T + 96) // 97), generator=g, device=DEV) < 0.5).to(torch.uint8)
    m = runs.repeat_interleave(97, dim=1)[:, :T].clone()
    m[1::3] &= (torch.rand((m[1::3].shape[0], T), generator=g, device=DEV) < 0.9).to(torch.uint8)
    m[0], m[-1] = 0, 7  # any nonzero byte is kept
    return m.contiguous()


def _select(d, mask, page_rows, cap, pages, bound):
    nseg, T = mask.shape
    table = torch.arange(nseg * pages, device=DEV, dtype=torch.int32).flip(0).reshape(nseg, pages).contiguous()
    ent = torch.full((nseg, bound, 4), -5, dtype=torch.int32, device=DEV)
    n, ln = (torch.full((nseg,), -5, dtype=torch.int32, device=DEV) for _ in range(2))
    used = torch.full((nseg, pages), 9, dtype=torch.uint8, device=DEV)
    ws = torch.empty(max(d.dkv_page_select_workspace_bytes(nseg, T), 16), dtype=torch.uint8, device=DEV)
    d.dkv_page_select(mask, table, page_rows, cap, ent, n, ln, ws, page_used=used)
    return table.cpu().numpy(), ent.cpu().numpy(), n.cpu().numpy(), ln.cpu().numpy(), used.cpu().numpy()


@pytest.mark.parametrize("nseg,T,page_rows,cap", [(64, 131072, 32, 37), (64, 131077, 32, 0), (72, 290001, 128, 300),
                                                  (40, 163840, 64, 1), (40, 163841, 64, 1), (4, 32768, 32, 5),
                                                  (4, 32769, 32, 5), (3, 17, 32, 40), (256, 10240, 64, 3),
                                                  (256, 10241, 64, 3), (257, 10240, 64, 3), (257, 32768, 128, 9),
                                                  (257, 32767, 128, 9), (512, 24000, 128, 9), (512, 23999, 128, 9),
                                                  (513, 24000, 128, 9), (64, 262144, 1024, 7), (64, 262145, 1024, 7),
                                                  (63, 131072, 1024, 7)])
def test_page_select_panels(d, nseg, T, page_rows, cap):
    """One panel, two and three, and either side of the rule that sends a call
    to the tile passes, against the oracle."""
    mask = _mask(nseg, T, nseg + T)
    pages = -(-(T + cap) // page_rows) + 2
    few = mask[[0, 1, nseg // 2, nseg - 1]]
    bound = T // 8 + pages + 8
    table, ent, n, ln, used = _select(d, mask, page_rows, cap, pages, bound)
    pick = [0, 1, nseg // 2, nseg - 1]
    want = o.page_select((few.cpu().numpy() != 0).astype(np.uint8), table[pick], page_rows, cap)
    for i, s in enumerate(pick):
        e = np.asarray(want["entries"][i]).reshape(-1, 4)
        assert n[s] == len(e) <= bound
        np.testing.assert_array_equal(ent[s, :len(e)], e)
        assert (ent[s, len(e):] == -5).all()
        assert ln[s] == want["seg_len"][i]
        np.testing.assert_array_equal(used[s], want["page_used"][i])


@pytest.mark.parametrize("nseg,T", [(5, 16384), (5, 20001), (130, 131072), (300, 33333)])
def test_page_select_bound_rule(d, nseg, T):
    """The caller's bound on the entries chooses between the whole-row kernel
    and the tile passes: a quarter of the positions, one more, and bounds below
    the entries there are (the first ones written, the true number reported)
    give the same outputs."""
    mask = _mask(nseg, T, T)
    pages = -(-(T + 5) // 64)
    first = None
    for bound in (T // 4, T // 4 + 1, T // 2, 200):
        _, ent, n, ln, used = _select(d, mask, 64, 5, pages, bound)
        if first is None:
            first = (ent, n, ln, used)
            assert n.max() > 200
        keep = min(bound, T // 4)
        for s in range(nseg):
            m = min(int(n[s]), keep)
            np.testing.assert_array_equal(ent[s, :m], first[0][s, :m])
            assert (ent[s, min(int(n[s]), bound):] == -5).all()
        for a, b in zip((n, ln, used), first[1:]):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("nseg,T,dim,dtype", [(64, 131085, 64, torch.bfloat16), (2, 131080, 64, torch.float32),
                                              (2, 32768, 128, torch.float32), (3, 32769, 128, torch.bfloat16),
                                              (33, 133333, 64, torch.bfloat16), (3, 9001, 128, torch.bfloat16),
                                              (3, 16383, 64, torch.bfloat16), (3, 16384, 64, torch.bfloat16),
                                              (3, 16385, 64, torch.bfloat16), (1024, 1023, 64, torch.bfloat16),
                                              (1025, 1023, 64, torch.bfloat16), (1024, 1040, 64, torch.bfloat16),
                                              (127, 33000, 64, torch.bfloat16), (128, 33001, 64, torch.bfloat16),
                                              (128, 32784, 64, torch.bfloat16), (1025, 4096, 64, torch.bfloat16),
                                              (1025, 4095, 64, torch.bfloat16), (128, 131072, 64, torch.bfloat16),
                                              (2, 131072, 128, torch.float32), (2, 131073, 128, torch.float32)])
def test_compact_panels(d, nseg, T, dim, dtype):
    mask = _mask(nseg, T, T)
    k = torch.randn((1, nseg, T, dim), device=DEV).to(dtype)
    v = -k
    lay = d.make_layout(1, nseg, nseg, dim, T, 0, 0, [0, T])
    cap = 3
    lens = (mask != 0).sum(dim=1)
    rows = int(lens.sum()) + nseg * cap
    ko, vo = torch.zeros((rows, dim), dtype=dtype, device=DEV), torch.zeros((rows, dim), dtype=dtype, device=DEV)
    off, ln = torch.empty(nseg, dtype=torch.int64, device=DEV), torch.empty(nseg, dtype=torch.int32, device=DEV)
    src = torch.full((rows,), -1, dtype=torch.int32, device=DEV)
    ws = torch.empty(d.dkv_compact_workspace_bytes(lay), dtype=torch.uint8, device=DEV)
    d.dkv_compact(lay, k, v, mask, cap, ko, vo, off, ln, ws, src_pos=src)
    assert torch.equal(ln.long(), lens)
    assert torch.equal(off, torch.cumsum(lens + cap, 0) - lens - cap)
    for s in range(0, nseg, max(1, nseg // 5)):
        pos = torch.nonzero(mask[s])[:, 0]
        a, n = int(off[s]), int(lens[s])
        assert torch.equal(src[a:a + n].long(), pos)
        assert torch.equal(ko[a:a + n], k[0, s, pos]) and torch.equal(vo[a:a + n], v[0, s, pos])
        assert (src[a + n:a + n + cap] == -1).all()


@pytest.mark.parametrize("dim,dtype", [(64, torch.bfloat16), (64, torch.float32), (128, torch.bfloat16),
                                       (128, torch.float32)])
def test_copy_chunk_edges(d, dim, dtype):
    """Kept lengths around 16, 32, 64 and 128 rows, and around the 112 from
    which workgroups move a second chunk of 512-byte rows, by mask and as a block
    gather (bins of one position: a chunk spans as many ranges as rows)."""
    lens = [0, 1, 15, 16, 17, 31, 33, 63, 64, 65, 111, 112, 113, 127, 128, 129, 190, 207, 208, 209, 211]
    T, cap, nseg = 211, 2, len(lens)
    rng = np.random.default_rng(dim)
    pat = np.zeros((1, nseg, T), dtype=np.uint8)
    for s, n in enumerate(lens):
        pat[0, s, rng.choice(T, n, replace=False)] = 1
    mask = torch.from_numpy(pat[0, :, ::-1].copy()).to(DEV)  # bin u is position T - 1 - u
    k = torch.randn((1, nseg, T, dim), device=DEV).to(dtype)
    lay = d.make_layout(1, nseg, nseg, dim, T, 0, 0, list(range(T + 1)))
    rows = sum(lens) + nseg * cap
    got = []
    for bins in (False, True):
        ko, vo = torch.zeros((rows, dim), dtype=dtype, device=DEV), torch.zeros((rows, dim), dtype=dtype, device=DEV)
        off, ln = torch.empty(nseg, dtype=torch.int64, device=DEV), torch.empty(nseg, dtype=torch.int32, device=DEV)
        f, w = ((d.dkv_compact_bins, d.dkv_compact_bins_workspace_bytes) if bins else
                (d.dkv_compact, d.dkv_compact_workspace_bytes))
        ws = torch.empty(w(lay), dtype=torch.uint8, device=DEV)
        f(lay, k, k, torch.from_numpy(pat).to(DEV) if bins else mask, cap, ko, vo, off, ln, ws)
        assert ln.tolist() == lens
        for s, n in enumerate(lens):
            a = int(off[s])
            want = k[0, s, torch.nonzero(mask[s])[:, 0]]
            assert torch.equal(ko[a:a + n], want) and torch.equal(vo[a:a + n], want)
        got.append(ko)
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("T", [1, 15, 16, 17, 250, 256, 4099, 16400])
@pytest.mark.parametrize("width", [1, 2, 5, 15, 16, 40, None])
def test_map_regions(d, T, width):
    """Bins narrower than a run of 16 positions, rows off the 16-byte grid,
    units of every length, edges that end before, at and past the context."""
    rng = np.random.default_rng([T, width or 0])
    S, R = (0, 0) if T < 16 else (int(rng.integers(0, 20)), int(rng.integers(0, 30)))
    if width is None:
        edges = np.concatenate([[0], np.cumsum(rng.integers(1, 9, size=min(500, T + 3)))]).tolist()
    else:
        edges = [width * i for i in range(max(2, min(400, T // width + int(rng.integers(0, 3)))))]
    N, Hkv, G, D = 3, 2, 3, len(edges) - 1
    pat = (rng.random((N, Hkv * G, D)) < 0.3).astype(np.uint8)
    ulen = np.array([T, max(0, T - 3), T // 2], dtype=np.int32)
    lay = d.make_layout(N, Hkv * G, Hkv, 64, T, S, R, edges)
    for ragged in (False, True):
        kv = torch.full((N, Hkv, T), 9, dtype=torch.uint8, device=DEV)
        qm = torch.full((N, Hkv * G, T), 9, dtype=torch.uint8, device=DEV)
        ln = torch.empty((N, Hkv), dtype=torch.int32, device=DEV)
        pt = torch.from_numpy(pat).to(DEV)
        if ragged:
            d.dkv_map_pattern_ragged(lay, torch.from_numpy(ulen).to(DEV), pt, kv, ln, q_mask=qm)
        else:
            d.dkv_map_pattern(lay, pt, kv, ln, q_mask=qm)
        want_q = np.zeros((N, Hkv * G, T), dtype=np.uint8)
        for n in range(N):
            t = int(ulen[n]) if ragged else T
            for j in range(t):
                u = t - 1 - j - R
                if j < S or u < 0:
                    want_q[n, :, j] = 1
                elif u < edges[-1]:
                    want_q[n, :, j] = pat[n, :, np.searchsorted(edges, u, side="right") - 1]
        want = want_q.reshape(N, Hkv, G, T).max(axis=2)
        np.testing.assert_array_equal(qm.cpu().numpy(), want_q)
        np.testing.assert_array_equal(kv.cpu().numpy(), want)
        np.testing.assert_array_equal(ln.cpu().numpy(), want.sum(axis=2))


@pytest.mark.parametrize("T", [(1 << 31) - 32, (1 << 31) - 17])
def test_map_longest_contexts(d, T):
    """The longest rows the map accepts, on and off the 16-byte grid: the last
    sweep ends within 32 positions of the largest int32."""
    S, R, W, D = 100, 1000, (1 << 17) - 1, 16384  # the last positions lie past the last bin
    rng = np.random.default_rng(T & 0xFF)
    pat = torch.from_numpy((rng.random((1, 2, D)) < 0.5).astype(np.uint8)).to(DEV)
    lay = d.make_layout(1, 2, 2, 128, T, S, R, [W * i for i in range(D + 1)])
    mask = torch.full((1, 2, T), 9, dtype=torch.uint8, device=DEV)
    n = torch.zeros((1, 2), dtype=torch.int32, device=DEV)
    d.dkv_map_pattern(lay, pat, mask, n)
    for h in range(2):
        kept = 0
        for lo in range(0, T, 1 << 27):
            j = torch.arange(lo, min(T, lo + (1 << 27)), dtype=torch.int64, device=DEV)
            delta = T - 1 - j
            u = (delta - R).clamp_(min=0)
            want = pat[0, h][(u // W).clamp_(max=D - 1)].to(torch.bool) & (u < W * D)
            want |= (j < S) | (delta < R)
            assert torch.equal(mask[0, h, lo:lo + len(j)], want.to(torch.uint8)), (h, lo)
            kept += int(want.sum())
        assert int(n[0, h]) == kept


@pytest.mark.parametrize("G", [1, 2, 3, 4, 5, 8, 9, 16])
@pytest.mark.parametrize("T,width", [(37, 1), (4099, 2), (4099, 3), (4112, 1), (4112, 17), (16400, 300), (2049, 5)])
def test_map_heads(d, G, T, width):
    """Every group size's masks per query head (the loads of the group's rows
    come in batches), with and without the per-head output, runs of one, two
    and more regions."""
    rng = np.random.default_rng([G, T, width])
    Hkv, S, R = 2, 5, 11
    edges = [width * i for i in range(max(2, T // width - 20))]
    pat = (rng.random((2, Hkv * G, len(edges) - 1)) < 0.3).astype(np.uint8)
    lay = d.make_layout(2, Hkv * G, Hkv, 64, T, S, R, edges)
    pt = torch.from_numpy(pat).to(DEV)
    kv, kv2 = (torch.full((2, Hkv, T), 9, dtype=torch.uint8, device=DEV) for _ in range(2))
    room = 64  # bytes behind the last head's row, which no store may touch
    qm = torch.full((2 * Hkv * G * T + room,), 9, dtype=torch.uint8, device=DEV)
    ln, ln2 = (torch.empty((2, Hkv), dtype=torch.int32, device=DEV) for _ in range(2))
    d.dkv_map_pattern(lay, pt, kv, ln, q_mask=qm[:-room].view(2, Hkv * G, T))
    d.dkv_map_pattern(lay, pt, kv2, ln2)
    want_q, want, want_len = o.map_pattern(pat, T, S, R, edges, Hkv)
    np.testing.assert_array_equal(qm[:-room].cpu().numpy().reshape(2, Hkv * G, T), want_q)
    assert (qm[-room:] == 9).all()
    for got, n in ((kv, ln), (kv2, ln2)):
        np.testing.assert_array_equal(got.cpu().numpy(), want)
        np.testing.assert_array_equal(n.cpu().numpy(), want_len)


@pytest.mark.parametrize("G", [1, 3, 8])
@pytest.mark.parametrize("T,D,span", [(17, 6, 17), (700, 340, 690), (1500, 500, 1100), (1500, 500, 760),
                                      (1504, 240, 1440), (1504, 240, 1441), (2049, 512, 1024),
                                      (2049, 512, 1025), (3000, 512, 3000)])
def test_map_narrow_unequal_bins(d, G, T, D, span):
    """Narrow bins of unequal widths, with a head's mask or without: either side
    of the rule that walks them position by position (six positions on average,
    half the row covered), uncovered ends, and contexts shorter than the row."""
    rng = np.random.default_rng([G, T, D, span])
    edges = [0] + sorted(rng.choice(np.arange(1, span), D - 1, replace=False).tolist()) + [span]
    Hkv, S, R = 2, 3, 7
    lens = np.array([T, T - 5, 0, T // 3], dtype=np.int32)
    pat = (rng.random((4, Hkv * G, D)) < 0.4).astype(np.uint8)
    lay = d.make_layout(4, Hkv * G, Hkv, 64, T, S, R, edges)
    kv = torch.full((4, Hkv, T), 9, dtype=torch.uint8, device=DEV)
    qm = torch.full((4, Hkv * G, T), 9, dtype=torch.uint8, device=DEV)
    n = torch.empty((4, Hkv), dtype=torch.int32, device=DEV)
    d.dkv_map_pattern_ragged(lay, torch.from_numpy(lens).to(DEV), torch.from_numpy(pat).to(DEV), kv, n, qm)
    want_q, want, want_len = o.map_pattern(pat, T, S, R, edges, Hkv, unit_len=lens)
    np.testing.assert_array_equal(qm.cpu().numpy(), want_q)
    np.testing.assert_array_equal(kv.cpu().numpy(), want)
    np.testing.assert_array_equal(n.cpu().numpy(), want_len)


@pytest.mark.parametrize("dim,dtype,T", [(64, torch.bfloat16, 1024), (64, torch.bfloat16, 4096), (64, torch.bfloat16, 4097),
                                         (128, torch.bfloat16, 128), (128, torch.bfloat16, 2048), (128, torch.float32, 64),
                                         (128, torch.float32, 1024), (128, torch.float32, 100)])
@pytest.mark.parametrize("nseg", [63, 64, 65])
def test_pack_grids_of_many_segments(d, dim, dtype, T, nseg):
    """Either side of the rule that gives every segment one idle workgroup more
    (64 segments, 128 workgroups a segment, a multiple of four), with full,
    empty and partly kept segments: the mask pack and the block gather of the
    same rows agree with each other and with the rows picked by the mask."""
    rng = np.random.default_rng([dim, T, nseg])
    edges = [0, T // 4, T // 2, T - T // 4, T]
    pat = (rng.random((nseg, 1, 4)) < 0.5).astype(np.uint8)
    pat[0], pat[-1] = 1, 0
    lay = d.make_layout(nseg, 1, 1, dim, T, 0, 0, edges)
    k, v = (torch.randn((nseg, 1, T, dim), device=DEV).to(dtype) for _ in range(2))
    pt = torch.from_numpy(pat).to(DEV)
    mask = torch.empty((nseg, 1, T), dtype=torch.uint8, device=DEV)
    kl = torch.empty((nseg, 1), dtype=torch.int32, device=DEV)
    d.dkv_map_pattern(lay, pt, mask, kl)
    rows = int(kl.sum()) + 3 * nseg
    keep = mask[:, 0].bool()
    lens = kl[:, 0].long()
    off = torch.cumsum(lens + 3, 0) - (lens + 3)
    at = torch.cat([off[s] + torch.arange(int(lens[s]), device=DEV) for s in range(nseg)])
    for bins in (False, True):
        ko, vo = (torch.full((rows, dim), 7.0, dtype=dtype, device=DEV) for _ in range(2))
        so, sl = torch.empty(nseg, dtype=torch.int64, device=DEV), torch.empty(nseg, dtype=torch.int32, device=DEV)
        if bins:
            ws = torch.empty(max(16, d.dkv_compact_bins_workspace_bytes(lay)), dtype=torch.uint8, device=DEV)
            d.dkv_compact_bins(lay, k, v, pt, 3, ko, vo, so, sl, ws)
        else:
            ws = torch.empty(d.dkv_compact_workspace_bytes(lay), dtype=torch.uint8, device=DEV)
            d.dkv_compact(lay, k, v, mask, 3, ko, vo, so, sl, ws)
        assert torch.equal(so, off) and torch.equal(sl.long(), lens)
        for got, src in ((ko, k), (vo, v)):
            want = torch.full((rows, dim), 7.0, dtype=dtype, device=DEV)
            want[at] = src[:, 0][keep]
            assert torch.equal(got, want)
