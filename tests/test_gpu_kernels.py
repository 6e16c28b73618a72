"""GPU tests of single kernels at the sizes where their splits and dispatch
rules can go wrong: remainders of tiles, the smallest and largest of a range,
misaligned buffers; each against the same operation in float64."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

DEV = "cuda"


def _offset_copy(t, by):
    """A contiguous copy of t whose first element lies `by` elements into its buffer."""
    buf = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
    v = buf[by:].view(t.shape)
    v.copy_(t)
    return v


# channel counts: one per lane (odd, or not a multiple of 16 bytes), whole 16-byte groups, more
# groups than a block has threads; rows: fewer than one chunk, chunk remainders, several chunks a block
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,c,shift", [(1, 1, 0), (63, 7, 0), (65, 16, 0), (1000, 48, 0), (1000, 48, 1), (777, 264, 0),
                                       (130, 2080, 0), (70001, 64, 0)])
def test_affine_act_bwd_shapes(dtype, n, c, shift):
    from paper_1904_08755_amd import gsc
    g = torch.Generator(DEV).manual_seed(n * 31 + c)
    scale = 0.5 + torch.rand(c, generator=g, device=DEV)
    if c > 4:
        scale[1] = 0.0
    sh = 0.3 * torch.randn(c, generator=g, device=DEV)
    S = torch.randn((n, c), generator=g, device=DEV)
    Y = _offset_copy(torch.clamp(S * scale + sh, min=0).to(dtype), shift)
    dY = _offset_copy(torch.randn((n, c), generator=g, device=DEV).to(dtype), shift)
    dZ, ds, dt = gsc.gsc_affine_act_bwd(Y, dY, scale, sh, relu=True)
    y, gr, sc, s0 = Y.double(), dY.double(), scale.double(), sh.double()
    G = torch.where(y > 0, gr, 0.0)
    # the product in float32 (half an ulp), rounded to the dtype (half an ulp)
    eps = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -23
    assert ((dZ.double() - G * sc).abs() <= (G * sc).abs() * eps + 1e-40).all()
    # sums: at most rows-per-lane + lanes float32 additions, each within 2^-24 of the sum of magnitudes
    bound = (n + 512) * 2.0 ** -24
    assert ((dt.double() - G.sum(0)).abs() <= G.abs().sum(0) * bound + 1e-30).all()
    ok = scale != 0
    z = (y - s0)[:, ok] / sc[ok]
    zmag = (G[:, ok].abs() * (y.abs() + s0.abs())[:, ok] / sc[ok]).sum(0)
    assert ((ds.double()[ok] - (G[:, ok] * z).sum(0)).abs() <= zmag * (bound + 2.0 ** -22) + 1e-30).all()
    if c > 4:   # a channel with scale 0: not finite when a row counts, 0 when none does
        counts = bool((G[:, 1] != 0).any())
        assert torch.isfinite(ds[1]).item() != counts
    again = gsc.gsc_affine_act_bwd(Y, dY, scale, sh, relu=True)
    assert torch.equal(again[1].nan_to_num(7.0), ds.nan_to_num(7.0)) and torch.equal(again[2], dt)


# scales whose quotients are ordinary numbers while their products with a gradient leave float32's range: decayed and
# grown ones, the smallest normal, a subnormal, the largest binade; and those with no quotient
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_affine_act_bwd_scale_range(dtype):
    from paper_1904_08755_amd import gsc
    inf = float("inf")
    scale = torch.tensor([1e-30, -1e-30, 1e30, -3e38, 2.0 ** -126, 1e-40, 1.0, -0.75, 0.0, -0.0, inf, float("nan")],
                         device=DEV)
    n, c = 700, len(scale)
    g = torch.Generator(DEV).manual_seed(3)
    Z = torch.randn((n, c), generator=g, device=DEV).clamp(-0.9, 0.9)   # (0.9 x 3e38 stays finite)
    Y = torch.where(torch.isfinite(scale), Z * scale, Z).to(dtype)
    Y[:, 8:10] = 0.5   # (y - shift) / 0 is infinite
    dY = (1e-16 * torch.randn((n, c), generator=g, device=DEV)).to(dtype)
    dY[:, 9] = dY[:, 9].abs()
    _, ds, dt = gsc.gsc_affine_act_bwd(Y, dY, scale)
    y, gr = Y[:, :8].double(), dY[:, :8].double()
    z = y / scale[:8].double()
    bound = (n + 512) * 2.0 ** -24
    assert ((ds[:8].double() - (gr * z).sum(0)).abs() <= (gr * z).abs().sum(0) * (bound + 2.0 ** -22)).all()
    assert ((dt.double() - dY.double().sum(0)).abs() <= dY.double().abs().sum(0) * bound).all()
    # sums of infinities of both signs, of one sign, of zeros, of NaN
    assert torch.isnan(ds[8]) and ds[9] == -inf and ds[10] == 0 and torch.isnan(ds[11])
    # rows that do not count add nothing to any of them
    assert (gsc.gsc_affine_act_bwd(Y, torch.zeros_like(dY), scale)[1] == 0).all()


# --------------------------------------------------------------------------- #
# the two forms of a coordinate table: grid and hashed slots
# --------------------------------------------------------------------------- #
def _pairs(src, dst, offs):
    """(input row, output row) per offset from a dict of rows."""
    at = {tuple(r): i for i, r in enumerate(src.tolist())}
    out = []
    for o in np.asarray(offs).tolist():
        hit = [(at.get((r[0],) + tuple(a + b for a, b in zip(r[1:], o))), j) for j, r in enumerate(dst.tolist())]
        out.append([(i, j) for i, j in hit if i is not None])
    return out


def _rows(seed, n, D, span, step=1, lo=-7, batch=2):
    rng = np.random.default_rng(seed)
    r = np.concatenate([rng.integers(0, batch, (4 * n, 1)), lo + step * rng.integers(0, span, (4 * n, D))], 1)
    r = np.unique(r, axis=0)
    return np.ascontiguousarray(rng.permutation(r)[:n].astype(np.int32))


GRID_ROWS = {
    "one_row": np.array([[3, -5, 7, 11]], np.int32),
    "line_1d": _rows(1, 130, 1, 400),
    "plane_2d": _rows(2, 257, 2, 40),
    "sparse_3d": _rows(3, 1025, 3, 40),
    "step2_3d": _rows(4, 700, 3, 20, step=2, lo=-8),
    "step4_wide_3d": _rows(5, 333, 3, 30, step=4, lo=1 << 28),
    "video_4d": _rows(6, 500, 4, 9),
    "sorted_run": np.array([[0, 0, y, z] for y in range(3) for z in range(70)], np.int32),
    "low_end": np.array([[0, -2**31, 0, 0], [0, -2**31 + 1, 0, 1], [1, -2**31, 1, 0]], np.int32),
    "split_box": np.array([[0, -2**29, 0, 0], [0, 2**29, 0, 0], [0, 2**29, 0, 1]], np.int32),   # hashed: too wide
    "five_5d": _rows(7, 200, 5, 4),
    "seven_7d": _rows(8, 300, 7, 3),
    # past the rows that one block builds a table of
    "block_3d": _rows(9, 3072, 3, 40),
    "past_block_3d": _rows(10, 3073, 3, 40),
    "big_line_1d": _rows(11, 5000, 1, 9000),
    "big_step2_3d": _rows(12, 4100, 3, 30, step=2, lo=-8),
    "big_video_4d": _rows(13, 3500, 4, 10),
    "big_wide_3d": _rows(14, 4000, 3, 900, step=4, lo=1 << 28),   # hashed: too many cells
    "big_seven_7d": _rows(15, 3300, 7, 4),
}


@pytest.mark.parametrize("form", ["any", "hash"])
@pytest.mark.parametrize("name", sorted(GRID_ROWS))
def test_table_forms(name, form, monkeypatch):
    """Kernel maps onto the rows themselves (cube 3, and cube 3 at twice the
    step), onto other rows (some far outside the box) and strided rows, from
    the form that the box gives and from hashed slots, against a dict."""
    from paper_1904_08755_amd import gsc, regions
    if form == "hash":
        monkeypatch.setenv("GSC_TABLE_CAP_LIMIT", str(1 << 40))
    host = GRID_ROWS[name]
    D = host.shape[1] - 1
    c = torch.from_numpy(host).to(DEV)
    table = gsc.gsc_coords_build(c)
    offs = regions.hypercube(3, D) if D <= 4 else regions.hypercross(3, D)
    step = 4 if "step4" in name else (2 if "step2" in name else 1)
    rng = np.random.default_rng(11)
    other = host[rng.integers(0, len(host), 90)].astype(np.int64)
    other[:, 1:] += rng.integers(-3, 4, other[:, 1:].shape)
    far = np.array([[0] + [2**31 - 1] * D, [0] + [-2**31] * D, [-2**31] + [0] * D, [2**31 - 1] + [0] * D])
    other = np.concatenate([other.clip(-2**31, 2**31 - 1), far]).astype(np.int32)
    for dst, ts in ((host, 1), (host, step), (host[::-1].copy(), step), (other, 1)):
        km = gsc.gsc_kernel_map(table, torch.from_numpy(dst).to(DEV), offs, tensor_stride=ts, dense=True)
        seg = km.seg.cpu().numpy()
        got_i, got_o, nbr = km.in_idx.cpu().numpy(), km.out_idx.cpu().numpy(), km.nbr.cpu().numpy()
        gidx = km.gidx.cpu().numpy()
        G = gsc.gsc_kmap_groups(len(dst))
        for k, pairs in enumerate(_pairs(host.astype(np.int64), dst.astype(np.int64), offs.astype(np.int64) * ts)):
            i, o = got_i[seg[k]:seg[k + 1]], got_o[seg[k]:seg[k + 1]]
            assert list(zip(i.tolist(), o.tolist())) == pairs, (name, k)
            dense = np.full(len(dst), -1)
            dense[o] = i
            assert (nbr[k] == dense).all()
            assert (gidx[k * G:(k + 1) * G] == seg[k] + np.searchsorted(o, 64 * np.arange(G))).all()
        assert gidx[-1] == seg[-1] == km.n_pairs
    if name in ("low_end", "split_box"):   # a strided value may leave int32 there
        return
    for s in (2, 3):
        out, out_table = gsc.gsc_coords_stride(c, s)
        want = host.astype(np.int64).copy()
        want[:, 1:] = want[:, 1:] // s * s
        seen = list(dict.fromkeys(tuple(r) for r in want.tolist()))
        assert [tuple(r) for r in out.cpu().tolist()] == seen
        up = gsc.gsc_kernel_map(out_table, out, np.zeros((1, D), np.int32))
        assert up.in_idx.cpu().tolist() == list(range(len(seen)))


@pytest.mark.parametrize("name", ["sparse_3d", "past_block_3d", "seven_7d", "big_seven_7d"])
def test_table_rows_misaligned(name):
    """Rows of four and eight columns that start 4 bytes past a multiple of 16."""
    from paper_1904_08755_amd import gsc, regions
    c = torch.from_numpy(GRID_ROWS[name]).to(DEV)
    c1 = _offset_copy(c, 1)
    assert c.data_ptr() % 16 == 0 and c1.data_ptr() % 16 == 4
    offs = regions.hypercross(3, c.shape[1] - 1)
    out, table = gsc.gsc_coords_stride(c, 2)
    out1, table1 = gsc.gsc_coords_stride(c1, 2)
    assert torch.equal(out, out1)
    for t, t1, u in ((gsc.gsc_coords_build(c), gsc.gsc_coords_build(c1), c), (table, table1, out)):
        m, m1 = gsc.gsc_kernel_map(t, u, offs), gsc.gsc_kernel_map(t1, _offset_copy(u, 1), offs)
        assert m.n_pairs >= len(u) and torch.equal(m.in_idx, m1.in_idx) and torch.equal(m.out_idx, m1.out_idx)


def _sorted_pairs(src, dst, offs):
    """[(input rows, output rows)] per offset by search of the sorted packed rows."""
    lo = torch.minimum(src.amin(0), dst.amin(0)).long() - 8
    ext = torch.maximum(src.amax(0), dst.amax(0)).long() + 9 - lo

    def pack(r):
        key = torch.zeros(len(r), dtype=torch.int64, device=r.device)
        for d in range(r.shape[1]):
            key = key * ext[d] + (r[:, d].long() - lo[d])
        return key

    keys, order = pack(src).sort()
    out = []
    for o in np.asarray(offs):
        q = pack(dst + torch.tensor([0, *o.tolist()], dtype=torch.int32, device=dst.device))
        at = torch.searchsorted(keys, q).clamp(max=len(keys) - 1)
        hit = (keys[at] == q).nonzero()[:, 0]
        out.append((order[at[hit]], hit))
    return out


# hashed maps on both sides of the row count from which a row range's blocks run one after another; blocks of 7, 8
# and 9 offsets (batches of 4 and 5), equal and unequal (8 + 8 + 8 + 5, 5 + 5)
@pytest.mark.parametrize("region", ["cross3", "cube2", "plane9", "cube3", "list29", "list10"])
@pytest.mark.parametrize("n", [200000, 200001])
def test_hashed_map_row_order(n, region, monkeypatch):
    from paper_1904_08755_amd import gsc, regions
    monkeypatch.setenv("GSC_TABLE_CAP_LIMIT", str(1 << 40))
    cube = regions.hypercube(3, 3)
    offs = {"cross3": regions.hypercross(3, 3), "cube2": regions.hypercube(2, 3), "plane9": cube[9:18], "cube3": cube,
            "list29": np.concatenate([cube, [[2, 0, 0], [0, -3, 1]]]).astype(np.int32), "list10": cube[:10]}[region]
    c = torch.from_numpy(np.ascontiguousarray(_rows(n, n, 3, 80))).to(DEV)
    assert len(c) == n
    km = gsc.gsc_kernel_map(gsc.gsc_coords_build(c), c, offs)
    seg = km.seg.tolist()
    for k, (i, o) in enumerate(_sorted_pairs(c, c, offs)):
        assert torch.equal(km.in_idx[seg[k]:seg[k + 1]].long(), i)
        assert torch.equal(km.out_idx[seg[k]:seg[k + 1]].long(), o)


@pytest.mark.parametrize("form", ["any", "hash"])
def test_table_forms_duplicates(form, monkeypatch):
    from paper_1904_08755_amd import gsc
    if form == "hash":
        monkeypatch.setenv("GSC_TABLE_CAP_LIMIT", str(1 << 40))
    c = torch.from_numpy(np.concatenate([GRID_ROWS["sparse_3d"], GRID_ROWS["sparse_3d"][500:501]])).to(DEV)
    with pytest.raises(gsc.GscError) as e:
        gsc.gsc_coords_build(c)
    assert e.value.code == gsc.GSC_EDUP


def _most_cells(n):
    """Cells of the largest grid over n rows, as table_layout.h sizes it."""
    cap = 64
    while cap < 4 * n:
        cap *= 2
    up16 = lambda b: (b + 15) // 16 * 16
    boxes = min(max((n + 1023) // 1024, 1), 256)
    room = 16 * cap - up16(4 * n) - up16(boxes * 33 * 4)
    return 4 * (min(18432 * 8 if n <= 3072 else 48 * n, room, 2**29) // 16 * 16)


# the last grid and the first box that is hashed, in the one-block build (1,200 rows: the table's room for words;
# 3,072 rows: all the words that LDS holds) and in the larger one (192 cells a row)
@pytest.mark.parametrize("n,cells", [(1200, 504_000), (3072, 589_824), (3073, 590_016), (6000, 1_152_000)])
@pytest.mark.parametrize("shape", ["line", "box"])
def test_grid_limit_of_cells(n, cells, shape):
    from paper_1904_08755_amd import gsc, regions
    assert cells == _most_cells(n)
    z = next(d for d in (64, 16, 4) if cells % d == 0)
    y = next(d for d in range(96, 0, -1) if cells // z % d == 0)
    for extra in (0, 1):
        # a line of any number of cells; a box of `cells`, or with one more layer
        ext = [cells + extra] if shape == "line" else [cells // z // y + extra, y, z]
        rng = np.random.default_rng(n + extra)
        last = int(np.prod(ext)) - 1
        flat = np.sort(np.concatenate([[0, last], 1 + rng.choice(last - 1, n - 2, replace=False)]))
        host = np.stack([0 * flat, *np.unravel_index(flat, ext)], 1).astype(np.int32)
        c = torch.from_numpy(host).to(DEV)
        table = gsc.gsc_coords_build(c)
        assert table[:4].cpu().numpy().tobytes() == (b"GSCT" if extra else b"GSCG")
        offs = regions.hypercube(3, len(ext))
        km = gsc.gsc_kernel_map(table, c, offs)
        seg = km.seg.tolist()
        for k, (i, o) in enumerate(_sorted_pairs(c, c, offs)):
            assert torch.equal(km.in_idx[seg[k]:seg[k + 1]].long(), i)
            assert torch.equal(km.out_idx[seg[k]:seg[k + 1]].long(), o)


def test_grid_cell_numbers_fit():
    """A box of just over 2^32 cells at 128 cells a row: rows whose cells agree
    in their low 32 bits are different rows."""
    from paper_1904_08755_amd import gsc
    i = torch.arange((1 << 25) + 100, dtype=torch.int64, device=DEV)
    cell = i * 128 + (i & 127)
    c = torch.stack([torch.zeros_like(i), cell >> 16, cell & 65535], 1).to(torch.int32)
    km = gsc.gsc_kernel_map(gsc.gsc_coords_build(c), c, np.zeros((1, 2), np.int32))
    assert torch.equal(km.in_idx.long(), i) and torch.equal(km.out_idx.long(), i)


@pytest.mark.parametrize("n,K", [(300, 2187), (300, 1024), (64 * 65536, 2), (64 * 65536 + 1, 2), (64 * 8192, 2),
                                 (64 * 8192 + 1, 2)])
def test_kernel_map_scan_limits(n, K):
    """Offsets and groups on both sides of the limits of the per-offset scan:
    rows on a line, offsets along it, so offset s pairs row j with j + s."""
    from paper_1904_08755_amd import gsc
    x = torch.arange(n, dtype=torch.int32, device=DEV)
    c = torch.stack([torch.zeros_like(x), x], 1).contiguous()
    o = np.arange(K)[:, None].astype(np.int32) * (1 if K > 2 else 70001)
    km = gsc.gsc_kernel_map(gsc.gsc_coords_build(c), c, o)
    seg = np.concatenate([[0], np.cumsum(np.maximum(n - o[:, 0].astype(np.int64), 0))])
    assert (km.seg.cpu().numpy() == seg).all() and km.n_pairs == seg[-1]
    want_o = torch.cat([x[:max(n - int(s), 0)] for s in o[:, 0]])
    want_i = torch.cat([x[int(s):] for s in o[:, 0]])
    assert torch.equal(km.out_idx, want_o) and torch.equal(km.in_idx, want_i)
    G = gsc.gsc_kmap_groups(n)
    k = K - 1
    assert km.gidx[k * G].item() == seg[k] and km.gidx[-1].item() == seg[-1]
    assert km.gidx[(k - 1) * G + G // 2].item() == seg[k - 1] + min(64 * (G // 2), seg[k] - seg[k - 1])
    if n > 1000:
        with pytest.raises(gsc.GscError) as e:
            gsc.gsc_kernel_map(gsc.gsc_coords_build(c), c, o, cap_pairs=int(seg[-1]) - 1)
        assert e.value.code == gsc.GSC_ESHORT


@pytest.mark.parametrize("form", ["any", "hash"])
@pytest.mark.parametrize("K", [9 * 65536 + 1, 7**7])
def test_kernel_map_many_offsets(K, form, monkeypatch):
    """More offsets than nine for each of the blocks that a launch's second dimension takes."""
    from paper_1904_08755_amd import gsc
    if form == "hash":
        monkeypatch.setenv("GSC_TABLE_CAP_LIMIT", str(1 << 40))
    c = torch.tensor([[0, 5], [0, 3], [0, 4]], dtype=torch.int32, device=DEV)
    o = (np.arange(K, dtype=np.int64) - (K - 2)).astype(np.int32)[:, None]   # ..., 0, 1 at the end
    km = gsc.gsc_kernel_map(gsc.gsc_coords_build(c), c, o, cap_pairs=16)
    want = {-2: [(1, 0)], -1: [(2, 0), (1, 2)], 0: [(0, 0), (1, 1), (2, 2)], 1: [(2, 1), (0, 2)]}
    pairs = [p for s in sorted(want) for p in want[s]]
    assert list(zip(km.in_idx.tolist(), km.out_idx.tolist())) == pairs
    seg = km.seg.cpu().numpy()
    assert (seg[:K - 3] == 0).all() and seg[K - 3:].tolist() == [1, 3, 6, 8]


@pytest.mark.parametrize("form", ["any", "hash"])
@pytest.mark.parametrize("n", [1, 200, 3072, 3073, 9000])
def test_quantize_sizes(n, form, monkeypatch):
    """Voxels, first points, labels and the inverse map by numpy, on both sides
    of the points that one block takes; unsorted points."""
    from paper_1904_08755_amd import gsc
    if form == "hash":
        monkeypatch.setenv("GSC_TABLE_CAP_LIMIT", str(1 << 40))
    rng = np.random.default_rng(n)
    pts = (rng.integers(-40, 41, (n, 3)) * 0.125 + 0.0625).astype(np.float32)   # exact quotients at 0.25
    batch = rng.integers(0, 3, n).astype(np.int32)
    labels = rng.integers(0, 2, n).astype(np.int32)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    q = gsc.gsc_quantize(dev(pts), 0.25, dev(batch), dev(labels), ignore_label=-7)
    rows = np.concatenate([batch[:, None], np.floor(pts / np.float32(0.25)).astype(np.int32)], 1)
    first, inverse = {}, []
    for i, r in enumerate(map(tuple, rows.tolist())):
        inverse.append(first.setdefault(r, (len(first), i))[0])
    rep = [i for _, i in first.values()]
    same = [set() for _ in first]
    for i, v in enumerate(inverse):
        same[v].add(int(labels[i]))
    assert q.coords.cpu().tolist() == [list(r) for r in first]
    assert q.rep.cpu().tolist() == rep and q.inverse.cpu().tolist() == inverse
    assert q.labels.cpu().tolist() == [s.pop() if len(s) == 1 else -7 for s in same]
    km = gsc.gsc_kernel_map(q.table, q.coords, np.zeros((1, 3), np.int32))
    assert km.in_idx.cpu().tolist() == list(range(len(first)))
    q2 = gsc.gsc_quantize(dev(pts), 0.25, dev(batch))
    assert torch.equal(q2.coords, q.coords) and torch.equal(q2.inverse, q.inverse) and q2.labels is None


def _first_rows(rows):
    """(distinct rows in the order of their first ones, first rows, row of each) by numpy."""
    _, first, inv = np.unique(rows, axis=0, return_index=True, return_inverse=True)
    order = np.argsort(first)
    place = np.empty_like(order)
    place[order] = np.arange(len(order))
    return rows[first[order]], first[order], place[inv.reshape(-1)]


# rows merged per block before they reach the table: on both sides of the sizes of its two block widths and of the
# most rows a stride's cell may hold unmerged (128); few cells with many rows each, shuffled, and distinct ones
@pytest.mark.parametrize("n", [4000, 65535, 65536])
@pytest.mark.parametrize("stride", [(4, 4, 8), (4, 4, 9), (16, 16, 16), (1, 1, 200), (1 << 20, 1, 1)])
def test_stride_rows_per_cell(n, stride):
    from paper_1904_08755_amd import gsc
    rows = _rows(n, n, 3, 60)
    out, table = gsc.gsc_coords_stride(torch.from_numpy(rows).to(DEV), stride)
    want, _, _ = _first_rows(np.concatenate([rows[:, :1], rows[:, 1:] // stride * stride], 1))
    assert np.array_equal(out.cpu().numpy(), want)
    up = gsc.gsc_kernel_map(table, out, np.zeros((1, 3), np.int32))
    assert torch.equal(up.in_idx.long(), torch.arange(len(want), device=DEV))


@pytest.mark.parametrize("n", [4000, 65535, 65536, 200000])
def test_quantize_hot_cells(n):
    """Points most of which share a few voxels, in no order."""
    from paper_1904_08755_amd import gsc
    rng = np.random.default_rng(n)
    pts = np.concatenate([rng.normal(0, 0.05, (n - n // 4, 3)), rng.uniform(-4, 4, (n // 4, 3))]).astype(np.float32)
    pts = np.ascontiguousarray(rng.permutation(pts))
    labels = (rng.random(n) < 1e-3).astype(np.int32)
    q = gsc.gsc_quantize(torch.from_numpy(pts).to(DEV), 0.125, None, torch.from_numpy(labels).to(DEV), ignore_label=9)
    rows = np.concatenate([np.zeros((n, 1), np.int32), np.floor(pts.astype(np.float64) / 0.125).astype(np.int32)], 1)
    want, first, inverse = _first_rows(rows)
    assert np.array_equal(q.coords.cpu().numpy(), want) and np.array_equal(q.rep.cpu().numpy(), first)
    assert np.array_equal(q.inverse.cpu().numpy(), inverse)
    ones, count = np.bincount(inverse, labels), np.bincount(inverse)
    assert np.array_equal(q.labels.cpu().numpy(), np.where(ones == 0, 0, np.where(ones == count, 1, 9)))


@pytest.mark.parametrize("n,by", [(3000, 0), (9000, 0), (9000, 40), (9000, -40)])
def test_quantize_labels_in_place(n, by):
    """out_labels may be the array of the points' labels, or overlap it."""
    from paper_1904_08755_amd import gsc
    rng = np.random.default_rng(n)
    dev = lambda a: torch.from_numpy(a).to(DEV)
    pts, labels = dev((rng.random((n, 3)) * 6).astype(np.float32)), dev(rng.integers(0, 2, n).astype(np.int32))
    want = gsc.gsc_quantize(pts, 0.5, None, labels, ignore_label=-7)
    L, P, c = gsc.lib(), gsc._ptr, gsc.ctypes
    buf = torch.empty(n + 100, dtype=torch.int32, device=DEV)
    inp, out = buf[50:50 + n], buf[50 + by:50 + by + n]
    inp.copy_(labels)
    rows, rep = (torch.empty(s, dtype=torch.int32, device=DEV) for s in ((n, 4), (n,)))
    table, ws = gsc._ws(gsc.gsc_table_bytes(n), DEV), gsc._ws(L.gsc_quantize_ws_bytes(n, 3), DEV)
    m = c.c_int64(0)
    gsc._check(L.gsc_quantize(P(pts), None, n, 3, (c.c_float * 3)(0.5, 0.5, 0.5), P(inp), -7, P(rows), c.byref(m),
                              P(rep), P(out), None, P(table), table.numel(), P(ws), ws.numel(), gsc._stream(None)))
    assert m.value == len(want.coords) and torch.equal(rows[:m.value], want.coords)
    assert torch.equal(out[:m.value], want.labels) and (want.labels == -7).any() and (want.labels >= 0).any()


# --------------------------------------------------------------------------- #
# block plans at the edges of the sort's tiles and the counted block tiles
# --------------------------------------------------------------------------- #
@pytest.mark.parametrize("K", [1, 8, 10, 11, 27, 32, 81])
@pytest.mark.parametrize("n", [1, 15, 17, 1023, 1025, 2049, 4097, 16385])
def test_plan_sizes(n, K):
    _plan_case(n, K)


@pytest.mark.parametrize("n", [98305, 99999, 100000, 102401])   # the later passes' tiles grow at 100,000 rows
def test_plan_tile_rule(n):
    _plan_case(n, 27)


def _plan_case(n, K):
    """The plan of a synthetic dense form: row order, block masks, item bases and
    items, with rows of equal keys in row order (random masks of few values)."""
    from paper_1904_08755_amd import gsc
    g = np.random.default_rng(n * 100 + K)
    has = g.random((K, n)) < g.choice([0.02, 0.5, 0.9], (1, n))
    nbr = np.where(has, g.integers(0, n, (K, n)), -1).astype(np.int32)
    km = gsc.KernelMap(None, None, torch.zeros(K + 1, dtype=torch.int64, device=DEV), None, None, n,
                       np.zeros((K, 3), np.int32), 0, torch.from_numpy(nbr).to(DEV))
    bufs = gsc.PlanBuffers(n, K, DEV)
    plan = gsc.gsc_conv_plan(km, bufs).plan
    gsc.gsc_conv_plan_status(km, bufs)
    R, nb = gsc.gsc_plan_ranges(K), gsc.gsc_plan_blocks(n)
    S = -(-K // R)
    perm, bmask = plan.perm.cpu().numpy(), plan.bmask.cpu().numpy().view(np.uint32)
    ibase, items = plan.ibase.cpu().numpy(), plan.items.cpu().numpy()
    for r in range(R):
        k0, kr = r * S, min(S, K - r * S)
        mask = (has[k0:k0 + kr].astype(np.int64) << np.arange(kr)[:, None]).sum(0)
        pbits = min(10 * -(-kr // 10) - kr, 32 - kr, 6)
        key = np.minimum(has[k0:k0 + kr].sum(0), 2 ** pbits - 1) << kr | mask
        want = np.argsort(key, kind="stable")
        assert np.array_equal(perm[r * n:(r + 1) * n], want)
        pad = np.zeros(nb * 16, np.int64)
        pad[:n] = mask[want]
        union = np.bitwise_or.reduce(pad.reshape(nb, 16), 1)
        assert np.array_equal(bmask[r * nb:(r + 1) * nb], union)
        base = np.concatenate([[0], np.cumsum([bin(u).count("1") for u in union.tolist()])])
        assert np.array_equal(ibase[r * (nb + 1):(r + 1) * (nb + 1)], base)
        got = items[k0 * nb:k0 * nb + base[-1]]
        rows = np.full(nb * 16, -1)
        rows[:n] = want
        at = 0
        for b, u in enumerate(union.tolist()):
            for k in range(kr):
                if u >> k & 1:
                    blk = rows[16 * b:16 * b + 16]
                    assert np.array_equal(got[at], np.where(blk >= 0, nbr[k0 + k][blk], -1))
                    at += 1


# --------------------------------------------------------------------------- #
# float32 row form with 32 or 64 channels on both sides
# --------------------------------------------------------------------------- #
def _conv64(X, W, km):
    Y = torch.zeros((km.n_out, W.shape[2]), dtype=torch.float64, device=DEV)
    seg = km.seg.tolist()
    for k in range(W.shape[0]):
        i, o = km.in_idx[seg[k]:seg[k + 1]].long(), km.out_idx[seg[k]:seg[k + 1]].long()
        Y[o] += X[i].double() @ W[k].double()
    return Y


# rows: remainders of a tile of 128, a tile, several; density: no pairs but the centre's to all offsets
# full; offsets up to the 64 of a lane each
@pytest.mark.parametrize("ca,cb", [(32, 32), (32, 64), (64, 32), (64, 64)])
@pytest.mark.parametrize("n,span,region", [(1, 1, "cube3"), (63, 4, "cube3"), (128, 6, "cube3"), (129, 30, "cube3"),
                                           (1000, 10, "cube3"), (1728, 12, "cube3"), (700, 9, "list64"),
                                           (5, 2000, "one")])
def test_conv_f32_wide_rows(n, span, region, ca, cb):
    from paper_1904_08755_amd import gsc, regions
    offs = {"cube3": regions.hypercube(3, 3), "one": np.zeros((1, 3), np.int32),
            "list64": regions.hypercube(4, 3)}[region]
    host = np.ascontiguousarray(_rows(n, n, 3, span, batch=1))
    c = torch.from_numpy(host).to(DEV)
    n, K = len(host), len(offs)
    km = gsc.gsc_kernel_map(gsc.gsc_coords_build(c), c, offs)
    g = torch.Generator(DEV).manual_seed(n + ca)
    X = torch.randn((n, ca), generator=g, device=DEV)
    W = torch.randn((K, ca, cb), generator=g, device=DEV) / (K * ca) ** 0.5
    Y = gsc.gsc_sparse_conv_fwd(X, W, km)
    ref = _conv64(X, W, km)
    mag = _conv64(X.abs(), W.abs(), km)
    bound = (ca + K + 2) * 2.0 ** -24          # products and additions of a sum, each half an ulp
    assert ((Y.double() - ref).abs() <= mag * bound).all()
    assert torch.equal(Y, gsc.gsc_sparse_conv_fwd(X, W, km))
    scale, shift = 0.5 + torch.rand(cb, generator=g, device=DEV), torch.randn(cb, generator=g, device=DEV)
    A = gsc.gsc_sparse_conv_fwd_affine(X, W, km, scale, shift, relu=True)
    want = torch.clamp(Y.double() * scale.double() + shift.double(), min=0)
    assert ((A.double() - want).abs() <= want.abs() * 2.0 ** -23 + 1e-30).all()
    # input gradient: the role-reversed map's products with W^T
    dY = torch.randn((n, ca), generator=g, device=DEV)
    V = torch.randn((K, cb, ca), generator=g, device=DEV) / (K * ca) ** 0.5
    tm = gsc.gsc_kernel_map_transpose(km, n)
    dX, _ = gsc.gsc_sparse_conv_bwd(torch.zeros((n, cb), device=DEV), V, dY, km, tm, np.arange(K), need_dw=False)
    T = V.transpose(1, 2).contiguous()
    tk = type(km)(tm.in_idx, tm.out_idx, tm.seg, tm.gidx, km.n_pairs, n, tm.offsets)
    assert ((dX.double() - _conv64(dY, T, tk)).abs() <= _conv64(dY.abs(), T.abs(), tk) * bound).all()


# features, weights, gradients and outputs that start 4 bytes past a multiple of 16
@pytest.mark.parametrize("ca,cb", [(16, 32), (32, 32), (64, 64)])
def test_conv_f32_misaligned(ca, cb):
    from paper_1904_08755_amd import gsc, regions
    offs = regions.hypercube(3, 3)
    c = torch.from_numpy(_rows(5, 300, 3, 8, batch=1)).to(DEV)
    n, K = len(c), len(offs)
    km = gsc.gsc_kernel_map(gsc.gsc_coords_build(c), c, offs)
    g = torch.Generator(DEV).manual_seed(ca + cb)
    X, dY = torch.randn((n, ca), generator=g, device=DEV), torch.randn((n, cb), generator=g, device=DEV)
    W = torch.randn((K, ca, cb), generator=g, device=DEV)
    sel = gsc.negation_permutation(offs)
    Y, (dX, dW) = gsc.gsc_sparse_conv_fwd(X, W, km), gsc.gsc_sparse_conv_bwd(X, W, dY, km, km, sel)
    X1, W1, dY1 = (_offset_copy(t, 1) for t in (X, W, dY))
    assert X1.data_ptr() % 16 == W1.data_ptr() % 16 == dY1.data_ptr() % 16 == 4
    Y1, dX1 = _offset_copy(torch.full_like(Y, 7.0), 1), _offset_copy(torch.full_like(dX, 7.0), 1)
    gsc.gsc_sparse_conv_fwd(X1, W1, km, Y=Y1)
    dW1 = gsc.gsc_sparse_conv_bwd(X1, W1, dY1, km, km, sel, dX=dX1)[1]
    assert torch.equal(Y1, Y) and torch.equal(dX1, dX) and torch.equal(dW1, dW)


# pairs of an offset: none, one, about a step of 32, about the ring's four steps, about a work item (1024 or
# 2048 pairs) and several; rows out of range on either side add nothing; more offsets than the items are
# ordered over (128); "bf16+1": rows that start 2 bytes past a multiple of 16
@pytest.mark.parametrize("ci,co,rep,dtype", [(64, 64, 1, "bf16"), (64, 64, 1, "bf16+1"), (64, 128, 1, "bf16+1"),
                                             (64, 64, 9, "bf16"), (64, 128, 1, "bf16"),
                                             (64, 64, 0, "bf16"), (64, 128, 0, "bf16"), (128, 128, 0, "bf16"),
                                             (64, 64, 0, "f32"), (32, 32, 1, "f32"), (3, 16, 0, "f32"),
                                             (128, 64, 1, "bf16"), (128, 128, 1, "bf16"), (256, 256, 1, "bf16")] +
                         # the same with several tiles of 64 x 64: halved items, and items of full size
                         [(96, 64, 1, "f32"), (96, 96, 1, "f32"), (130, 70, 1, "f32"), (96, 96, 0, "f32"),
                          (96, 96, 1, "bf16")] +
                         [(a, b, 1, t) for t in ("f32", "bf16")   # the kernel for any width: 16 and more on a side
                          for a, b in ((1, 1), (3, 16), (16, 17), (17, 16), (24, 48), (70, 5))])
def test_dw_pairs(ci, co, rep, dtype):
    from paper_1904_08755_amd import gsc, regions
    sizes = [0, 1, 31, 32, 33, 96, 128, 129, 1024, 1025, 2047, 2048, 2049, 4300, 0] * max(rep, 1)
    if rep == 0:   # enough pairs for items of full size (1024 or 2048)
        sizes += [256 * (1024 if ci * co <= 64 * 64 else 2048) + 7]
    K, n_in, n_out = len(sizes), 900, 900
    host = np.ascontiguousarray(_rows(3, 50, 3, 6, batch=1))
    c = torch.from_numpy(host).to(DEV)
    km = gsc.gsc_kernel_map(gsc.gsc_coords_build(c), c, regions.hypercube(3, 3))
    g = torch.Generator(DEV).manual_seed(ci + co)
    P = sum(sizes)
    ii = torch.randint(0, n_in, (P,), generator=g, device=DEV, dtype=torch.int32)
    oi = torch.randint(0, n_out, (P,), generator=g, device=DEV, dtype=torch.int32)
    seg = torch.tensor([0] + list(np.cumsum(sizes)), dtype=torch.int64, device=DEV)
    bad = torch.rand(P, generator=g, device=DEV) < 0.02
    bad[seg[2]:seg[4]] = False
    in_bad, out_bad = ii.clone(), oi.clone()
    in_bad[bad] = torch.tensor([-1, n_in], dtype=torch.int32, device=DEV)[torch.arange(int(bad.sum())) % 2]
    out_bad[bad.roll(1)] = n_out
    skip = bad | bad.roll(1)
    m = type(km)(in_bad, out_bad, seg, km.gidx, P, n_out, np.zeros((K, 3), np.int32), n_bound=P)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    shift = int(dtype.endswith("+1"))
    X = _offset_copy(torch.randn((n_in, ci), generator=g, device=DEV).to(dt), shift)
    dY = _offset_copy(torch.randn((n_out, co), generator=g, device=DEV).to(dt), shift)
    W = torch.zeros((K, ci, co), device=DEV, dtype=dt)
    run = lambda: gsc.gsc_sparse_conv_bwd(X, W, dY, m, m, np.arange(K), need_dx=False)[1]
    dW = run()
    for k in range(K):
        a, b = int(seg[k]), int(seg[k + 1])
        keep = ~skip[a:b]
        x, y = X[ii[a:b].long()[keep]].double(), dY[oi[a:b].long()[keep]].double()
        # a product is half an ulp off at most (none in bf16), an addition too, or one where the matrix unit
        # cuts off
        assert ((dW[k].double() - x.t() @ y).abs() <= (x.abs().t() @ y.abs()) * (b - a + 2) * 2.0 ** -23).all()
    assert torch.equal(dW, run())
